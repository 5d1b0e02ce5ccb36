// ct_rns_plan.h -- host side of the products through residues (ct_rns.h):
// which layers take them, how the layers of a call share the scratch, and the
// tables of the launches.
#pragma once

#include <algorithm>
#include <cstring>
#include <vector>

#include "ct_rns.h"

namespace ct {

// Most scratch for residue planes and residues by default.  A call whose layers
// need more runs them in groups, one after the other: twelve encoders took 7.9
// ms in groups of half a GiB, 7.5 ms of one GiB and of sixteen.  Just below 2
// GiB, where hipMalloc takes 70 us (330 us from 2 GiB on).
constexpr int64_t RNS_SCRATCH_BYTES = CT_SCRATCH_BYTES;
constexpr int RNS_MAX_CHUNKS = 64;

// What the cost of a layer's products depends on: nl left and nr right
// operands, outs products of segs segments each.
struct RnsShape {
    int64_t M = 0, K = 0, N = 0;
    int nl = 0, nr = 0, outs = 0, segs = 2;
    double rate = 1.0e5;  // operand elements converted and read back per microsecond, beyond the digit path's
    double refetch = 0;    // bytes that the conversion reads and the digit path does not
    int64_t res_bytes() const { return (int64_t)outs * RNS_N * rns_blocks(M) * rns_blocks(N) * 1024; }
    int64_t bytes(int64_t kc) const {
        return res_bytes() + RNS_N * (nl * rns_plane_bytes(M, kc) + nr * rns_plane_bytes(N, kc));
    }
    int64_t chunk_len(int c) const { return ((K + c - 1) / c + RNS_BK - 1) / RNS_BK * RNS_BK; }
    // fewest chunks of K whose planes fit beside the residues in cap bytes; 0: none
    int chunks(int64_t cap) const {
        if (segs * K > RNS_MAX_TERMS) return 0;
        for (int c = 1; c <= RNS_MAX_CHUNKS; c++)  // some c leave their last chunks empty: the length is rounded up
            if ((c - 1) * chunk_len(c) < K && bytes(chunk_len(c)) <= cap) return c;
        return 0;
    }
    double macs() const { return (double)outs * segs * M * K * N; }
    double digits_us() const { return macs() * (136 / 1.2e9); }
    // Time the residue path saves against the digit path, in microseconds:
    // 136 against 36 matrix products per multiply-add (1.2e15 digit and 0.9e15
    // residue products a second), against the 20 bytes more per operand element
    // and the residues of the outputs.  Fitted to 78 single layers (2 to 4
    // parties, both protocols) and 60 batches timed on either path.  With two
    // parties and CompactTag a layer of 2048^3 takes 2061 us by residues and 3661
    // by digits, 256 x 768 x 768 201 and 211, 64 x 4096 x 4096 1438 and 1224; an
    // encoder in SPDZ2k 1152 and 1191, which rns_choose leaves with digits (the
    // estimate, 76 of 821 us of digit products, is below its tenth).  The sign
    // changes near M N / (M + N) = 80.
    double saves_us() const {
        const double pm = 32.0 * rns_blocks(M), pn = 32.0 * rns_blocks(N);
        return digits_us() - (double)outs * segs * pm * K * pn * (36 / 0.9e9) - (nl * pm + nr * pn) * K / rate - refetch / 5.5e6 -
               outs * pm * pn / 5.3e4;
    }
};

// The products of the online phase of a layer with n parties: E [B]_p +
// ([A]_p or A_0 + E) U, in SPDZ2k also E [tB]_p + ([tA]_p + [Delta]_p E) U.
inline RnsShape rns_online_shape(const ct_layer_desc &d, int np, bool compact) {
    RnsShape s;
    s.M = d.M; s.K = d.K; s.N = d.N;
    s.nl = s.nr = compact ? np + 1 : 2 * np + 1;
    s.outs = compact ? np : 2 * np;
    if (np > 2 && compact) s.rate = 0.85e5;  // an encoder of three parties: 1314 us by digits, 1340 by residues
    if (np == 2 && compact) {
        const bool cm = CT_COMPRESS_ALONG_M(d.M, d.N, d.compress);
        // one pass opens, compresses and converts, but along M only the digit path's (595 us for a drawn batch of
        // such layers by digits, 650 by residues where 1.0e5 sent them there)
        if (d.conv_c == 0) s.rate = cm ? 0.76e5 : 1.38e5;
        // only layers compressed along M open U apart from its conversion here and together with it there
        if (d.conv_c == 0 && cm) s.refetch = 48.0 * d.K * d.N;
    }
    return s;
}

// Which of the layers of a call (those with N > SKINNY_MAX_N) take the residue
// path.  Each path brings launches of its own, tens of microseconds on a small
// call, so a few layers on the slower side follow the others (up to 100 us of
// digit products), and a call that would gain less than 18 us, or less than
// 80 us and keep both paths for it, stays with digits.  So does one that would
// gain little for its size: a fifth below 300 us of digit products (seven
// layers with 200 us of them took 457 us by digits and 476 by residues, at 17%),
// a tenth above; and a quarter of any beside skinny layers, whose pass, bound by
// HBM, overlaps with the digit products but not with the conversions (1176 us
// and 1217).
inline std::vector<char> rns_choose(const std::vector<RnsShape> &s, int64_t cap, bool skinny) {
    std::vector<char> take(s.size(), 0);
    double gain = 0, taken_us = 0, rest_us = 0, rest_loss = 0;
    bool others = false, able = true;
    for (size_t i = 0; i < s.size(); i++) {
        const double save = s[i].saves_us();
        const bool can = s[i].chunks(cap) > 0;
        if (can && save > 4) {
            take[i] = 1;
            gain += save;
            taken_us += s[i].digits_us();
        } else {
            others = true;
            able &= can;
            rest_us += s[i].digits_us();
            rest_loss -= save;
        }
    }
    if (others && able && rest_us < 100 && gain > rest_loss) {
        take.assign(s.size(), 1);
        gain -= rest_loss;
        taken_us += rest_us;
        others = false;
    }
    const double part = skinny ? 0.25 : taken_us < 300 ? 0.2 : 0.1;
    if (gain < (others ? 80 : 18) || gain < part * taken_us) take.assign(s.size(), 0);
    return take;
}

struct RnsOperand {
    const u128 *src;
    int side;
};
struct RnsProduct {
    int outs, L0, L1, L2, R0, R1, R2;  // operand numbers; L1 < 0: one segment
    const u128 *base[2];
    u128 *out[2];
};
// A layer's products over its operands.
struct RnsLayer {
    RnsShape shape;
    const ConvGeom *cv = nullptr;
    std::vector<RnsOperand> ops;
    std::vector<RnsProduct> prods;
    int open = -1;  // >= 0: index of the layer, whose openings write the planes (operands E, A_0 + E, [A]_1, [B]_0,
                    // [B]_1, U, in SPDZ2k then [tA]_p + [Delta]_p E, [tB]_p); -1: every operand is converted
                    // from memory
    int Kc = 0;
    uint8_t *at = nullptr;  // residues
};

// Launches of one group of layers: per K chunk (one, or the chunks of a layer
// that is by itself) the openings, conversions and products, then one
// reconstruction.
struct RnsGroup {
    int job0 = 0, prob0 = 0, open0 = 0;            // first table entries
    int chunks = 1;
    bool whole = false;                            // takes the whole scratch, not one half
    int half = 0;
    int nopen = 0, left = 0, right = 0;            // openings and their workgroups
    int njobs = 0, wgs = 0;                        // conversions
    int n2 = 0, blocks2 = 0, n1 = 0, blocks1 = 0;  // problems of two products and of one, workgroups per XCD
    int fold_items = 0;
};
struct RnsPlan {
    int njobs = 0, nprobs = 0, nopen = 0;      // table entries of all groups
    std::vector<RnsGroup> groups;
};

inline int64_t rns_align(int64_t b) { return (b + 4095) & ~(int64_t)4095; }

// Cuts shapes (in the given order) into consecutive groups: group[i] receives
// the number of shape i's group.  Groups take the two halves of the scratch in
// turn, so that one group's openings and other passes (bound by HBM) can run
// beside the products of another: RNS_GROUPS groups, none below
// RNS_GROUP_MIN bytes, where the ends of the launches cost more than the
// overlap gives.  A shape larger than a half has the whole scratch, and its
// group, to itself.
constexpr int RNS_GROUPS = 4;
constexpr int64_t RNS_GROUP_MIN = 1LL << 30;
inline int64_t rns_half(int64_t cap) { return cap / 2 & ~(int64_t)4095; }
inline void rns_groups(const std::vector<RnsShape> &s, int64_t cap, std::vector<int> &group) {
    int64_t total = 0, used = 0;
    for (const auto &r : s) total += rns_align(r.bytes(r.chunk_len(1)));
    const int64_t part = total <= RNS_GROUP_MIN ? cap : std::min(rns_half(cap), std::max(total / RNS_GROUPS, RNS_GROUP_MIN));
    int g = -1;
    bool alone = true;
    group.assign(s.size(), 0);
    for (size_t i = 0; i < s.size(); i++) {
        const int64_t b = rns_align(s[i].bytes(s[i].chunk_len(1)));
        if (alone || used + b > part) {
            g++;
            used = 0;
        }
        alone = b > part;
        used += b;
        group[i] = g;
    }
}

// Assigns scratch and fills the tables; the layers are sorted, large ones
// first (the last workgroups of a launch are then short).
inline void rns_plan(std::vector<RnsLayer> &ls, uint8_t *scratch, int64_t cap, RnsJob *jobs, RnsProb *probs, RnsOpen *opens,
                     RnsPlan &P) {
    P = RnsPlan();
    std::stable_sort(ls.begin(), ls.end(), [](const RnsLayer &a, const RnsLayer &b) {
        return a.shape.M * a.shape.K * a.shape.N > b.shape.M * b.shape.K * b.shape.N;
    });
    std::vector<RnsShape> shapes;
    std::vector<int> group;
    for (const auto &r : ls) shapes.push_back(r.shape);
    rns_groups(shapes, cap, group);
    int next = 0;
    for (size_t first = 0, last; first < ls.size(); first = last) {
        for (last = first; last < ls.size() && group[last] == group[first]; last++) {}
        RnsGroup G;
        G.job0 = P.njobs;
        G.prob0 = P.nprobs;
        G.open0 = P.nopen;
        G.chunks = ls[first].shape.chunks(cap);
        int64_t bytes = 0;
        for (size_t l = first; l < last; l++) bytes += rns_align(ls[l].shape.bytes(ls[l].shape.chunk_len(G.chunks)));
        G.whole = bytes > rns_half(cap);
        G.half = G.whole ? 0 : next++ & 1;
        int wg = 0, wg_left = 0, wg_right = 0;
        uint8_t *w = scratch + G.half * rns_half(cap);
        std::vector<std::vector<uint8_t *>> at(last - first);
        for (size_t l = first; l < last; l++) {
            RnsLayer &r = ls[l];
            const RnsShape &s = r.shape;
            r.Kc = (int)s.chunk_len(G.chunks);
            uint8_t *const begin = w;
            for (const auto &o : r.ops) {
                const int64_t major = o.side ? s.N : s.M, plane = rns_plane_bytes(major, r.Kc);
                if (r.open < 0) {
                    RnsJob j;
                    std::memset(&j, 0, sizeof(j));
                    j.src = o.src;
                    j.dst = w;
                    j.plane = plane;
                    j.rows = (int32_t)(o.side ? s.K : s.M);
                    j.cols = (int32_t)(o.side ? s.N : s.K);
                    j.side = o.side;
                    j.Kc = r.Kc;
                    j.kt = r.Kc / 32;
                    j.majb = (int32_t)rns_blocks(major);
                    j.wg_begin = wg;
                    j.wgs = o.side ? (j.majb + 3) / 4 * j.kt : j.majb * ((j.kt + 3) / 4);
                    if (o.side && r.cv) j.cv = *r.cv;
                    wg += j.wgs;
                    jobs[P.njobs++] = j;
                }
                at[l - first].push_back(w);
                w += RNS_N * plane;
            }
            if (r.open >= 0) {
                RnsOpen j;
                std::memset(&j, 0, sizeof(j));
                j.left = at[l - first][0];
                j.right = at[l - first][3];
                if (r.ops.size() > 6) {
                    j.left_tag = at[l - first][6];
                    j.right_tag = at[l - first][8];
                }
                j.planeL = rns_plane_bytes(s.M, r.Kc);
                j.planeR = rns_plane_bytes(s.N, r.Kc);
                j.layer = r.open;
                j.Kc = r.Kc;
                j.kt = r.Kc / 32;
                j.mb = (int32_t)rns_blocks(s.M);
                j.nb = (int32_t)rns_blocks(s.N);
                j.wg_left = wg_left;
                j.wg_right = wg_right;
                wg_left += j.kt * j.mb;
                wg_right += j.kt * ((j.nb + 3) / 4);
                opens[P.nopen++] = j;
            }
            r.at = w;
            w = begin + rns_align(s.bytes(r.Kc));
        }
        G.njobs = P.njobs - G.job0;
        G.wgs = wg;
        G.nopen = P.nopen - G.open0;
        G.left = wg_left;
        G.right = wg_right;
        // problems of two products first; per XCD the workgroups of 5 or 4 of
        // the 36 moduli, the larger share going where the launch has less so far
        for (int outs = 2; outs >= 1; outs--) {
            int64_t load[8] = {};
            int count = 0;
            for (size_t l = first; l < last; l++) {
                const RnsLayer &r = ls[l];
                const RnsShape &s = r.shape;
                uint8_t *res = r.at;
                for (const auto &pr : r.prods) {
                    uint8_t *mine = res;
                    res += (int64_t)pr.outs * RNS_N * rns_blocks(s.M) * rns_blocks(s.N) * 1024;
                    if (pr.outs != outs) continue;
                    RnsProb p;
                    std::memset(&p, 0, sizeof(p));
                    auto op = [&](int i) -> const uint8_t * { return i >= 0 ? at[l - first][i] : nullptr; };
                    p.L0 = op(pr.L0); p.L1 = op(pr.L1); p.L2 = op(pr.L2);
                    p.R0 = op(pr.R0); p.R1 = op(pr.R1); p.R2 = op(pr.R2);
                    p.res = mine;
                    for (int o = 0; o < pr.outs; o++) { p.base[o] = pr.base[o]; p.out[o] = pr.out[o]; }
                    p.planeL = rns_plane_bytes(s.M, r.Kc);
                    p.planeR = rns_plane_bytes(s.N, r.Kc);
                    p.M = (int32_t)s.M; p.N = (int32_t)s.N; p.K = (int32_t)s.K; p.Kc = r.Kc; p.kt = r.Kc / 32;
                    p.outs = pr.outs; p.segs = s.segs;
                    p.mb = (int32_t)rns_blocks(s.M); p.nb = (int32_t)rns_blocks(s.N);
                    p.tiles_m = (p.mb + RNS_TM / 32 - 1) / (RNS_TM / 32);
                    p.tiles_n = (p.nb + RNS_TN / 32 - 1) / (RNS_TN / 32);
                    p.fold_begin = G.fold_items;
                    G.fold_items += pr.outs * p.mb * p.nb;
                    p.rot = load[0] + load[1] + load[2] + load[3] <= load[4] + load[5] + load[6] + load[7] ? 0 : 4;
                    for (int x = 0; x < 8; x++) {
                        const int q0 = (x - p.rot) & 7;
                        p.begin[x] = (int32_t)load[x];
                        load[x] += (int64_t)((RNS_N - q0 + 7) / 8) * p.tiles_m * p.tiles_n;
                    }
                    probs[P.nprobs++] = p;
                    count++;
                }
            }
            const int most = (int)*std::max_element(load, load + 8);
            (outs == 2 ? G.n2 : G.n1) = count;
            (outs == 2 ? G.blocks2 : G.blocks1) = most;
        }
        P.groups.push_back(G);
    }
}

}  // namespace ct
