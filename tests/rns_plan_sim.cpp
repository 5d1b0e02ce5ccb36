// Host-only checks of the plan of the residue products (ct_rns_plan.h) on
// random batches, parties, protocols and scratch sizes: the scratch ranges of
// a group lie in its part of the scratch and do not meet, the chunks cover K,
// and the tables send every workgroup of a launch to one piece of work, every
// piece once, found the way the kernels find it.  Nothing is dereferenced.
// Prints one "ok ..." line with what was covered; exits non-zero on the first
// violated invariant.
#include <algorithm>
#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <random>
#include <set>
#include <vector>

#include "ct_rns_plan.h"

using namespace ct;

#define CHECK(c)                                                                   \
    do {                                                                           \
        if (!(c)) {                                                                \
            std::fprintf(stderr, "FAIL %s:%d: %s\n", __FILE__, __LINE__, #c);      \
            std::exit(1);                                                          \
        }                                                                          \
    } while (0)

struct Range {
    const uint8_t *begin, *end;
    bool operator<(const Range &o) const { return begin < o.begin; }
};

// A layer's operands and products as a call forms them: E, A_0 + E, [A]_1 ..,
// then [B]_p, U; in SPDZ2k the folded tag operands and [tB]_p.
static RnsLayer layer(const ct_layer_desc &d, int np, bool compact, int open, const ConvGeom *cv) {
    RnsLayer r;
    r.shape = rns_online_shape(d, np, compact);
    r.open = open;
    r.cv = cv;
    for (int i = 0; i <= np; i++) r.ops.push_back({nullptr, 0});
    for (int i = 0; i <= np; i++) r.ops.push_back({nullptr, 1});
    const int u = 2 * np + 1;
    auto pairs = [&](int left, int right) {
        for (int p = 0; p < np; p += 2) {
            const bool two = p + 1 < np;
            r.prods.push_back({two ? 2 : 1, 0, left + p, two ? left + p + 1 : -1, right + p, two ? right + p + 1 : -1, u, {}, {}});
        }
    };
    pairs(1, np + 1);
    if (!compact) {
        for (int i = 0; i < np; i++) r.ops.push_back({nullptr, 0});
        for (int i = 0; i < np; i++) r.ops.push_back({nullptr, 1});
        pairs(u + 1, u + 1 + np);
    }
    return r;
}

static int64_t groups_seen = 0, halves_seen = 0, chunked = 0, opened = 0, packed = 0;

static void check_batch(std::vector<RnsLayer> ls, int np, int64_t cap) {
    const int n = (int)ls.size();
    const std::vector<RnsLayer> before = ls;
    std::vector<RnsJob> jobs((4 * np + 2) * n);  // the sizes of a lane's tables
    std::vector<RnsProb> probs(2 * np * n);
    std::vector<RnsOpen> opens(n);
    uint8_t *const scratch = reinterpret_cast<uint8_t *>((uintptr_t)1 << 40);
    RnsPlan P;
    rns_plan(ls, scratch, cap, jobs.data(), probs.data(), opens.data(), P);
    CHECK(P.njobs <= (int)jobs.size() && P.nprobs <= (int)probs.size() && P.nopen <= n);
    size_t at = 0;  // layer of the sorted list
    int jobs_at = 0, probs_at = 0, opens_at = 0;
    for (const RnsGroup &G : P.groups) {
        CHECK(G.job0 == jobs_at && G.prob0 == probs_at && G.open0 == opens_at);
        jobs_at += G.njobs;
        probs_at += G.n2 + G.n1;
        opens_at += G.nopen;
        groups_seen++;
        halves_seen += !G.whole;
        chunked += G.chunks > 1;
        const uint8_t *const lo = scratch + G.half * rns_half(cap), *const hi = G.whole ? scratch + cap : lo + rns_half(cap);
        CHECK(!G.whole || G.half == 0);
        // the group's layers: those whose residues lie between its problems' first and last
        std::vector<Range> used;
        size_t count = 0;
        int problems = 0;
        while (at + count < ls.size() && problems < G.n2 + G.n1) problems += (int)ls[at + count++].prods.size();
        CHECK(problems == G.n2 + G.n1);
        CHECK(G.chunks >= 1 && (G.chunks == 1 || count == 1));
        for (size_t i = at; i < at + count; i++) {
            const RnsLayer &r = ls[i];
            CHECK(r.Kc % RNS_BK == 0 && (int64_t)(G.chunks - 1) * r.Kc < r.shape.K && (int64_t)G.chunks * r.Kc >= r.shape.K);
            CHECK(r.shape.segs * r.shape.K <= RNS_MAX_TERMS);
            used.push_back({r.at, r.at + r.shape.res_bytes()});
            // the planes lie before the residues, operand after operand
            const uint8_t *w = r.at;
            for (size_t o = r.ops.size(); o-- > 0;) {
                const int64_t bytes = RNS_N * rns_plane_bytes(r.ops[o].side ? r.shape.N : r.shape.M, r.Kc);
                used.push_back({w - bytes, w});
                w -= bytes;
            }
        }
        std::sort(used.begin(), used.end());
        for (size_t i = 0; i < used.size(); i++) {
            CHECK(used[i].begin >= lo && used[i].end <= hi);
            CHECK(i == 0 || used[i - 1].end <= used[i].begin);
        }
        const std::set<Range> ranges(used.begin(), used.end());
        auto exact = [&](const uint8_t *b, int64_t bytes) {  // [b, b + bytes) is one of the ranges
            const auto it = ranges.find({b, b});
            return it != ranges.end() && it->end == b + bytes;
        };
        // conversions: every fragment of a chunk once
        int wg = 0;
        for (int j = G.job0; j < G.job0 + G.njobs; j++) {
            const RnsJob &J = jobs[j];
            const int64_t major = J.side ? J.cols : J.rows, K = J.side ? J.rows : J.cols;
            CHECK(J.wg_begin == wg && J.kt * 32 == J.Kc && J.majb == rns_blocks(major));
            CHECK(J.plane == rns_plane_bytes(major, J.Kc) && exact(J.dst, RNS_N * J.plane));
            wg += J.wgs;
            for (int chunk = 0; chunk < G.chunks; chunk++) {
                const int64_t kc = std::min<int64_t>(J.Kc, K - (int64_t)chunk * J.Kc), frags = (kc + 63) / 64 * 2;
                CHECK(kc > 0 && frags <= J.kt);
                std::vector<char> hit(frags * J.majb, 0);
                for (int local = 0; local < J.wgs; local++)
                    for (int wave = 0; wave < 4; wave++) {
                        int mb, ks;
                        if (J.side) {
                            const int groups = (J.majb + 3) / 4;
                            ks = local / groups;
                            mb = (local - ks * groups) * 4 + wave;
                        } else {
                            const int groups = (J.kt + 3) / 4;
                            mb = local / groups;
                            ks = (local - mb * groups) * 4 + wave;
                        }
                        if (mb >= J.majb || ks >= frags) continue;
                        const int64_t off = ((int64_t)(ks >> 1) * J.majb + mb) * 2048 + (ks & 1) * 1024;
                        CHECK(off + 1024 <= J.plane && !hit[ks * J.majb + mb]);
                        hit[ks * J.majb + mb] = 1;
                    }
                CHECK(std::count(hit.begin(), hit.end(), 1) == (int64_t)hit.size());
            }
            packed++;
        }
        CHECK(wg == G.wgs);
        int left = 0, right = 0;
        for (int j = G.open0; j < G.open0 + G.nopen; j++) {
            const RnsOpen &J = opens[j];
            CHECK(J.layer >= 0 && J.wg_left == left && J.wg_right == right && J.kt * 32 == J.Kc);
            left += J.kt * J.mb;
            right += J.kt * ((J.nb + 3) / 4);
            for (int o = 0; o < 3; o++) {
                CHECK(exact(J.left + o * RNS_N * J.planeL, RNS_N * J.planeL));
                CHECK(exact(J.right + o * RNS_N * J.planeR, RNS_N * J.planeR));
            }
            for (int o = 0; o < 2 && J.left_tag; o++) {
                CHECK(exact(J.left_tag + o * RNS_N * J.planeL, RNS_N * J.planeL));
                CHECK(exact(J.right_tag + o * RNS_N * J.planeR, RNS_N * J.planeR));
            }
            opened++;
        }
        CHECK(left == G.left && right == G.right);
        // products: every modulus and tile of every problem once, in a launch of 8 blocks_x workgroups
        for (int outs = 2; outs >= 1; outs--) {
            const RnsProb *p0 = probs.data() + G.prob0 + (outs == 2 ? 0 : G.n2);
            const int np0 = outs == 2 ? G.n2 : G.n1, blocks = outs == 2 ? G.blocks2 : G.blocks1;
            std::vector<std::vector<char>> hit(np0);
            for (int i = 0; i < np0; i++) hit[i].assign((size_t)RNS_N * p0[i].tiles_m * p0[i].tiles_n, 0);
            for (int x = 0; x < 8 && np0 > 0; x++)
                for (int idx = 0; idx < blocks; idx++) {
                    int i = 0;
                    while (i + 1 < np0 && p0[i + 1].begin[x] <= idx) i++;
                    const RnsProb &p = p0[i];
                    const int tiles = p.tiles_m * p.tiles_n, local = idx - p.begin[x], qi = local / tiles;
                    const int q = ((x - p.rot) & 7) + 8 * qi;
                    CHECK(local >= 0 && p.outs == outs);
                    if (q >= RNS_N) continue;
                    const int t = local - qi * tiles, grp = t / (8 * p.tiles_n), gm = std::min(8, p.tiles_m - 8 * grp);
                    const int r = t - grp * 8 * p.tiles_n, tn = r / gm, tm = 8 * grp + r - tn * gm;
                    CHECK(tm < p.tiles_m && tn < p.tiles_n);
                    char &h = hit[i][((size_t)q * p.tiles_m + tm) * p.tiles_n + tn];
                    CHECK(!h);
                    h = 1;
                }
            for (const auto &h : hit) CHECK(std::count(h.begin(), h.end(), 1) == (int64_t)h.size());
        }
        // reconstruction items, and the residues of a layer's products one after another
        int items = 0;
        for (int i = G.prob0; i < G.prob0 + G.n2 + G.n1; i++) {
            const RnsProb &p = probs[i];
            CHECK(p.fold_begin == items && p.mb == rns_blocks(p.M) && p.nb == rns_blocks(p.N));
            items += p.outs * p.mb * p.nb;
            for (const uint8_t *b : {p.L0, p.L1, p.outs == 2 ? p.L2 : p.L1}) CHECK(exact(b, RNS_N * p.planeL));
            for (const uint8_t *b : {p.R0, p.R2, p.outs == 2 ? p.R1 : p.R0}) CHECK(exact(b, RNS_N * p.planeR));
            const int64_t bytes = (int64_t)p.outs * RNS_N * p.mb * p.nb * 1024;
            bool inside = false;
            for (size_t l = at; l < at + count; l++)
                inside |= p.res >= ls[l].at && p.res + bytes <= ls[l].at + ls[l].shape.res_bytes();
            CHECK(inside);
        }
        CHECK(items == G.fold_items);
        at += count;
    }
    CHECK(at == ls.size() && jobs_at == P.njobs && probs_at == P.nprobs && opens_at == P.nopen);
    // every layer is planned once
    std::multiset<std::vector<int64_t>> a, b;
    for (const auto &r : before) a.insert({r.shape.M, r.shape.K, r.shape.N, r.open});
    for (const auto &r : ls) b.insert({r.shape.M, r.shape.K, r.shape.N, r.open});
    CHECK(a == b);
}

static ct_layer_desc desc(int64_t M, int64_t K, int64_t N, int compress = 0) {
    ct_layer_desc d;
    std::memset(&d, 0, sizeof(d));
    d.M = M; d.K = K; d.N = N; d.compress = compress;
    return d;
}

static int taken(const std::vector<ct_layer_desc> &ds, int np, bool compact) {
    std::vector<RnsShape> s;
    for (const auto &d : ds) s.push_back(rns_online_shape(d, np, compact));
    const std::vector<char> t = rns_choose(s, RNS_SCRATCH_BYTES, false);
    return (int)std::count(t.begin(), t.end(), 1);
}

int main() {
    std::mt19937_64 rng(20231104);
    auto log_int = [&](int64_t lo, int64_t hi) {
        const double u = std::uniform_real_distribution<double>(std::log((double)lo), std::log((double)hi))(rng);
        return std::min(hi, std::max(lo, (int64_t)std::llround(std::exp(u))));
    };
    // chunks(): as few as fit, found past counts that leave their last chunks empty (1025 = 8 * 128 + 1)
    for (int c : {1, 2, 3, 6, 9, 17}) {
        const RnsShape s = rns_online_shape(desc(449, 1025, 481), 2, true);
        CHECK(s.chunks(s.bytes(s.chunk_len(c))) == c && s.chunks(s.bytes(RNS_BK) - 1) == 0);
    }
    ConvGeom cv;
    std::memset(&cv, 0, sizeof(cv));
    cv.on = 1;
    int64_t batches = 0, layers = 0;
    for (int step = 0; step < 1500; step++) {
        const int np = rng() % 2 ? 2 : 2 + (int)(rng() % 4), n = (int)log_int(1, 24);
        const bool compact = rng() % 2;
        const int64_t cap = rng() % 3 ? log_int(8 << 20, RNS_SCRATCH_BYTES) : RNS_SCRATCH_BYTES;
        std::vector<RnsLayer> ls;
        for (int l = 0; l < n; l++) {
            const ct_layer_desc d = desc(log_int(9, 4096), log_int(1, 4734), log_int(9, 4096), rng() % 4 == 0);
            const bool conv = np == 2 && rng() % 5 == 0, cm = compact && CT_COMPRESS_ALONG_M(d.M, d.N, d.compress);
            RnsLayer r = layer(d, np, compact, np == 2 && !conv && !cm ? l : -1, conv ? &cv : nullptr);
            if (r.shape.chunks(cap) > 0) ls.push_back(r);  // the others stay with digits
        }
        if (ls.empty()) continue;
        check_batch(ls, np, cap);
        batches++;
        layers += (int64_t)ls.size();
    }
    CHECK(batches > 500 && chunked > 100 && halves_seen > 100 && groups_seen > batches && opened > 100 && packed > 100);
    std::printf("ok plans batches=%lld layers=%lld groups=%lld halves=%lld chunked=%lld\n", (long long)batches, (long long)layers,
                (long long)groups_seen, (long long)halves_seen, (long long)chunked);
    // the rule on an encoder's layers: by residues with CompactTag, by digits in SPDZ2k and with three parties
    const std::vector<ct_layer_desc> encoder = {desc(128, 768, 2304), desc(128, 768, 768), desc(128, 768, 3072), desc(128, 3072, 768)};
    std::printf("ok rule compact=%d spdz2k=%d parties3=%d square=%d small=%d\n", taken(encoder, 2, true), taken(encoder, 2, false),
                taken(encoder, 3, true), taken({desc(2048, 2048, 2048)}, 2, true), taken({desc(64, 128, 32)}, 2, true));
    return 0;
}
