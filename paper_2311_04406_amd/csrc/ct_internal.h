// ct_internal.h -- library-internal types shared by the host side of
// libcompacttag and its HIP kernels.  Not part of the C ABI.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "compacttag.h"

namespace ct {

// Element of Z_{2^128}: value = lo + 2^64 hi (same layout as ct_u128).
struct u128 {
    uint64_t lo, hi;
};
// An element of Z_{2^64}: shares and tags of the k = s = 32 parameter set.
struct r64 {
    uint64_t v;
};

// Generator stream purposes; stream = (layer_id << 16) | purpose.
enum Purpose : uint32_t {
    P_LIFT_X = 0x01, P_LIFT_Y = 0x02, P_LIFT_A = 0x03, P_LIFT_B = 0x04, P_LIFT_R = 0x05,
    P_LIFT_RF = 0x06,  // upper limb of the lift of the truncated mask R^f
    P_VSH = 0x10,  // + object 1..7
    P_TSH = 0x20,  // + object 1..7
    P_CHI = 0x30, P_CHIHAT = 0x31, P_CHI_E = 0x32, P_CHI_U = 0x33, P_CHI_D = 0x34,
    P_KEY = 0x40,  // + party, on the global layer id 0xFFFF
};
enum Obj : int { OBJ_X = 1, OBJ_Y = 2, OBJ_A = 3, OBJ_B = 4, OBJ_C = 5, OBJ_R = 6, OBJ_RF = 7 };
constexpr int NUM_OBJ = 7;
constexpr uint64_t GLOBAL_LAYER = 0xFFFF;

// Index of each generator key in LayerDev::key.
enum KeyIdx : int {
    K_LIFT_X = 0, K_LIFT_Y, K_LIFT_A, K_LIFT_B, K_LIFT_R, K_LIFT_RF,
    K_VSH_X, K_VSH_Y, K_VSH_A, K_VSH_B, K_VSH_C, K_VSH_R, K_VSH_RF,
    K_TSH_X, K_TSH_Y, K_TSH_A, K_TSH_B, K_TSH_C, K_TSH_R, K_TSH_RF,
    K_CHI, K_CHIHAT, K_CHI_E, K_CHI_U, K_CHI_D,
    K_COUNT
};

// Geometry of a convolution layer whose right operand is the implicit im2col
// matrix of a c x h x w input (Eq. (4)); on = 0 for a plain product.
struct ConvGeom {
    int32_t on, c, h, w, k, s, p, wo;
};

// Element of the input under entry (k, n) of the im2col matrix:
// k = (c k + dy) k + dx, n = y wo + x -> (c, y s + dy - p, x s + dx - p);
// -1 where that falls in the zero padding.  k < 2^21, n < 2^22.
__host__ __device__ inline int64_t conv_src(const ConvGeom &g, int32_t k, int32_t n) {
    const uint32_t kk = (uint32_t)(g.k * g.k);
    const uint32_t c = (uint32_t)k / kk, t = (uint32_t)k - c * kk;
    const uint32_t dy = t / (uint32_t)g.k, dx = t - dy * (uint32_t)g.k;
    const uint32_t y = (uint32_t)n / (uint32_t)g.wo, x = (uint32_t)n - y * (uint32_t)g.wo;
    const int32_t iy = (int32_t)(y * g.s + dy) - g.p, ix = (int32_t)(x * g.s + dx) - g.p;
    if (iy < 0 || iy >= g.h || ix < 0 || ix >= g.w) return -1;
    return ((int64_t)c * g.h + iy) * g.w + ix;
}
// Index of right-operand entry (k, n) in a layer's K x N-shaped or input-shaped buffers.
__host__ __device__ inline int64_t kn_src(const ConvGeom &g, int64_t N, int64_t k, int64_t n) {
    return g.on ? conv_src(g, (int32_t)k, (int32_t)n) : k * N + n;
}

// Per-layer descriptor as the kernels see it (device memory).
// The two-party kernels use slots 0 and 1 of the per-party arrays; the
// n-party kernels (np > 2) slots 0 .. np - 1.
constexpr int MAXP = CT_MAX_PARTIES;
struct LayerDev {
    int64_t M, K, N;
    uint64_t delta[MAXP];       // key shares
    uint64_t key[K_COUNT];      // SplitMix64 stream keys
    u128 *X[MAXP], *tX[MAXP], *A[MAXP], *tA[MAXP];
    u128 *Y[MAXP], *tY[MAXP], *B[MAXP], *tB[MAXP];
    u128 *C[MAXP], *tC[MAXP], *R[MAXP], *tR[MAXP], *Z[MAXP], *tZ[MAXP];
    u128 *E, *U, *D, *cvec;
    u128 *work;                 // caller workspace: A_0 + E | tA_p + Delta_p E for p < np (M x K each), then
                                // the packed operands
    u128 *acc;                  // check accumulators, ACC_PER_LAYER entries (context scratch)
    unsigned long long *uc;     // FO_RNS: RP_COPIES copies of the check sums of U (RP_CELLS cells), k_rns_open_right's
    u128 *Rf[MAXP], *tRf[MAXP], *Zf[MAXP], *tZf[MAXP];  // f > 0: truncated mask and output (M x N)
    int32_t f, in_bits;         // truncated fractional bits; dealer input width (0: uniform)
    int32_t cm;                 // CompactTag compresses along M (W^c = chi^T W) instead of N
    int32_t np;                 // parties
    ConvGeom cv;                // convolution geometry (cv.on = 0: plain product)
    int64_t nr;                 // elements of Y, tY, B, tB, U: K N, or c h w of a convolution
    // share streams of parties 1 .. np - 2 (party 0 uses key[K_VSH_X + obj - 1] and
    // key[K_TSH_X + obj - 1]; the last party completes the sums)
    uint64_t vsh[MAXP - 2][NUM_OBJ], tsh[MAXP - 2][NUM_OBJ];
    // two-party matrix-core layers that are not convolutions: FO_DIGITS: U is opened by
    // k_open_pack, which also writes the digit tiles of [B]_0, [B]_1 and U
    // (rp[0..2], in the workspace); FO_RNS: E and U are opened by the kernels
    // that write the operands' residue planes.  k_open_u skips both
    int32_t fo;
    int32_t out_index;          // position of the layer's check record in the caller's result array
    int32_t row_seg, row_segs;  // row pass: elements of an item, items per row (row_seg below)
    int32_t cm_rows;            // the same compressing along M: rows of a wavefront (cm_rb below)
    int32_t cm_items;           // and the number of items (of a workgroup with cm_share, else of a wavefront)
    int32_t cm_share;
    u128 *rp[3];
};

enum Fo : int32_t { FO_NONE = 0, FO_DIGITS = 1, FO_RNS = 2 };

// cvec offsets of n parties, compressing along N (see compacttag.h): U^c,
// tB^c_p (K each), then D^c, E U^c, tC^c_p, tR^c_p, tZ^c_p, tD^c_p (M each).
struct NpCvec {
    int64_t Uc, tBc, Dc, EUc, tCc, tRc, tZc, tDc, K, M;
    __host__ __device__ int64_t tb(int p) const { return tBc + p * K; }
    __host__ __device__ int64_t tc(int p) const { return tCc + p * M; }
    __host__ __device__ int64_t tr(int p) const { return tRc + p * M; }
    __host__ __device__ int64_t tz(int p) const { return tZc + p * M; }
    __host__ __device__ int64_t td(int p) const { return tDc + p * M; }
};
__host__ __device__ inline NpCvec np_cvec(int64_t M, int64_t K, int np) {
    NpCvec o;
    o.K = K; o.M = M;
    o.Uc = 0; o.tBc = K; o.Dc = (1 + np) * K; o.EUc = o.Dc + M;
    o.tCc = o.Dc + 2 * M; o.tRc = o.tCc + np * M; o.tZc = o.tRc + np * M; o.tDc = o.tZc + np * M;
    return o;
}

// Layers with N <= SKINNY_MAX_N take their output products on the VALU inside
// the pass that opens E (no MFMA tiles, no workspace).
constexpr int SKINNY_MAX_N = 8;

// Elements of one row of E per work item of the row pass (a multiple of 64):
// long rows are cut into several items, so that a layer with few rows still
// spreads over the whole GPU; segments double while the layer keeps at least
// 16384 items.  Each item ends in wavefront reductions and atomic additions of
// its row products, so short items cost: on the batched set (K from 32 to
// 4096) the pass took 1.22 ms with items of at least 256 elements, 0.87 ms
// with 512 and 0.77 ms with 1024.  A layer with fewer than ROW_ITEMS items of
// 1024 (two wavefronts a compute unit) is bound by the chain of an item's
// iterations, about 2 us each, and is cut shorter, down to two iterations: the
// pass took 28 us instead of 39 on an encoder's layers, 0.58 ms instead of
// 0.75 on 64 uneven ones; with four times as many items 0.75, with half 0.58.
constexpr int64_t ROW_ITEMS = 512, ROW_SEG_MIN = 128;
inline int64_t row_seg(int64_t M, int64_t K) {
    int64_t s = 1024;
    while (s < 4096 && M * ((K + 2 * s - 1) / (2 * s)) >= 16384) s *= 2;
    while (s > ROW_SEG_MIN && M * ((K + s - 1) / s) < ROW_ITEMS) s /= 2;
    return s;
}
inline int64_t row_items(int64_t M, int64_t K) {
    const int64_t s = row_seg(M, K);
    return M * ((K + s - 1) / s);
}

// Flags of the fused passes.
enum PassFlags : int {
    F_CHECK = 1,    // accumulate the MAC-check sums of the values the pass opens
    F_COMPACT = 2,  // CompactTag protocol (compression, compact tag)
    F_SPDZ = 4,     // SPDZ2k protocol (per-element tags by products)
};

// Check accumulators per layer.  Two parties: for W in (E, U, D) at 3 W:
// [sum chi*tW_0, sum chi*tW_1, sum chi*W].  n parties: at W (CT_MAX_PARTIES + 1):
// [sum chi*tW_p for p < n ..., sum chi*W at slot CT_MAX_PARTIES].
constexpr int ACC_W = CT_MAX_PARTIES + 1;
// The row passes add their check sums of E into copies of their
// accumulators held as 32-bit limbs in 64-bit cells (atomic_add_limbs), from
// element ACC_RP of the layer's accumulators on: workgroup b adds into copy
// b % RP_COPIES (two parties: 3 sums, 12 cells a copy) or b % NP_RP_COPIES
// (n parties: ACC_W sums, 4 ACC_W cells), so that concurrent workgroups add
// to different cells without waiting; k_finalize / k_np_finalize add the
// copies to the E sums.
constexpr int ACC_RP = 3 * ACC_W;
constexpr int RP_CELLS = 1536;  // 64-bit cells (768 elements of 16 bytes)
constexpr int RP_COPIES = RP_CELLS / 12;
constexpr int NP_RP_COPIES = RP_CELLS / (4 * ACC_W);
// The layers' accumulators lie this far apart, in a block of device memory of
// their own (lane_init), with nothing else of a layer between them: thousands of
// workgroups of k_check_batch and the passes add to the same few elements, and
// how fast the memory takes that depends on where they lie.  k_check_batch of
// 14 layers in SPDZ2k (SPDZ2K_CHECK in tests/test_accumulators.py) takes 620 us
// so (178 of them without the additions); 785 with the accumulators behind the
// lane's tables, 805 with twice the spacing, 840 with both.
constexpr int ACC_PER_LAYER = 3 * ACC_W + RP_CELLS / 2;

// cvec offsets (elements), see compacttag.h.  Compressing along M the same
// offsets are taken with M replaced by N (cvec_off(N, K)), and the three
// K-long vectors hold E^c, [tA^c]_0, [tA^c]_1 in place of U^c, [tB^c]_p.
struct CvecOff {
    int64_t Uc, tBc0, tBc1, Dc, EUc, tCc0, tCc1, tRc0, tRc1, tZc0, tZc1, tDc0, tDc1;
};
__host__ __device__ inline CvecOff cvec_off(int64_t M, int64_t K) {
    CvecOff o;
    o.Uc = 0; o.tBc0 = K; o.tBc1 = 2 * K; o.Dc = 3 * K; o.EUc = 3 * K + M;
    o.tCc0 = 3 * K + 2 * M; o.tCc1 = 3 * K + 3 * M; o.tRc0 = 3 * K + 4 * M; o.tRc1 = 3 * K + 5 * M;
    o.tZc0 = 3 * K + 6 * M; o.tZc1 = 3 * K + 7 * M; o.tDc0 = 3 * K + 8 * M; o.tDc1 = 3 * K + 9 * M;
    return o;
}

// Length of the compressed M x N quantities (D^c, the compact tags): M when
// compressing along N, N when compressing along M.
__host__ __device__ inline int64_t cvec_rows(const LayerDev &L) { return L.cm ? L.N : L.M; }

// Variant of the row pass a layer takes: 0 for matrix-core layers, else the
// smallest of 1, 2, 4, 8 that holds N.  Each variant is its own kernel so the
// register budget (and occupancy) of one does not limit the others.
__host__ __device__ inline int row_variant(int64_t N) {
    return N > SKINNY_MAX_N ? 0 : (N <= 1 ? 1 : (N <= 2 ? 2 : (N <= 4 ? 4 : SKINNY_MAX_N)));
}

// With more than two parties, the fused row pass serves matrix-core layers and
// layers with N <= 2 (its per-party row products fit in registers); layers
// with 2 < N <= SKINNY_MAX_N take the separate opening, product and compact
// passes.
__host__ __device__ inline bool np_fused_row(int64_t N) { return N > SKINNY_MAX_N || N <= 2; }

// Row pass of a layer compressed along M: lanes own columns; a wavefront takes
// a strip of cm_cw(N) * 64 columns over up to CM_RB rows and keeps the column
// sums chi_m E_mk, chi_m [tA]_p,mk in registers until its rows are done
// (narrower strips for skinny layers, whose row products take registers too).
// A layer with fewer than CM_WAVES such wavefronts (or more than CM_ADDS row
// blocks) shares: its rows come one after another, a few us each, and the
// atomic additions of a column follow one another, so its wavefronts take fewer
// rows, and the four of a workgroup, on neighbouring rows, add their sums
// before they go out.  512 x 4608 x 49 took 167 us with 32 rows a wavefront, 102
// with 8, 90 shared (its 377 MB take 80); 1024^3 175, 79 and 48; 3000 x 64 x 2000
// 53, 76 (with 2 rows) and 22.  Layers with enough wavefronts are slower shared:
// 3104 us for 4096 x 25088 x 1 by wavefronts, 3180 shared.
constexpr int CM_RB = 32, COL_WAVES = 4;
constexpr int64_t CM_WAVES = 1024, CM_RB_MIN = 2, CM_ADDS = 256;
__host__ __device__ constexpr int cm_cw_variant(int ns) { return ns == 0 || ns == 1 ? 4 : (ns == 2 ? 2 : 1); }
__host__ __device__ inline int cm_cw(int64_t N) {
    return cm_cw_variant(N > 8 ? 0 : (N <= 1 ? 1 : (N <= 2 ? 2 : (N <= 4 ? 4 : 8))));
}
// Bits of the row-pass variant set: v for k_row_pass<v>, VARIANT_E for
// k_row_pass_e (the pass of FO_RNS layers, which reads the opened E),
// VARIANT_CM + cm_index(v) for k_row_pass_cm<v> (v = 0, 1, 2, 4, 8), and
// VARIANT_CM_SHARED + cm_index(v) for the same with shared items.
constexpr int VARIANT_E = 9, VARIANT_CM = 16, VARIANT_CM_SHARED = 21;
constexpr int cm_index(int v) { return v == 8 ? 4 : v == 4 ? 3 : v; }
__host__ __device__ inline int64_t cm_strips(int64_t K, int cw) { return (K + 64 * cw - 1) / (64 * cw); }
inline bool cm_share(int64_t M, int64_t K, int64_t N) {
    const int64_t blocks = (M + CM_RB - 1) / CM_RB;
    return cm_strips(K, cm_cw(N)) * blocks < CM_WAVES || blocks > CM_ADDS;
}
inline int64_t cm_rb(int64_t M, int64_t K, int64_t N) {
    const int64_t strips = cm_strips(K, cm_cw(N));
    int64_t rb = CM_RB;
    if (cm_share(M, K, N))
        while (rb > CM_RB_MIN && strips * ((M + rb - 1) / rb) < CM_WAVES && M <= CM_ADDS * COL_WAVES * (rb / 2)) rb /= 2;
    return rb;
}
inline int64_t cm_items(int64_t M, int64_t K, int64_t N) {
    const int64_t rows = (cm_share(M, K, N) ? COL_WAVES : 1) * cm_rb(M, K, N);
    return cm_strips(K, cm_cw(N)) * ((M + rows - 1) / rows);
}

// Column sweep (sums down the columns of a rows x N matrix): workgroup items of
// COL_WAVES wavefronts, each with rb groups of 64 / G rows (N <= 32,
// G = pow2ceil(N)) or with 64 columns x rb rows (one per lane); one atomic per
// column per item.  Additions to the same address follow one another, about
// 0.1 us each, so rb = col_sweep_rb keeps them near COL_ADDS per column at
// most, without starving the sweep of wavefronts.
// One wavefront per item and 256 additions took 33 us in k_col_tag of
// 512 x 4608 x 49 and 67 us in k_post of 1024^3; workgroup items took 33, 23,
// 19 and 23 us (46, 45, 47 and 67) with 32, 64, 128 and 256.
constexpr int64_t COL_ADDS = 128, COL_RB_MIN = 4;
__host__ __device__ inline int64_t col_sweep_group(int64_t N) {
    int64_t g = 1;
    while (g < N) g <<= 1;
    return g;
}
__host__ __device__ inline int64_t col_sweep_rb(int64_t rows, int64_t N) {
    if (N <= 32) {
        const int64_t per = (64 / col_sweep_group(N)) * COL_WAVES * COL_ADDS, rb = (rows + per - 1) / per;
        return rb < 1 ? 1 : rb;
    }
    const int64_t rb = (rows + COL_WAVES * COL_ADDS - 1) / (COL_WAVES * COL_ADDS);
    return rb < COL_RB_MIN ? COL_RB_MIN : rb;
}
__host__ __device__ inline int64_t col_sweep_items(int64_t rows, int64_t N) {
    const int64_t rb = col_sweep_rb(rows, N);
    if (N <= 32) {
        const int64_t per = (64 / col_sweep_group(N)) * COL_WAVES * rb;
        return (rows + per - 1) / per;
    }
    return ((N + 63) / 64) * ((rows + COL_WAVES * rb - 1) / (COL_WAVES * rb));
}

// Operands of the matrix-core products are converted once into "digit
// tiles": for an operand with major dimension D (rows of a left operand,
// columns of a right operand) and contraction length K, tile (t, ks) covers
// major indices [64 t, 64 t + 64) and k in [32 ks, 32 ks + 32); it occupies
// TILE_ELEMS elements at ((t * KT) + ks) * TILE_ELEMS and holds one plane of
// signed 8-bit digits per digit of an element (plane d = digit d; 16 planes,
// 32 KB, for Z_{2^128}; 8 planes, 16 KB, for Z_{2^64}) of 64 x 32 bytes, in the
// byte order of the GEMM's LDS stage.  Out-of-range entries are zero.
constexpr int TILE_ELEMS = 2048;

inline int64_t packed_elems(int64_t major, int64_t K) { return ((major + 63) / 64) * ((K + 31) / 32) * TILE_ELEMS; }

// Workspace of a layer with N > SKINNY_MAX_N (element offsets): the folded
// left operands written by the row pass, then the digit tiles of every
// operand of the matrix-core products.
struct WorkOff {
    int64_t AE0, tAE0, tAE1;                  // u128, M x K each
    int64_t Ep, AE0p, A1p, tAE0p, tAE1p;      // packed left operands
    int64_t B0p, B1p, Up, tB0p, tB1p;         // packed right operands
    int64_t total;
};
inline WorkOff work_off(int64_t M, int64_t K, int64_t N) {
    WorkOff o;
    const int64_t mk = M * K, pl = packed_elems(M, K), pr = packed_elems(N, K);
    o.AE0 = 0; o.tAE0 = mk; o.tAE1 = 2 * mk;
    o.Ep = 3 * mk; o.AE0p = o.Ep + pl; o.A1p = o.Ep + 2 * pl; o.tAE0p = o.Ep + 3 * pl; o.tAE1p = o.Ep + 4 * pl;
    o.B0p = o.Ep + 5 * pl; o.B1p = o.B0p + pr; o.Up = o.B0p + 2 * pr; o.tB0p = o.B0p + 3 * pr;
    o.tB1p = o.B0p + 4 * pr;
    o.total = o.B0p + 5 * pr;
    return o;
}

// One packing job: src (row-major rows x cols) -> dst digit tiles.
// side 0: left operand (major = row, k = column); side 1: right operand
// (major = column, k = row).
struct PackJob {
    const u128 *src;
    u128 *dst;
    int32_t rows, cols, side, majt, kt, tile_begin, tiles, pad;
    ConvGeom cv;  // right operand read as the implicit im2col matrix of src (cv.on)
};

// One ring GEMM problem over packed operands (one party's product of a layer;
// the products of a layer form a group whose tiles are interleaved):
//   out (+)= base + L1 * R1 + L2 * R2     (all mod 2^128)
// Lp1, Lp2: packed M x K left operands; Rp1, Rp2: packed K x N right
// operands; out, base: M x N row-major.  Lp2 == nullptr: single segment.
// accumulate != 0: out already holds base and partial sums of K splits are
// added atomically.
struct GemmProb {
    const u128 *Lp1, *Lp2, *Rp1, *Rp2, *base;
    u128 *out;
    int32_t M, N, K, accumulate;
    int32_t tiles_m, tiles_n, splits, steps_per_split;  // steps are 32-wide K slices
    int32_t kt, nsteps, tile_begin, tiles;  // tile_begin, tiles: of the problem's layer group
    int32_t group_m;  // tile order: column sweeps over groups of group_m row tiles
    int32_t gfirst;   // index of the first problem of the layer group (problems of one layer
    int32_t gsize;    //   share M, N, K and splits and are interleaved in the tile order)
    int32_t mt;       // 32 x 32 output tiles per wavefront, stacked in M (the same for every
                      // problem of a launch): workgroup tiles of 64 mt x 64 outputs
    int32_t wshape;   // WaveShape of the workgroup tile (register-streamed kernel, mt = 1)
};

// Arrangement of the four wavefronts of a register-streamed workgroup at one
// 32 x 32 output tile each: 2 x 2 (64 x 64 outputs), 1 x 4 (32 x 128) or
// 4 x 1 (128 x 32).  The wavefronts load their fragments independently, so
// any arrangement reads the same packed operand tiles; the narrow ones pad a
// product's M (or N) to 32 instead of 64.  WS_K4: all four on one tile, a
// quarter of the K slices each (k_ring_gemm_k4, every problem of a launch or none).
enum WaveShape : int { WS_64x64 = 0, WS_32x128 = 1, WS_128x32 = 2, WS_K4 = 3 };

// Product kernels: operand tiles staged through LDS, or fragments streamed
// from global memory into registers.
enum GemmKernel : int { GEMM_LDS = 0, GEMM_REGS = 1, GEMM_K4 = 2 };

// Launch configuration of the matrix-core products (chosen by ct_autotune).
struct GemmTuning {
    int32_t group_m;       // row tiles per group of the tile order (1 = row-major order)
    int32_t xcd_remap;     // 0: identity; 1: contiguous range per XCD; G >= 2: groups of G tiles per XCD
    int32_t split_target;  // K slices per tile; 0 = enough tiles for two rounds over the CUs
    int32_t tile;          // CT_TILE_*: kernel and workgroup tile (0 = by the launch's size)
    int32_t shared = 0;    // 1: tuned launches may have their wavefronts share K slices (WS_K4), as untuned ones may
};

// Unpacked product for the dealer's layers with N <= SKINNY_MAX_N:
// out = L * R (L: M x K, R: K x N, row-major).
struct SkinnyProb {
    const u128 *L, *R;
    u128 *out;
    int32_t M, N, K, pad;
};

// The two-party online phase of a batch as one persistent launch
// (k_online_persist): the stages' tables as the staged kernels take them, and
// the launch's counters, sync[0 .. 12), all 0 at the launch: sync[0] counts
// workgroup arrivals at the grid barriers, sync[1] is set when a barrier wait
// ran out (after wait_ticks of the 100 MHz wall clock), sync[4 + x] hands
// out the product tiles of XCD x.
struct PersistArgs {
    const LayerDev *Ls;
    const PackJob *jobs;
    const GemmProb *probs;
    ct_check_result *out;
    uint32_t *sync;
    uint64_t wait_ticks;
    int32_t n, flags, zero_what, njobs, pack_tiles, nprobs, total_tiles, xcd_remap, any_accum, mt;
};

// ---- launchers (defined in the .hip files) ----
// eb: bytes per ring element, 16 (k = s = 64) or 8 (k = s = 32).
hipError_t launch_pack(int eb, const PackJob *jobs_dev, int njobs, int total_tiles, hipStream_t st);
// kernel: GEMM_LDS (operand tiles staged through LDS, k_ring_gemm) or
// GEMM_REGS (fragments streamed into registers, k_ring_gemm_rs)
hipError_t launch_gemm(int eb, const GemmProb *probs_dev, int nprobs, int total_tiles, int xcd_remap, int mt,
                       int kernel, hipStream_t st);
// The persistent launch: `wgs` workgroups of 256 threads, one per compute
// unit (all must be resident at once: the stages meet at grid barriers).
hipError_t launch_online_persist(int eb, const PersistArgs &a, int wgs, hipStream_t st);
hipError_t launch_skinny(int eb, const SkinnyProb *probs_dev, int nprobs, int max_rows, hipStream_t st);

hipError_t launch_fill_zero(int eb, u128 *p, int64_t n, hipStream_t st);
hipError_t launch_deal_lift(int eb, const LayerDev *L, int n, int64_t max_elems, hipStream_t st);
hipError_t launch_deal_auth(int eb, const LayerDev *L, int n, int obj, int64_t max_elems, hipStream_t st);
hipError_t launch_zero_acc(int eb, const LayerDev *L, int n, int what, int64_t max_elems, hipStream_t st);
hipError_t launch_open_u(int eb, const LayerDev *L, int n, int flags, int64_t max_items, hipStream_t st);
hipError_t launch_open_pack(int eb, const LayerDev *L, int n, int flags, int max_tiles, hipStream_t st);
// variants: bit v (bit VARIANT_CM + v) set if some layer takes row-pass variant v (0, 1, 2, 4, 8)
// (of the pass of layers compressed along M)
hipError_t launch_row_pass(int eb, const LayerDev *L, int n, int flags, int64_t max_items, int variants, hipStream_t st);
// Layers compressed along M take a kernel of their own, with a grid of its own:
// max_items of the other layers, max_col_items of these (0: there are none;
// all_cm: there are no others).  Every workgroup of a layer that is not the
// kernel's leaves at once, but is launched: the pass over 27 layers (k = s = 32)
// took 387 us with the larger of the two grids for both kernels, 369 so.
hipError_t launch_post(int eb, const LayerDev *L, int n, int flags, int64_t max_items, int64_t max_col_items, bool all_cm,
                       hipStream_t st);
hipError_t launch_compact_final(int eb, const LayerDev *L, int n, int flags, hipStream_t st);
hipError_t launch_col_tag(int eb, const LayerDev *L, int n, int64_t max_items, hipStream_t st);
hipError_t launch_conv_compress(int eb, const LayerDev *L, int n, int64_t max_items, hipStream_t st);

// n-party path (ct_parties.hip)
hipError_t launch_np_lift(int eb, const LayerDev *L, int n, int64_t max_elems, hipStream_t st);
hipError_t launch_np_auth(int eb, const LayerDev *L, int n, int obj_mask, int64_t max_elems, hipStream_t st);
hipError_t launch_np_zero(int eb, const LayerDev *L, int n, int what, int64_t max_elems, hipStream_t st);
hipError_t launch_np_open(int eb, const LayerDev *L, int n, int which, int flags, int64_t max_elems, hipStream_t st);
hipError_t launch_prob_base(int eb, const GemmProb *probs, int nprobs, int64_t max_mn, hipStream_t st);
hipError_t launch_np_skinny(int eb, const LayerDev *L, int n, int flags, int64_t max_items, hipStream_t st);
hipError_t launch_np_post(int eb, const LayerDev *L, int n, int flags, int64_t max_elems, hipStream_t st);
hipError_t launch_np_compress(int eb, const LayerDev *L, int n, int64_t max_items, hipStream_t st);
// variants: bit v set if some fused layer takes row-pass variant v (0, 1, 2)
hipError_t launch_np_row_pass(int eb, int np, const LayerDev *L, int n, int flags, int64_t max_items, int variants,
                              hipStream_t st);
hipError_t launch_np_gemv(int eb, const LayerDev *L, int n, int64_t max_items, hipStream_t st);
hipError_t launch_np_compact_final(int eb, const LayerDev *L, int n, int flags, hipStream_t st);
hipError_t launch_np_check_batch(int eb, int np, const LayerDev *L, int n, int which_mask, int64_t max_elems, hipStream_t st);
hipError_t launch_np_check_compact(int eb, const LayerDev *L, int n, hipStream_t st);
hipError_t launch_np_finalize(int eb, const LayerDev *L, int n, ct_check_result *out, hipStream_t st);
hipError_t launch_check_batch(int eb, const LayerDev *L, int n, int which, int64_t max_elems, hipStream_t st);
hipError_t launch_check_compact(int eb, const LayerDev *L, int n, hipStream_t st);
hipError_t launch_finalize(int eb, const LayerDev *L, int n, ct_check_result *out, hipStream_t st);

// Number of wavefront work items of a row sweep over an R x N matrix (the
// grid of the sweeping kernels is sized from it).
inline int64_t sweep_items(int64_t rows, int64_t N) {
    if (N <= 64) {
        int64_t g = 1;
        while (g < N) g <<= 1;
        const int64_t rpw = 64 / g;
        return (rows + rpw - 1) / rpw;
    }
    return rows * ((N + 511) / 512);
}

// Workgroup items of k_conv_compress: (input channel, segment of 512 output
// positions) of a convolution with c input channels and N output positions.
inline int64_t conv_compress_items(int64_t c, int64_t N) { return c * ((N + 511) / 512); }

}  // namespace ct
