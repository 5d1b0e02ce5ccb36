// ct_rns.h -- exact products over Z_{2^128} through a residue number system:
// constants and the records the host and the kernels of ct_rns.hip share.
//
// A product sum P = sum_k x_k y_k over the integers (x_k, y_k taken as signed
// 128-bit integers, |x_k y_k| <= 2^254) is determined by its residues modulo
// pairwise coprime m_1, ..., m_n with |P| < prod m_i / 2 (Chinese remainder
// theorem), and only P mod 2^128 is wanted.  With every m_i <= 256 a residue
// fits a signed byte, so the residues of P are n independent int8 matrix
// products: n = 36 for up to RNS_MAX_TERMS terms, where the digit
// decomposition of ct_gemm.hip multiplies 136 digit pairs.  An operand takes
// n bytes per element instead of 16, so the rule that sends a product here
// weighs the saved matrix work against the extra bytes (RnsShape::saves_us).
#pragma once

#include "ct_internal.h"

namespace ct {

constexpr int RNS_N = 36;
// The 36 pairwise coprime moduli <= 256 with the largest product found
// (3 * 83 and 5 * 47 instead of 3 * 5 * 17 leave one more modulus above 96):
// log2 of the product is 268.2.
constexpr int RNS_M[RNS_N] = {256, 253, 251, 249, 247, 241, 239, 235, 233, 229, 227, 223, 217, 211, 199, 197, 193, 191,
                              181, 179, 173, 167, 163, 157, 151, 149, 139, 137, 131, 127, 113, 109, 107, 103, 101, 97};

constexpr bool rns_coprime() {
    for (int i = 0; i < RNS_N; i++)
        for (int j = 0; j < i; j++) {
            int a = RNS_M[i], b = RNS_M[j];
            while (b) { const int t = a % b; a = b; b = t; }
            if (a != 1) return false;
        }
    return true;
}
static_assert(rns_coprime(), "moduli must be pairwise coprime");

// Largest number of terms x_k y_k of a product sum: |P| <= terms 2^254 must
// stay below (1/2 - 2^-11) prod m_i; the 2^-11 leaves room for the fixed-point
// quotient of the reconstruction (its error is below 2^-12).
constexpr int64_t rns_max_terms() {
    double r = 1.0;  // prod m_i / 2^254, scaled as it grows
    int e = 0;
    for (int i = 0; i < RNS_N; i++) {
        r *= RNS_M[i];
        while (r >= 2.0) { r /= 2.0; e++; }
    }
    for (; e > 254; e--) r *= 2.0;
    return (int64_t)(r * (0.5 - 1.0 / 1024));
}
constexpr int64_t RNS_MAX_TERMS = rns_max_terms();
static_assert(RNS_MAX_TERMS > 2 * 4608 && RNS_MAX_TERMS < 2 * 4744, "range of the residue system");

// Residue planes of an operand: for each modulus one plane of signed bytes,
// cut into fragments of 32 major indices (rows of a left operand, columns of
// a right one) x 32 k, 1 KB each, in the order the matrix cores read them:
// byte b of lane l is major l % 32, k = 16 (l / 32) + b.  A plane holds, for
// each K slice of 64, the two fragments of every major block in turn: what the
// workgroups of a launch read at about the same time is contiguous and spreads
// over the cache and memory channels.
constexpr int RNS_BK = 64;    // K slice of a stage of k_rns_gemm
constexpr int RNS_TM = 128, RNS_TN = 128;  // output tile of a workgroup of k_rns_gemm, for one or two products
inline int64_t rns_blocks(int64_t major) { return (major + 31) / 32; }
inline int64_t rns_plane_bytes(int64_t major, int64_t kc) { return rns_blocks(major) * ((kc + 63) / 64 * 2) * 1024; }

// One operand to convert: rows [chunk Kc, (chunk + 1) Kc) of the contraction
// range of src become the planes at dst (plane q at q * plane_bytes).
struct RnsJob {
    const u128 *src;
    uint8_t *dst;
    int64_t plane;              // bytes per plane
    int32_t rows, cols, side;   // src is rows x cols; side 0: left (major = row), 1: right (major = column)
    int32_t Kc, kt, majb;       // chunk length (multiple of RNS_BK), Kc / 32, major blocks of 32
    int32_t wg_begin, wgs;      // workgroups of four fragments each
    ConvGeom cv;                // right operand read as the implicit im2col matrix of src (cv.on)
};

// A two-party layer whose openings write the planes themselves: E, A_0 + E,
// [A]_1 from `left` on and [B]_0, [B]_1, U from `right` on, RNS_N planes each;
// in SPDZ2k also [tA]_p + [Delta]_p E from `left_tag` and [tB]_p from
// `right_tag` on.
struct RnsOpen {
    uint8_t *left, *right, *left_tag, *right_tag;
    int64_t planeL, planeR;
    int32_t layer, Kc, kt, mb, nb;
    int32_t wg_left, wg_right;  // first workgroups (of one left fragment, of four right ones)
};

// One or two products that share operands, over operand planes of one K chunk:
//   out_0 = L0 R0 + L1 R2,  out_1 = L0 R1 + L2 R2   (outs = 2), out_0 alone (outs = 1),
//   segs = 1: without the second terms.
// Their residues go to res: plane (q * outs + o), tiles of 32 x 32 outputs of
// 1 KB each (the accumulator order of a wavefront).  Later chunks add to them.
struct RnsProb {
    const uint8_t *L0, *L1, *L2, *R0, *R1, *R2;
    uint8_t *res;
    const u128 *base[2];        // constant terms (null: zero)
    u128 *out[2];               // M x N row-major
    int64_t planeL, planeR;
    int32_t M, N, K, Kc, kt, outs, segs;
    int32_t mb, nb;             // blocks of 32 rows and columns
    int32_t tiles_m, tiles_n;   // workgroup tiles
    int32_t fold_begin;         // first wavefront item of the reconstruction
    int32_t rot;                // modulus q runs on XCD (q + rot) % 8
    int32_t begin[8];           // per XCD: position of the problem's workgroups
};

hipError_t launch_rns_pack(const RnsJob *jobs, int njobs, int wgs, int chunk, hipStream_t st);
hipError_t launch_rns_open(const LayerDev *L, const RnsOpen *jobs, int njobs, int wgs_left, int wgs_right, int flags, int chunk,
                           hipStream_t st);
// blocks_x: most workgroups on one XCD (the grid is 8 times that)
hipError_t launch_rns_gemm(int outs, const RnsProb *probs, int nprobs, int blocks_x, int chunk, hipStream_t st);
hipError_t launch_rns_fold(const RnsProb *probs, int nprobs, int items, hipStream_t st);

}  // namespace ct
