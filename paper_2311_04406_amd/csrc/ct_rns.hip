// ct_rns.hip -- matrix products over Z_{2^128} by residues (see ct_rns.h):
// k_rns_pack converts operands to residue planes, k_rns_gemm multiplies them
// modulo each m_q on the int8 matrix cores, k_rns_fold reconstructs the sums
// mod 2^128 and adds the constant term.
#include "ct_rns.h"
#include "ct_sweep.h"

#include <type_traits>

namespace ct {

typedef int v4i __attribute__((ext_vector_type(4)));
typedef int v16i __attribute__((ext_vector_type(16)));
typedef unsigned __int128 x128;

// ---------------------------------------------------------------- constants
// Both conversions, of operands to residues and of residues to an element,
// are small matrix products with constant matrices and run on the matrix
// cores, with a block-diagonal left matrix: a lane of the right operand holds
// 16 bytes (an element's, or 16 residues of an output), and the rows that the
// lane receives back are nonzero only on its own k block, so each lane gets
// sums over its own 16 bytes -- 4 of them with v_mfma_i32_16x16x64_i8 (lane
// 16 h + c: k block h, rows 4 h + r), 16 with v_mfma_i32_32x32x32_i8 (lane
// 32 h + c: k block h, row 8 (r / 4) + 4 h + r % 4 in register r).
constexpr int mod_pos(x128 v, int m) { return (int)(v % (unsigned)m); }
constexpr int balanced(int v, int m) { return v >= (m + 1) / 2 ? v - m : v; }  // [-m/2, m/2): a signed byte

constexpr int rns_inverse(int i) {  // (prod_{j != i} m_j)^-1 mod m_i
    int prod = 1;
    for (int j = 0; j < RNS_N; j++)
        if (j != i) prod = prod * (RNS_M[j] % RNS_M[i]) % RNS_M[i];
    for (int v = 1; v < RNS_M[i]; v++)
        if (prod * v % RNS_M[i] == 1) return v;
    return 0;
}
constexpr x128 rns_others(int i) {  // prod_{j != i} m_j mod 2^128 (i < 0: of all)
    x128 prod = 1;
    for (int j = 0; j < RNS_N; j++)
        if (j != i) prod *= (unsigned)RNS_M[j];
    return prod;
}
constexpr int digit128(x128 v, int j) {  // balanced base-256 digit j
    x128 k = 0;
    for (int i = 0; i < 16; i++) k = (k << 8) | 0x80;
    return (int)((unsigned)((v + k) >> (8 * j)) & 0xff) - 128;
}

constexpr int CONV_GROUPS = RNS_N / 4;     // a conversion's instruction takes 4 moduli
constexpr int GROUPS = (RNS_N + 15) / 16;  // a reconstruction's takes 16
static_assert(RNS_N % 4 == 0, "moduli come in fours");

struct RnsTables {
    int8_t conv[2][CONV_GROUPS][1024];  // side 0 (left: also times (M / m_q)^-1), 1 (right): residue weights of the bytes
    int8_t fold[GROUPS][1024];     // digits of (M / m_q) mod 2^128
    int8_t quot[GROUPS][1024];     // digits of 2^24 / m_q
    uint32_t start[2][RNS_N];  // accumulator start of a conversion, as float bits (see convert)
    float inv[RNS_N];        // 1 / m_q
    uint32_t cmp[RNS_N];     // 256 - m_q mod 256
    int32_t m[RNS_N];
};

constexpr int conv_weight(int side, int q, int b) {  // 256^b mod m_q (left operands: times the inverse)
    const int m = RNS_M[q];
    int w = side ? 1 % m : rns_inverse(q) % m;
    for (int j = 0; j < b; j++) w = w * 256 % m;
    return balanced(w, m);
}

constexpr RnsTables make_tables() {
    RnsTables t{};
    for (int side = 0; side < 2; side++)
        for (int q = 0; q < RNS_N; q++) {
            const int m = RNS_M[q], g = q / 4, r = q % 4;
            int sum = 0;  // of the weights of bytes 0 .. 14
            for (int b = 0; b < 16; b++) {
                const int w = conv_weight(side, q, b);
                if (b < 15) sum += w;
                for (int h = 0; h < 4; h++) t.conv[side][g][(16 * h + 4 * h + r) * 16 + b] = (int8_t)w;
            }
            // a multiple of m near 1.5 * 2^23, plus the bytes' offset
            t.start[side][q] = 0x4B000000u + (uint32_t)((12582912 / m) * m - 8388608 + 128 * sum);
        }
    for (int g = 0; g < GROUPS; g++)
        for (int lane = 0; lane < 64; lane++) {
            const int row = lane & 31, half = lane >> 5;
            if (((row >> 2) & 1) != half) continue;  // the other k block: zero
            const int r = (row >> 3) * 4 + (row & 3);
            for (int b = 0; b < 16; b++) {
                const int s = 16 * g + b;  // byte b is the residue of modulus s, register r digit r
                if (s >= RNS_N) break;
                t.fold[g][lane * 16 + b] = (int8_t)digit128(rns_others(s), r);
                if (r < 3) t.quot[g][lane * 16 + b] = (int8_t)digit128(((2u << 24) / RNS_M[s] + 1) / 2, r);
            }
        }
    for (int q = 0; q < RNS_N; q++) {
        t.inv[q] = 1.0f / (float)RNS_M[q];
        t.cmp[q] = (uint32_t)(256 - RNS_M[q]) & 255;
        t.m[q] = RNS_M[q];
    }
    return t;
}
__device__ const RnsTables g_rns = make_tables();

// ---------------------------------------------------------------- operands to residues
__device__ __forceinline__ v4i as_bytes(u128 x) {
    // bytes 0 .. 14 as (byte - 128), byte 15 signed: x as a signed 128-bit
    // integer is sum_j 256^j s_j + 128 sum_{j<15} 256^j
    const uint64_t lo = x.lo ^ 0x8080808080808080ull, hi = x.hi ^ 0x0080808080808080ull;
    return v4i{(int)(uint32_t)lo, (int)(uint32_t)(lo >> 32), (int)(uint32_t)hi, (int)(uint32_t)(hi >> 32)};
}

// Low bytes of a, b, c, d as one dword.
__device__ __forceinline__ uint32_t pack4(uint32_t a, uint32_t b, uint32_t c, uint32_t d) {
    return __builtin_amdgcn_perm(__builtin_amdgcn_perm(d, c, 0x0c0c0400u), __builtin_amdgcn_perm(b, a, 0x0c0c0400u), 0x05040100u);
}

// The residues of the 16 elements of a lane (consecutive in k), 16 bytes per
// plane stored at dst + q plane.  Per residue: the matrix cores form
// S = sum_j s_j w_j + (offset) on top of a multiple B of m written as the bits
// of a float in [2^23, 2^24), so that the sum's bits are the float B + S
// without a conversion; one fma with 1 / m and 2^23 rounds (B + S) / m to an
// integer q in its low mantissa bits (off from the nearest integer by less
// than 1 / m: |S - m q| <= 127 for every odd m <= 253), and q times (256 - m)
// added to the bits leaves S - m q in the low byte.  Four moduli at a time: 16
// bytes of theirs take few registers, which leaves room for the loads of the
// next operand.  The planes go past the caches: a launch writes far more than
// they hold, and the products, which read them next, ran 2.72 ms on twelve
// encoders with ordinary stores and 2.25 with these (the openings 3% longer).
__device__ __forceinline__ void convert(const u128 (&x)[16], int side, uint8_t *dst, int64_t plane) {
    const int lane = threadIdx.x & 63;
#pragma unroll
    for (int g = 0; g < CONV_GROUPS; g++) {
        const v4i w = *reinterpret_cast<const v4i *>(&g_rns.conv[side][g][lane * 16]);
        v4i start;
#pragma unroll
        for (int r = 0; r < 4; r++) start[r] = (int)g_rns.start[side][4 * g + r];
        uint32_t out[4][4];
#pragma unroll
        for (int d = 0; d < 4; d++) {
            v4i acc[4];
#pragma unroll
            for (int i = 0; i < 4; i++)
                acc[i] = __builtin_amdgcn_mfma_i32_16x16x64_i8(w, as_bytes(x[4 * d + i]), start, 0, 0, 0);
#pragma unroll
            for (int r = 0; r < 4; r++) {
                uint32_t b[4];
#pragma unroll
                for (int i = 0; i < 4; i++) {
                    const float t = __builtin_fmaf(__int_as_float(acc[i][r]), g_rns.inv[4 * g + r], 8388608.0f);
                    b[i] = __umul24((uint32_t)__float_as_int(t), g_rns.cmp[4 * g + r]) + (uint32_t)acc[i][r];
                }
                out[r][d] = pack4(b[0], b[1], b[2], b[3]);
            }
        }
#pragma unroll
        for (int r = 0; r < 4; r++)
            __builtin_nontemporal_store(ct_u32x4{out[r][0], out[r][1], out[r][2], out[r][3]},
                                        global_ptr<ct_u32x4>(dst + (int64_t)(4 * g + r) * plane));
    }
}

// One wavefront per fragment (32 major indices x 32 k).  Right operands: a
// lane loads its column's 16 k directly (512-byte row segments per
// instruction); the four wavefronts of a workgroup take neighbouring columns.
// Left operands: row segments are loaded across the lanes and transposed
// through LDS (units permuted by the row so that both directions spread over
// the banks); the four wavefronts take neighbouring k.
__global__ __launch_bounds__(256) void k_rns_pack(const RnsJob *__restrict__ jobs, int njobs, int chunk) {
    __shared__ __attribute__((aligned(16))) u128 raw[4][1024];
    const int wg = blockIdx.x;
    int lo = 0, hi = njobs - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (jobs[mid].wg_begin <= wg) lo = mid; else hi = mid - 1;
    }
    const RnsJob &J = jobs[lo];
    const int local = wg - J.wg_begin, lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int K = J.side ? J.rows : J.cols, major = J.side ? J.cols : J.rows;
    const int k_base = chunk * J.Kc, kc = min(J.Kc, K - k_base), frags = (kc + 63) / 64 * 2;
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
    const bool ok = mb < J.majb && ks < frags;  // the same for the whole wavefront
    if (!ok) return;
    const u128 *src = J.src;
    const int k0 = k_base + 32 * ks;
    u128 x[16];
    if (J.side) {
        const int n = 32 * mb + (lane & 31);
#pragma unroll
        for (int i = 0; i < 16; i++) {
            const int k = k0 + 16 * (lane >> 5) + i;
            x[i] = u128{0, 0};
            if (k < K && n < major) {
                const int64_t e = kn_src(J.cv, J.cols, k, n);
                if (e >= 0) x[i] = ld(src, e);
            }
        }
    } else {
        const int k = lane & 31;
#pragma unroll
        for (int i = 0; i < 16; i++) {
            const int m = 32 * mb + 2 * i + (lane >> 5);
            x[i] = k0 + k < K && m < major ? ld(src, (int64_t)m * K + k0 + k) : u128{0, 0};
        }
#pragma unroll
        for (int i = 0; i < 16; i++) {
            const int r = 2 * i + (lane >> 5);
            raw[wave][r * 32 + (k ^ (r & 15))] = x[i];
        }
        wave_sync();
        const int r = lane & 31;
#pragma unroll
        for (int i = 0; i < 16; i++) x[i] = raw[wave][r * 32 + ((16 * (lane >> 5) + i) ^ (r & 15))];
    }
    convert(x, J.side, J.dst + ((int64_t)(ks >> 1) * J.majb + mb) * 2048 + (ks & 1) * 1024 + lane * 16, J.plane);
}

hipError_t launch_rns_pack(const RnsJob *jobs, int njobs, int wgs, int chunk, hipStream_t st) {
    if (njobs <= 0 || wgs <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_rns_pack, dim3(wgs), dim3(256), 0, st, jobs, njobs, chunk);
    return hipGetLastError();
}

// ---------------------------------------------------------------- open and convert
// Two-party layers that are neither convolutions nor compressed along M: the
// opened values go to residues in the pass that opens them, so no share array
// of the products is read twice.

// Sums of 16 values over the 32 lanes of a half wavefront: lane l of a half
// receives the total of value (l >> 1) & 15.  A butterfly that halves the
// values it still carries at each step: 16 exchanges for 16 sums, not 80.
__device__ __forceinline__ u128 half_sums(const u128 (&v)[16]) {
    const int lane = threadIdx.x & 63;
    u128 a[8], b[4], c[2];
    auto fold = [&](u128 lo, u128 hi, int bit) {  // lanes with the bit keep hi, the others lo
        const bool up = lane & bit;
        const u128 keep = up ? hi : lo, give = up ? lo : hi;
        return add(keep, shfl_xor128(give, bit));
    };
#pragma unroll
    for (int i = 0; i < 8; i++) a[i] = fold(v[i], v[i + 8], 16);
#pragma unroll
    for (int i = 0; i < 4; i++) b[i] = fold(a[i], a[i + 4], 8);
#pragma unroll
    for (int i = 0; i < 2; i++) c[i] = fold(b[i], b[i + 2], 4);
    const u128 d = fold(c[0], c[1], 2);
    return add(d, shfl_xor128(d, 1));
}

// Right operands: opens U = ([Y]_0 - [B]_0) + ([Y]_1 - [B]_1) (Fig. 7 online
// step 1), accumulates its batch check sums (Pi_BatchRec, Fig. 1), forms U^c
// and [tB^c]_p (Pi_Compress along N) and writes the planes of [B]_0, [B]_1 and
// U.  One wavefront per fragment, the four of a workgroup on neighbouring
// columns: the shares come in operand by operand (each lane 16 rows of its
// column), and [B]_0 + [B]_1 stays in registers for U; the row sums are added
// over the workgroup before they go out as atomics.  Bound by HBM (252 bytes
// an element with CompactTag and checks, with the left operands 4.3 TB/s at
// 2048 x 4096 x 2048 and 4.5 on an encoder's layers, where a large copy reaches
// 4.8; SPDZ2k 3.8: its 324 bytes come with five conversions).  One
// operand per wavefront instead took 5.2 ms, not 4.8, over twelve encoders.
__global__ __launch_bounds__(256, 2) void k_rns_open_right(const LayerDev *__restrict__ Ls, const RnsOpen *__restrict__ jobs,
                                                           int njobs, int flags, int chunk) {
    __shared__ u128 rows[3][WAVES][32];
    const int wg = blockIdx.x;
    int lo = 0, hi = njobs - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (jobs[mid].wg_right <= wg) lo = mid; else hi = mid - 1;
    }
    const RnsOpen &J = jobs[lo];
    const LayerDev &L = Ls[J.layer];
    const int groups = (J.nb + WAVES - 1) / WAVES, local = wg - J.wg_right, lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int K = (int)L.K, N = (int)L.N, k_base = chunk * J.Kc, frags = (min(J.Kc, K - k_base) + 63) / 64 * 2;
    const int ks = local / groups, nb = (local - ks * groups) * WAVES + wave;
    if (ks >= frags) return;
    const int n = 32 * nb + (lane & 31), kw = k_base + 32 * ks, k0 = kw + 16 * (lane >> 5);
    const bool check = flags & F_CHECK, compact = flags & F_COMPACT, tags = flags & F_SPDZ, live = nb < J.nb;
    const CvecOff o = cvec_off(L.M, K);
    uint8_t *dst = J.right + ((int64_t)(ks >> 1) * J.nb + nb) * 2048 + (ks & 1) * 1024 + lane * 16;
    // element i of a lane: the wavefront's row kw + i, plus the lane's own offset
    const int64_t e0 = (int64_t)kw * N + 32 * nb;
    const uint32_t le = (uint32_t)(16 * (lane >> 5)) * (uint32_t)N + (lane & 31);
    const int kn = n < N ? min(16, K - k0) : 0;  // rows of this lane (at most 0: none)
    const uint64_t xn = compact && n < N ? sdraw(L.key[K_CHI], (uint64_t)n) : 0, kcu = L.key[K_CHI_U];
    u128 chk[3] = {u128{0, 0}, u128{0, 0}, u128{0, 0}};
    auto load = [&](const u128 *p, u128 (&v)[16]) {
#pragma unroll
        for (int i = 0; i < 16; i++) v[i] = i < kn ? ld_nt(p + e0 + (int64_t)i * N, le) : u128{0, 0};
    };
    // sum over the wavefront's columns of v xn, row by row
    auto row_sums = [&](const u128 (&v)[16], int which) {
        u128 w[16];
#pragma unroll
        for (int i = 0; i < 16; i++) w[i] = mul64(v[i], xn);
        const u128 sum = half_sums(w);
        if (!(lane & 1)) rows[which][wave][16 * (lane >> 5) + ((lane >> 1) & 15)] = sum;
    };
    if (live) {
        u128 x[16], s[16];
        load(L.B[0], s);
        convert(s, 1, dst, J.planeR);
        load(L.B[1], x);
        convert(x, 1, dst + RNS_N * J.planeR, J.planeR);
#pragma unroll
        for (int i = 0; i < 16; i++) s[i] = add(s[i], x[i]);
        load(L.Y[0], x);
#pragma unroll
        for (int i = 0; i < 16; i++) s[i] = sub(x[i], s[i]);
        load(L.Y[1], x);
#pragma unroll
        for (int i = 0; i < 16; i++) {
            x[i] = add(s[i], x[i]);  // U
            if (i < kn) {
                st_nt(L.U + e0 + (int64_t)i * N, le, x[i]);
                if (check) chk[2] = mad64(chk[2], x[i], sdraw(kcu, (uint64_t)(e0 + (int64_t)i * N) + le));
            }
        }
        if (compact) row_sums(x, 0);
        convert(x, 1, dst + 2 * RNS_N * J.planeR, J.planeR);
        // the tag shares: compressed (CompactTag) or converted (SPDZ2k), and checked
        if (check || compact || tags) {
#pragma unroll
            for (int p = 0; p < 2; p++) {
                load(L.tB[p], x);
                if (check) {
                    load(L.tY[p], s);
#pragma unroll
                    for (int i = 0; i < 16; i++)
                        chk[p] = mad64(chk[p], sub(s[i], x[i]), sdraw(kcu, (uint64_t)(e0 + (int64_t)i * N) + le));
                }
                if (compact) row_sums(x, 1 + p);
                if (tags) convert(x, 1, J.right_tag + (dst - J.right) + p * RNS_N * J.planeR, J.planeR);
            }
        }
    } else if (compact) {
        for (int i = lane; i < 96; i += 64) rows[i / 32][wave][i & 31] = u128{0, 0};
    }
    if (compact) {
        __syncthreads();
        const int which = threadIdx.x / 32, r = threadIdx.x & 31, k = k_base + 32 * ks + r;
        if (which < 3 && k < K) {
            u128 v = rows[which][0][r];
#pragma unroll
            for (int w = 1; w < WAVES; w++) v = add(v, rows[which][w][r]);
            atomic_add128(L.cvec + (which == 0 ? o.Uc : which == 1 ? o.tBc0 : o.tBc1) + k, v);
        }
    }
    if (check) wave_accumulate_limbs<3>(chk, L.uc + 12 * ((wg * WAVES + wave) % RP_COPIES));
}

// Left operands: opens E = ([X]_0 - [A]_0) + ([X]_1 - [A]_1) and writes the
// planes of E (wavefront 0), A_0 + E (1), [A]_1 (2) and, with TAGS (SPDZ2k),
// of [tA]_p + [Delta]_p E (3 + p); the pass over M x K then reads E.  Elements
// are loaded along k and transposed through LDS.
template <bool TAGS>
__global__ __launch_bounds__(TAGS ? 320 : 192) void k_rns_open_left(const LayerDev *__restrict__ Ls,
                                                                    const RnsOpen *__restrict__ jobs, int njobs, int chunk) {
    __shared__ __attribute__((aligned(16))) u128 raw[TAGS ? 5 : 3][1024];
    const int wg = blockIdx.x;
    int lo = 0, hi = njobs - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (jobs[mid].wg_left <= wg) lo = mid; else hi = mid - 1;
    }
    const RnsOpen &J = jobs[lo];
    const LayerDev &L = Ls[J.layer];
    const int local = wg - J.wg_left, lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int K = (int)L.K, M = (int)L.M, k_base = chunk * J.Kc, frags = (min(J.Kc, K - k_base) + 63) / 64 * 2;
    const int mb = local / J.kt, ks = local - mb * J.kt;
    if (ks >= frags) return;
    const int k = k_base + 32 * ks + (lane & 31);
    const u128 *ta = TAGS && wave >= 3 ? L.tA[wave - 3] : nullptr;
    const uint64_t delta = TAGS && wave >= 3 ? L.delta[wave - 3] : 0;
#pragma unroll
    for (int g = 0; g < 4; g++) {
        u128 x0[4], x1[4], a0[4], a1[4], t[4];
#pragma unroll
        for (int i = 0; i < 4; i++) {
            const int m = 32 * mb + 2 * (4 * g + i) + (lane >> 5);
            x0[i] = x1[i] = a0[i] = a1[i] = t[i] = u128{0, 0};
            if (k < K && m < M) {
                const int64_t e = (int64_t)m * K + k;
                a1[i] = ld(L.A[1], e);
                if (wave != 2) {
                    x0[i] = ld(L.X[0], e);
                    x1[i] = ld(L.X[1], e);
                    a0[i] = ld(L.A[0], e);
                }
                if (TAGS && wave >= 3) t[i] = ld(ta, e);
            }
        }
#pragma unroll
        for (int i = 0; i < 4; i++) {
            const int r = 2 * (4 * g + i) + (lane >> 5), m = 32 * mb + r;
            u128 v = a1[i];
            if (wave != 2) {
                const u128 x = sub(add(x0[i], x1[i]), a1[i]);  // A_0 + E
                v = wave == 1 ? x : sub(x, a0[i]);
                if (wave == 0 && k < K && m < M) st(L.E, (int64_t)m * K + k, v);
                if (TAGS && wave >= 3) v = mad64(t[i], v, delta);
            }
            raw[wave][r * 32 + ((lane & 31) ^ (r & 15))] = v;
        }
    }
    wave_sync();
    const int r = lane & 31;
    u128 x[16];
#pragma unroll
    for (int i = 0; i < 16; i++) x[i] = raw[wave][r * 32 + ((16 * (lane >> 5) + i) ^ (r & 15))];
    uint8_t *dst = wave < 3 ? J.left + wave * RNS_N * J.planeL : J.left_tag + (wave - 3) * RNS_N * J.planeL;
    convert(x, 0, dst + ((int64_t)(ks >> 1) * J.mb + mb) * 2048 + (ks & 1) * 1024 + lane * 16, J.planeL);
}

hipError_t launch_rns_open(const LayerDev *L, const RnsOpen *jobs, int njobs, int wgs_left, int wgs_right, int flags, int chunk,
                           hipStream_t st) {
    if (njobs <= 0) return hipSuccess;
    if (wgs_left > 0 && (flags & F_SPDZ))
        hipLaunchKernelGGL(k_rns_open_left<true>, dim3(wgs_left), dim3(320), 0, st, L, jobs, njobs, chunk);
    else if (wgs_left > 0)
        hipLaunchKernelGGL(k_rns_open_left<false>, dim3(wgs_left), dim3(192), 0, st, L, jobs, njobs, chunk);
    if (wgs_right > 0) hipLaunchKernelGGL(k_rns_open_right, dim3(wgs_right), dim3(256), 0, st, L, jobs, njobs, flags, chunk);
    return hipGetLastError();
}

// ---------------------------------------------------------------- products of residues
typedef __attribute__((address_space(3))) void lds_void;

constexpr int STAGES = 3;
constexpr int EXACT_TERMS = 1024;  // 1024 * 127^2 + 127 < 2^24 (products modulo 256 need no quotient)

// acc (|acc| < 2^28) less a multiple of m near it
__device__ __forceinline__ int reduce(int acc, float inv, int m) {
    const float t = __builtin_fmaf((float)acc, inv, 12582912.0f);
    return acc - __mul24(__float_as_int(t) - 0x4B400000, m);
}

// all LDS reads returned and at most n copies outstanding
#define WAIT_VM_LGKM(n) __builtin_amdgcn_s_waitcnt(0x0070 | (n))
__device__ __forceinline__ void barrier() {
    __asm__ volatile("" ::: "memory");
    __builtin_amdgcn_s_barrier();
    __asm__ volatile("" ::: "memory");
}

// Workgroup: one modulus, 64 WI x 64 WJ outputs (32 WI x 32 WJ per wavefront,
// 2 x 2 wavefronts) of OUTS products at once, which share the operand that is
// common in each segment.
template <int OUTS, int WI, int WJ>
struct Shape {
    static constexpr int BI = 2 * WI, BJ = 2 * WJ;  // 32-row blocks of the workgroup tile
    // blocks of a stage: segment 0 reads one left operand and OUTS right ones, segment 1 OUTS left and one right
    static constexpr int B0 = BI + OUTS * BJ, B1 = OUTS * BI + BJ, BMAX = B0 > B1 ? B0 : B1, BMIN = B0 < B1 ? B0 : B1;
    static constexpr int STAGE_BYTES = BMAX * 2048;
    static_assert(BI % 4 == 0 && BJ % 4 == 0, "blocks are copied by four wavefronts");
};

template <int OUTS, int WI, int WJ>
__device__ __forceinline__ void rns_tile(const RnsProb &P, int q, int tm, int tn, int chunk, uint8_t *lds) {
    using S = Shape<OUTS, WI, WJ>;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int wm = wave >> 1, wn = wave & 1;
    const int mb = P.mb, nb = P.nb;
    const int kc = min(P.Kc, P.K - chunk * P.Kc), nst = (kc + RNS_BK - 1) / RNS_BK, total = nst * P.segs;
    const int mod = g_rns.m[q];
    const float inv = g_rns.inv[q];

    v16i acc[OUTS][WI][WJ];
    uint8_t *res = P.res + ((int64_t)q * OUTS) * mb * nb * 1024;
    // the output tiles of this wavefront (a tile past the last block is not stored)
    const int rm0 = tm * S::BI + wm * WI, rn0 = tn * S::BJ + wn * WJ;
    auto tile_off = [&](int o, int i, int j) { return (((int64_t)o * mb + rm0 + i) * nb + rn0 + j) * 1024 + lane * 16; };
    if (chunk > 0) {
#pragma unroll
        for (int o = 0; o < OUTS; o++)
#pragma unroll
            for (int i = 0; i < WI; i++)
#pragma unroll
                for (int j = 0; j < WJ; j++) {
                    ct_u32x4 v = ct_u32x4{0, 0, 0, 0};
                    if (rm0 + i < mb && rn0 + j < nb) v = *global_ptr<ct_u32x4>(res + tile_off(o, i, j));
                    const uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
                    for (int r = 0; r < 16; r++) acc[o][i][j][r] = (int)(int8_t)(w[r >> 2] >> (8 * (r & 3)));
                }
    } else {
#pragma unroll
        for (int o = 0; o < OUTS; o++)
#pragma unroll
            for (int i = 0; i < WI; i++)
#pragma unroll
                for (int j = 0; j < WJ; j++) acc[o][i][j] = v16i{0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0};
    }

    // The blocks this wavefront copies of each stage, block 4 t + wave of the
    // stage: sources in the first segment, then in the second
    const int64_t stepL = (int64_t)mb * 2048, stepR = (int64_t)nb * 2048;
    auto left = [&](const uint8_t *base, int b) { return base + q * P.planeL + (int64_t)min(tm * S::BI + b, mb - 1) * 2048; };
    auto right = [&](const uint8_t *base, int b) { return base + q * P.planeR + (int64_t)min(tn * S::BJ + b, nb - 1) * 2048; };
    const uint8_t *src[S::BMAX / 4], *src1[S::B1 / 4];
#pragma unroll
    for (int t = 0; t < S::BMAX / 4; t++) {
        const int b = 4 * t + wave, o = (4 * t - S::BI) / S::BJ;
        src[t] = 4 * t < S::BI ? left(P.L0, b) : right(o == 0 || OUTS == 1 ? P.R0 : P.R1, b - S::BI - o * S::BJ);
    }
#pragma unroll
    for (int t = 0; t < S::B1 / 4; t++) {
        const int b = 4 * t + wave, o = 4 * t / S::BI;
        src1[t] = o < OUTS ? left(o == 0 ? P.L1 : P.L2, b - o * S::BI) : right(P.R2, b - OUTS * S::BI);
    }
    auto copy = [&](const uint8_t *from, uint8_t *dst) {
#pragma unroll
        for (int f = 0; f < 2; f++)
            __builtin_amdgcn_global_load_lds((const void *)(from + f * 1024 + lane * 16), (lds_void *)(dst + f * 1024), 16, 0, 0);
    };
    auto issue = [&](int s, uint8_t *stage) {
        const bool first = s < nst;
        if (s == nst) {
#pragma unroll
            for (int t = 0; t < S::B1 / 4; t++) src[t] = src1[t];
        }
#pragma unroll
        for (int t = 0; t < S::BMAX / 4; t++) {
            if (4 * t < S::BMIN || first == (S::B0 > S::B1)) copy(src[t], stage + (4 * t + wave) * 2048);
            const int64_t step0 = 4 * t < S::BI ? stepL : stepR, step1 = 4 * t < OUTS * S::BI ? stepL : stepR;
            src[t] += first ? step0 : step1;
        }
    };
    constexpr int COPIES = S::BMIN / 4 * 2;  // of a stage, at least
    const int fa = wm * WI * 2048 + lane * 16, fb = wn * WJ * 2048 + lane * 16;

    // Software pipeline.  A stage has two k halves; while the products of one
    // half run, the fragments of the next are read.  Before the products of
    // the second half every wavefront holds the stage's last fragments and
    // meets the others at a barrier: the stage after is then complete in LDS,
    // and the copies of the third stage after go where this one was.
#pragma unroll
    for (int s = 0; s < STAGES; s++)
        if (s < total) issue(s, lds + s * S::STAGE_BYTES);
    struct Frags {
        v4i a[OUTS][WI], b[OUTS][WJ];  // one of them for the shared operand
    };
    Frags fx, fy;  // of the first and the second half
    auto read = [&](Frags &f, const uint8_t *stage, int h, bool second) {
#pragma unroll
        for (int o = 0; o < (second ? OUTS : 1); o++)
#pragma unroll
            for (int i = 0; i < WI; i++)
                f.a[o][i] = *reinterpret_cast<const v4i *>(stage + (o * S::BI + i) * 2048 + fa + h * 1024);
#pragma unroll
        for (int o = 0; o < (second ? 1 : OUTS); o++)
#pragma unroll
            for (int j = 0; j < WJ; j++)
                f.b[o][j] = *reinterpret_cast<const v4i *>(stage + ((second ? OUTS : 1) * S::BI + o * S::BJ + j) * 2048 + fb + h * 1024);
    };
    // the products of one half: its first WJ, or the others
    auto multiply = [&](const Frags &f, bool second, bool first) {
#pragma unroll
        for (int o = 0; o < OUTS; o++)
#pragma unroll
            for (int i = 0; i < WI; i++)
#pragma unroll
                for (int j = 0; j < WJ; j++)
                    if ((o == 0 && i == 0) == first)
                        acc[o][i][j] = __builtin_amdgcn_mfma_i32_32x32x32_i8(f.a[second ? o : 0][i], f.b[second ? 0 : o][j],
                                                                             acc[o][i][j], 0, 0, 0);
    };
    int cur = 0;
    if (rm0 >= mb || rn0 >= nb) {
        // no outputs: this wavefront only copies for the others
        for (int s = -1; s + 1 < total; s++) {
            if (s + 2 < total) WAIT_VM_LGKM(COPIES); else WAIT_VM_LGKM(0);
            barrier();
            if (s >= 0 && s + STAGES < total) issue(s + STAGES, lds + cur * S::STAGE_BYTES);
            if (s >= 0) cur = cur == STAGES - 1 ? 0 : cur + 1;
        }
        return;
    }

    // Stages [s0, s1) of one segment.
    auto run = [&](int s0, int s1, auto seg) {
        constexpr bool second = decltype(seg)::value;
        // stage s + 1 has landed (s + 2 may still be on its way) and every
        // wavefront holds the last fragments of stage s
        auto next_stage = [&](int s) {
            if (s + 2 < total) WAIT_VM_LGKM(COPIES); else WAIT_VM_LGKM(0);
            barrier();
            if (s >= 0) {
                if (s + STAGES < total) issue(s + STAGES, lds + cur * S::STAGE_BYTES);
                cur = cur == STAGES - 1 ? 0 : cur + 1;
            }
            read(fx, lds + cur * S::STAGE_BYTES, 0, second);
            __builtin_amdgcn_sched_barrier(0);
        };
        next_stage(s0 - 1);
        for (int s = s0; s < s1; s++) {
            // the first products wait for fx (read long before): only then the reads of fy,
            // which a wait in front of them would include
            multiply(fx, second, true);
            __builtin_amdgcn_sched_barrier(0);
            read(fy, lds + cur * S::STAGE_BYTES, 1, second);
            __builtin_amdgcn_sched_barrier(0);
            multiply(fx, second, false);
            __builtin_amdgcn_sched_barrier(0);
            if (s + 1 < s1) next_stage(s);
            multiply(fy, second, true);
            multiply(fy, second, false);
            __builtin_amdgcn_sched_barrier(0);
        }
    };
    run(0, nst, std::false_type());
    if (total > nst) run(nst, total, std::true_type());

    // up to EXACT_TERMS terms the sums are below 2^24 and exact as floats; the
    // quotient of a larger one is off by a few units, which a first reduction
    // (to 2^9 and less) removes
    const bool wide = kc * P.segs > EXACT_TERMS;
    const uint32_t cmp = (uint32_t)(256 - mod) & 255;
#pragma unroll
    for (int o = 0; o < OUTS; o++)
#pragma unroll
        for (int i = 0; i < WI; i++)
#pragma unroll
            for (int j = 0; j < WJ; j++) {
                if (wide) {
#pragma unroll
                    for (int r = 0; r < 16; r++) acc[o][i][j][r] = reduce(acc[o][i][j][r], inv, mod);
                }
                uint32_t w[4];
#pragma unroll
                for (int d = 0; d < 4; d++) {
                    uint32_t b[4];
#pragma unroll
                    for (int r = 0; r < 4; r++) {
                        // low byte of acc - q m: the magic constant's 2^22 times (256 - m) leaves it alone
                        const int v = acc[o][i][j][4 * d + r];
                        const float t = __builtin_fmaf((float)v, inv, 12582912.0f);
                        b[r] = __umul24((uint32_t)__float_as_int(t), cmp) + (uint32_t)v;
                    }
                    w[d] = pack4(b[0], b[1], b[2], b[3]);
                }
                if (rm0 + i < mb && rn0 + j < nb)
                    __builtin_nontemporal_store(ct_u32x4{w[0], w[1], w[2], w[3]}, global_ptr<ct_u32x4>(res + tile_off(o, i, j)));
            }
}

// Bound by the matrix cores and the LDS that feeds them: 1.88e15 int8
// operations a second on a 2048^3 layer (slope between sizes 2.2e15), where the
// digit products ran at 1.75e15 but needed 136 products, not 36: 6.54 ms then,
// 2.93 ms now for 2048 x 4096 x 2048.  At M = 128 the planes' bytes bind
// (encoder layers: 1.1e15).  128 x 128 outputs of two products that share E and
// U, two workgroups a compute unit: 128 x 256 with one wavefront per SIMD gave
// 1.36e15, the launch's ends no longer hidden.  Blocks are dispatched
// round-robin over the XCDs (block b on XCD b % 8): a modulus of a problem
// stays on one XCD, so its operand planes are fetched into one L2 only.  A
// launch takes the problems of one kind (OUTS products).
template <int OUTS, int WI, int WJ, int OCC>
__global__ __launch_bounds__(256, OCC) void k_rns_gemm(const RnsProb *__restrict__ probs, int nprobs, int chunk) {
    __shared__ __attribute__((aligned(1024))) uint8_t lds[STAGES * Shape<OUTS, WI, WJ>::STAGE_BYTES];
    const int x = blockIdx.x & 7, idx = blockIdx.x >> 3;
    int lo = 0, hi = nprobs - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (probs[mid].begin[x] <= idx) lo = mid; else hi = mid - 1;
    }
    const RnsProb &P = probs[lo];
    const int tiles = P.tiles_m * P.tiles_n, local = idx - P.begin[x];
    const int qi = local / tiles, q = ((x - P.rot) & 7) + 8 * qi;
    if (q >= RNS_N) return;
    // groups of 8 row tiles, column by column
    const int t = local - qi * tiles, grp = t / (8 * P.tiles_n), gm = min(8, P.tiles_m - 8 * grp);
    const int r = t - grp * 8 * P.tiles_n, tn = r / gm, tm = 8 * grp + r - tn * gm;
    rns_tile<OUTS, WI, WJ>(P, q, tm, tn, chunk, lds);
}

hipError_t launch_rns_gemm(int outs, const RnsProb *probs, int nprobs, int blocks_x, int chunk, hipStream_t st) {
    if (nprobs <= 0 || blocks_x <= 0) return hipSuccess;
    if (outs == 2)
        hipLaunchKernelGGL((k_rns_gemm<2, 2, RNS_TN / 64, RNS_TN == 128 ? 2 : 1>), dim3(8 * blocks_x), dim3(256), 0, st, probs, nprobs, chunk);
    else
        hipLaunchKernelGGL((k_rns_gemm<1, 2, RNS_TN / 64, 2>), dim3(8 * blocks_x), dim3(256), 0, st, probs, nprobs, chunk);
    return hipGetLastError();
}

// ---------------------------------------------------------------- residues to elements
// P = sum_q y_q (M / m_q) - t M with y_q = P (M / m_q)^-1 mod m_q (any
// representative; the inverse is part of the left operand's residues) and
// t = round(sum_q y_q / m_q), all mod 2^128.  Bound by HBM: 68 bytes an output
// (36 residues, constant term, result), 3.9 TB/s at 2048 x 2048 x 2.  The sums of the digits of
// (M / m_q) mod 2^128 and of 2^24 / m_q weighted by y_q come from the matrix
// cores; one wavefront reconstructs a 32 x 32 tile, 16 outputs per lane.
__device__ __forceinline__ void transpose4(const uint32_t (&a)[4], uint32_t (&b)[4]) {
    const uint32_t t0 = __builtin_amdgcn_perm(a[1], a[0], 0x05010400u), t1 = __builtin_amdgcn_perm(a[1], a[0], 0x07030602u);
    const uint32_t t2 = __builtin_amdgcn_perm(a[3], a[2], 0x05010400u), t3 = __builtin_amdgcn_perm(a[3], a[2], 0x07030602u);
    b[0] = __builtin_amdgcn_perm(t2, t0, 0x05040100u);
    b[1] = __builtin_amdgcn_perm(t2, t0, 0x07060302u);
    b[2] = __builtin_amdgcn_perm(t3, t1, 0x05040100u);
    b[3] = __builtin_amdgcn_perm(t3, t1, 0x07060302u);
}

__global__ __launch_bounds__(256, 2) void k_rns_fold(const RnsProb *__restrict__ probs, int nprobs, int items) {
    const int lane = threadIdx.x & 63;
    const int item = __builtin_amdgcn_readfirstlane(blockIdx.x * 4 + (threadIdx.x >> 6));
    if (item >= items) return;
    int lo = 0, hi = nprobs - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (probs[mid].fold_begin <= item) lo = mid; else hi = mid - 1;
    }
    const RnsProb &P = probs[lo];
    const int tiles = P.mb * P.nb, local = item - P.fold_begin;
    const int o = local / tiles, tile = local - o * tiles, rm = tile / P.nb, rn = tile - rm * P.nb;
    const CT_GLOBAL ct_u32x4 *src = global_ptr<ct_u32x4>(P.res + ((int64_t)o * tiles + tile) * 1024) + lane;
    const int64_t step = (int64_t)P.outs * tiles * 64;  // 16 bytes a lane, per modulus
    ct_u32x4 y[RNS_N];
#pragma unroll
    for (int q = 0; q < RNS_N; q++) y[q] = src[q * step];
    v4i wf[GROUPS], wq[GROUPS];
#pragma unroll
    for (int g = 0; g < GROUPS; g++) {
        wf[g] = *reinterpret_cast<const v4i *>(&g_rns.fold[g][lane * 16]);
        wq[g] = *reinterpret_cast<const v4i *>(&g_rns.quot[g][lane * 16]);
    }
    const v16i zero = {0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0};
    constexpr x128 MALL = rns_others(-1);
    const u128 mall{(uint64_t)MALL, (uint64_t)(MALL >> 64)};
    const u128 *base = P.base[o];
    u128 *out = P.out[o];
    const int col = rn * 32 + (lane & 31);
#pragma unroll
    for (int d = 0; d < 4; d++) {  // outputs 4 d .. 4 d + 3: rows 8 d + 4 (lane / 32) + e
        uint32_t b[GROUPS * 4][4];
#pragma unroll
        for (int h = 0; h < RNS_N / 4; h++) {
            uint32_t a[4];
#pragma unroll
            for (int j = 0; j < 4; j++) {
                const ct_u32x4 v = y[4 * h + j];
                a[j] = d == 0 ? v.x : d == 1 ? v.y : d == 2 ? v.z : v.w;
            }
            transpose4(a, b[h]);
        }
#pragma unroll
        for (int h = RNS_N / 4; h < GROUPS * 4; h++)
#pragma unroll
            for (int e = 0; e < 4; e++) b[h][e] = 0;
#pragma unroll
        for (int e = 0; e < 4; e++) {
            const int row = rm * 32 + 8 * d + 4 * (lane >> 5) + e;
            const bool ok = row < P.M && col < P.N;
            const int64_t idx = (int64_t)row * P.N + col;
            u128 v = u128{0, 0};
            if (ok && base) v = ld_nt(base, idx);
            v16i D = zero, Q = zero;
#pragma unroll
            for (int g = 0; g < GROUPS; g++) {
                const v4i yb = {(int)b[4 * g][e], (int)b[4 * g + 1][e], (int)b[4 * g + 2][e], (int)b[4 * g + 3][e]};
                D = __builtin_amdgcn_mfma_i32_32x32x32_i8(wf[g], yb, D, 0, 0, 0);
                Q = __builtin_amdgcn_mfma_i32_32x32x32_i8(wq[g], yb, Q, 0, 0, 0);
            }
            const int t = (int)((uint32_t)Q[0] + ((uint32_t)Q[1] << 8) + ((uint32_t)Q[2] << 16) + (1u << 23)) >> 24;
            // sum_j D_j 2^{8 j}: four limbs of 32 bits, each from four digit sums
            int64_t l[4];
#pragma unroll
            for (int i = 0; i < 4; i++)
                l[i] = (int64_t)(D[4 * i] + D[4 * i + 1] * 256) + (int64_t)(D[4 * i + 2] + D[4 * i + 3] * 256) * 65536;
            const uint64_t a01 = (uint64_t)l[0] + ((uint64_t)l[1] << 32);  // low 64 bits; the carry below
            const uint64_t c01 = (uint64_t)((l[1] + (l[0] >> 32)) >> 32);
            const u128 s{a01, (uint64_t)l[2] + ((uint64_t)l[3] << 32) + c01};
            const int64_t ts = t;
            const u128 tm = mul(mall, u128{(uint64_t)ts, (uint64_t)(ts >> 63)});
            v = add(v, sub(s, tm));
            if (ok) st_nt(out, idx, v);
        }
    }
}

hipError_t launch_rns_fold(const RnsProb *probs, int nprobs, int items, hipStream_t st) {
    if (nprobs <= 0 || items <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_rns_fold, dim3((items + 3) / 4), dim3(256), 0, st, probs, nprobs, items);
    return hipGetLastError();
}

}  // namespace ct
