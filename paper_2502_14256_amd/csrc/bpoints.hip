// Point sets without the structure the fast transforms need; they feed QMC
// means (the RQMC estimate over given coordinates, ldk_rqmc_points).
//
// Digital sequences in a prime base b (Sec. 4.3 allows any prime base):
// point i has the base-b digits a_k of i (least significant first) and the
// digits z_t = sum_k C[t][k] a_k mod b, digit t weighing b^-(t+1).
//   Faure: one prime b >= d; dimension j (from 0) uses C = P^j mod b, P the
//   upper-triangular Pascal matrix, whose entries are binom(k, t) j^(k-t).
//   Halton (Sec. 4.4): dimension j uses the (j+1)-th prime and C = I, so z is
//   the digit expansion of the radical inverse of i.
// Randomizations, each optional, in this order: linear matrix scrambling
// z <- S z mod b (S lower triangular with a nonzero diagonal), a permutation
// of the digit values per digit position, a digital shift z_t + delta_t mod
// b.  T digits are kept, the largest T with b^T <= 2^53, so the coordinate is
// the integer v = sum_t z_t b^(T-1-t) < 2^53 divided by b^T, rounded once.
//
// A block takes 64 or 128 consecutive indices of one replication, one or two
// per lane; its eight waves split the dimensions.  The digits of an index live
// in registers, four to a 32-bit word, so a row of S (or of Faure's C) times the
// digit vector is one v_dot4_u32_u8 per word; the sum stays below 2^21 and is
// reduced mod b by a 32-bit reciprocal (32-bit products run at full rate here).
// Four output digits make one 32-bit integer before they join the FP64 Horner
// sum.  The Faure matrices come packed from a small kernel, formed once per call
// into the workspace.
//
// Nested uniform scrambling of a base-2 net (Sec. 4.3, NUS): the point word
// z = C i (64 digits), then digit t = 1..64 is flipped when the top bit of
// mix64(key XOR seed) is set, key = 2^(t-1) + the unscrambled digits before
// t as an integer; mix64 is the SplitMix64 finaliser (Steele, Lea and Flood,
// 2014, with Stafford's Mix13 constants).  For base 2 a permutation of the
// digit values is the identity or the flip, and this draws one independently
// for every prefix, as nested uniform scrambling asks.
#include "common.hpp"

// dynamic LDS of the tile kernels: the output tile
extern __shared__ __align__(16) unsigned char g_bp_lds[];

namespace ldk {

namespace {

constexpr int BP_T = LDK_BDIGITS_MAX;  // digit rows of the scramble layouts
constexpr int BP_MAX_D = 54;    // the first 54 primes are below 256
constexpr int BP_KMAX = 32;     // index digits (i < 2^32)
constexpr int BP_QW = BP_KMAX / 4;  // words of a packed digit row
constexpr int BP_TT = 512;      // threads of a tile block (Halton, Faure)
constexpr int BP_WAVES = BP_TT / 64;
constexpr int BP_P = 64;        // points per tile block and point of a lane
constexpr int BP_DCH = 64;      // dimensions per output tile
constexpr size_t LDS_PER_CU = 163840;

struct BpArgs {
    int d, flags;
    int64_t n_min, cnt;
    uint32_t lms_off;  // byte offset of lms within its first word
    // per dimension (Halton; Faure uses entry 0 for every dimension), 32-bit
    // words so that a uniform index reads them with scalar loads
    uint32_t base[BP_MAX_D], T[BP_MAX_D], M[BP_MAX_D];
    uint32_t inv[BP_MAX_D];  // ceil(2^32 / b)
    double rb[BP_MAX_D];     // 1 / b, rounded
    double bT[BP_MAX_D], ibT[BP_MAX_D];  // b^T, exact; 1 / b^T, rounded
    double bTM[BP_MAX_D];    // b^(T - min(M, T)), exact
    uint32_t small;          // every index below 2^24: digits by one reciprocal product each
    // Halton: wave w computes dimensions ord[q] for wbeg[w] <= q < wbeg[w + 1]
    uint32_t ord[BP_MAX_D], wbeg[BP_WAVES + 1];
};

// Faure matrix of dimension j = blockIdx.x, packed for the point kernel:
// C[t][k] = binom(k, t) j^(k-t) mod b for t <= k < T (zero elsewhere), rows
// t < 4 mj and columns k < 4 mj, four columns to a word: [d][4 mj][mj].
__global__ __launch_bounds__(64) void k_faure_cmat(int b, int T, int mj, uint32_t *__restrict__ cmat)
{
    __shared__ uint8_t binom[BP_T][BP_T];  // [k][t]
    __shared__ uint8_t pw[BP_T];
    const int j = blockIdx.x, t = threadIdx.x;
    if (t == 0) {
        int p = 1 % b;
        for (int e = 0; e < T; ++e) {
            pw[e] = (uint8_t)p;
            p = (p * (j % b)) % b;
        }
    }
    // Pascal's rule, one row k at a time: binom(k, t) = binom(k-1, t-1) + binom(k-1, t)
    for (int k = 0; k < T; ++k) {
        if (t < T) {
            int v;
            if (t > k) v = 0;
            else if (t == 0 || t == k) v = 1 % b;
            else v = (binom[k - 1][t - 1] + binom[k - 1][t]) % b;
            binom[k][t] = (uint8_t)v;
        }
        __syncthreads();
    }
    if (t < 4 * mj)
        for (int q = 0; q < mj; ++q) {
            uint32_t w = 0;
            for (int c = 0; c < 4; ++c) {
                const int k = 4 * q + c;
                if (t < T && k < T && k >= t) w |= (uint32_t)((binom[k][t] * pw[k - t]) % b) << (8 * c);
            }
            cmat[((size_t)j * 4 * mj + t) * mj + q] = w;
        }
}

// s mod b for s < 2^24 and b <= 251: with inv = ceil(2^32 / b), e = inv b -
// 2^32 < b gives s e < 2^32, so floor(s inv / 2^32) = floor(s / b) exactly.
__device__ __forceinline__ uint32_t mod_b(uint32_t s, uint32_t b, uint32_t inv)
{
    return s - __umul24(__umulhi(s, inv), b);
}

// floor(x / b) and the remainder for x < 2^32: x RN(1/b) in FP64 lies within
// 2^-20 of x / b, below the next integer (the fraction of x / b is at most
// 1 - 1/b), so truncation is exact except at multiples of b, where it can
// fall one short.
__device__ __forceinline__ uint32_t div_b(uint32_t x, uint32_t b, double rb, uint32_t &rem)
{
    uint32_t q = (uint32_t)((double)x * rb);
    uint32_t r = x - q * b;
    if (r >= b) {
        r -= b;
        ++q;
    }
    rem = r;
    return q;
}

// Base-b digits of an index, least significant first, four to a word
// (digit k in byte k % 4 of word k / 4); M digits, the rest zero.
template <int MJ>
__device__ __forceinline__ void index_digits_packed(const BpArgs &a, int j, uint32_t x, uint32_t (&z)[MJ])
{
    const uint32_t b = a.base[j], inv = a.inv[j];
    const int M = a.M[j];
    const double rb = a.rb[j];
#pragma unroll
    for (int q = 0; q < MJ; ++q) z[q] = 0;
#pragma unroll
    for (int k = 0; k < 4 * MJ; ++k)
        if (k < M) {
            uint32_t dg;
            if (a.small) {
                const uint32_t q = __umulhi(x, inv);
                dg = x - __umul24(q, b);
                x = q;
            } else {
                x = div_b(x, b, rb, dg);
            }
            z[k >> 2] |= dg << (8 * (k & 3));
        }
}

// Lane t (t < T) fetches row t of S, packed four columns to a word over the
// columns below 4 MJ, keeping only k <= t (S is lower triangular): the row's
// bytes start o bytes past the word array W, and MJ + 1 words from the word
// boundary at or below cover them (within the row's 53 bytes).  Lanes t >= T
// hold zeros.
template <int MJ>
__device__ __forceinline__ void lane_row(const uint32_t *__restrict__ W, uint64_t o, int t, int T,
                                         uint32_t (&row)[MJ])
{
#pragma unroll
    for (int q = 0; q < MJ; ++q) row[q] = 0;
    if (t >= T) return;
    uint32_t wd[MJ + 1];
#pragma unroll
    for (int q = 0; q <= MJ; ++q) wd[q] = W[(o >> 2) + q];
    const uint32_t sh = (uint32_t)(o & 3) * 8;
#pragma unroll
    for (int q = 0; q < MJ; ++q) {
        const int lo = 4 * q;
        uint32_t x = (uint32_t)((((uint64_t)wd[q + 1] << 32) | wd[q]) >> sh);
        if (t < lo) x = 0;
        else if (t < lo + 3) x &= 0xffffffffu >> (8 * (3 - (t - lo)));
        row[q] = x;
    }
}

// K <= 4 consecutive output digits of a coordinate of each of the lane's P
// points: their values g before the permutation go through pi_t and + delta_t
// mod b, and join the Horner sum as one integer below b^K < 2^32.
// (The permutation's bytes held four to a lane and moved by ds_bpermute
// measured slower than the K P gathers in flight: 186 -> 213 us with every
// scramble on at R = 16, n = 2^15, d = 52.)
template <int K, int F, int P>
__device__ __forceinline__ void digits_join(uint32_t (&g)[P][K], uint32_t dlane, const uint8_t *prow, int t0,
                                            uint32_t b, double bK, double (&v)[P])
{
    if constexpr (F & LDK_BR_DP) {
#pragma unroll
        for (int p = 0; p < P; ++p)
#pragma unroll
            for (int k = 0; k < K; ++k) g[p][k] = prow[(t0 + k) * 256 + g[p][k]];
    }
#pragma unroll
    for (int p = 0; p < P; ++p) {
        if constexpr (F & LDK_BR_DS) {
#pragma unroll
            for (int k = 0; k < K; ++k) {
                g[p][k] += __builtin_amdgcn_readlane(dlane, t0 + k);
                g[p][k] = min(g[p][k], g[p][k] - b);  // the difference wraps where it is negative
            }
        }
        uint32_t acc = g[p][0];
#pragma unroll
        for (int k = 1; k < K; ++k) acc = __umul24(acc, b) + g[p][k];  // acc below b^3 < 2^24
        v[p] = fma(v[p], bK, (double)acc);
    }
}
// Digits t0 .. t0 + K - 1 (all below T) of S z mod b: row t of S is lane t's,
// read by v_readlane (once for the P points).
template <int K, int MJ, int F, int P>
__device__ __forceinline__ void digits_lms(const uint32_t (&srows)[MJ], uint32_t dlane, const uint8_t *prow,
                                           const uint32_t (&z)[P][MJ], int t0, uint32_t b, uint32_t inv, double bK,
                                           double (&v)[P])
{
    uint32_t g[P][K];
#pragma unroll
    for (int k = 0; k < K; ++k) {
        uint32_t s[P] = {};
#pragma unroll
        for (int q = 0; q < MJ; ++q) {
            const uint32_t w = __builtin_amdgcn_readlane(srows[q], t0 + k);
#pragma unroll
            for (int p = 0; p < P; ++p) s[p] = __builtin_amdgcn_udot4(w, z[p][q], s[p], false);
        }
#pragma unroll
        for (int p = 0; p < P; ++p) g[p][k] = mod_b(s[p], b, inv);
    }
    digits_join<K, F, P>(g, dlane, prow, t0, b, bK, v);
}

// Coordinates of the lane's P points in dimension j of replication r (rj = r d
// + j, parameters at index p): digit t of the output is w_t = (S z)_t mod b,
// then pi_t(w_t), then + delta_t mod b (each step as the flags F ask);
// Horner's rule in FP64 is exact (every partial sum is an integer below 2^53)
// and the one division rounds.  The wave's lanes first fetch one row of S and
// one delta each.  Digits go four at a time, as one 32-bit integer each four.
// Without S the digits past the index's own M are zero before the
// permutation, the same for every lane (skipped where nothing maps them).
// v / b^T from the rounded reciprocal: two corrections by the exact remainder
// (the first leaves less than an ulp, the second then rounds correctly).
template <int MJ, int F, int P>
__device__ __forceinline__ void coordinate(const BpArgs &a, int pi, const uint32_t *__restrict__ lmsw,
                                           const uint8_t *__restrict__ shift,
                                           const uint8_t *__restrict__ perm, const uint32_t (&z)[P][MJ],
                                           size_t rj, int lane, double (&x)[P])
{
    constexpr bool LMS = F & LDK_BR_LMS, DP = F & LDK_BR_DP, DS = F & LDK_BR_DS;
    const uint8_t *prow = DP ? perm + rj * BP_T * 256 : nullptr;
    const uint32_t b = a.base[pi], inv = a.inv[pi];
    const int T = a.T[pi];
    const double bd = (double)b, b2 = bd * bd, b4 = b2 * b2;
    uint32_t dlane = 0;
    if constexpr (DS) dlane = lane < T ? shift[rj * BP_T + lane] : 0u;
    double v[P] = {};
    if constexpr (LMS) {
        uint32_t srows[MJ];
        lane_row<MJ>(lmsw, a.lms_off + ((uint64_t)rj * BP_T + lane) * BP_T, lane, T, srows);
        int t0 = 0;
        for (; t0 + 4 <= T; t0 += 4)
            digits_lms<4, MJ, F, P>(srows, dlane, prow, z, t0, b, inv, b4, v);
        if (t0 + 2 <= T) {
            digits_lms<2, MJ, F, P>(srows, dlane, prow, z, t0, b, inv, b2, v);
            t0 += 2;
        }
        if (t0 < T) digits_lms<1, MJ, F, P>(srows, dlane, prow, z, t0, b, inv, bd, v);
    } else {
        // with a map every digit takes part; those past M start from zero
        const int rows = DP || DS ? T : min(T, (int)a.M[pi]);
#pragma unroll
        for (int q = 0; q < MJ; ++q) {
            if (4 * q + 4 <= rows) {
                uint32_t g[P][4];
#pragma unroll
                for (int p = 0; p < P; ++p)
#pragma unroll
                    for (int k = 0; k < 4; ++k) g[p][k] = (z[p][q] >> (8 * k)) & 255u;
                digits_join<4, F, P>(g, dlane, prow, 4 * q, b, b4, v);
            } else {
#pragma unroll
                for (int k = 0; k < 3; ++k)
                    if (4 * q + k < rows) {
                        uint32_t one[P][1];
#pragma unroll
                        for (int p = 0; p < P; ++p) one[p][0] = (z[p][q] >> (8 * k)) & 255u;
                        digits_join<1, F, P>(one, dlane, prow, 4 * q + k, b, bd, v);
                    }
            }
        }
        if constexpr (DP || DS) {
            int t0 = 4 * MJ;
            for (; t0 + 4 <= T; t0 += 4) {
                uint32_t g[P][4] = {};
                digits_join<4, F, P>(g, dlane, prow, t0, b, b4, v);
            }
            for (; t0 < T; ++t0) {
                uint32_t g[P][1] = {};
                digits_join<1, F, P>(g, dlane, prow, t0, b, bd, v);
            }
        } else {
#pragma unroll
            for (int p = 0; p < P; ++p) v[p] *= a.bTM[pi];  // exact: below b^T
        }
    }
    const double bT = a.bT[pi], ib = a.ibT[pi];
#pragma unroll
    for (int p = 0; p < P; ++p) {
        double q = v[p] * ib;
        q = fma(fma(-bT, q, v[p]), ib, q);
        x[p] = fma(fma(-bT, q, v[p]), ib, q);
    }
}

// Write a finished tile: rows p < valid of dimensions j0 .. j0+dch-1 of the
// [R][cnt][d] output.  With every dimension in the tile the rows are one
// contiguous run.
template <int PTS>
__device__ __forceinline__ void flush_tile(double *__restrict__ out, const double *tile, int64_t cnt, int d,
                                           int r, int64_t i0, int j0, int dch, int tid)
{
    const int64_t rest = cnt - i0;
    const int valid = rest < PTS ? (int)rest : PTS;
    double *dst = out + ((size_t)r * cnt + i0) * d + j0;
    if (dch == d) {
        for (int e = tid; e < valid * dch; e += BP_TT) dst[e] = tile[e];
    } else {
        for (int e = tid; e < valid * dch; e += BP_TT) {
            const int p = e / dch;
            dst[(size_t)p * d + (e - p * dch)] = tile[e];
        }
    }
}

template <int MJ, int F, int P>
__device__ __forceinline__ void halton_coordinate(const BpArgs &a, const uint32_t *__restrict__ lmsw,
                                                  const uint8_t *__restrict__ shift,
                                                  const uint8_t *__restrict__ perm, const uint32_t (&i)[P],
                                                  int r, int j, int lane, double (&x)[P])
{
    uint32_t z[P][MJ];
#pragma unroll
    for (int p = 0; p < P; ++p) index_digits_packed<MJ>(a, j, i[p], z[p]);
    coordinate<MJ, F, P>(a, j, lmsw, shift, perm, z, (size_t)r * a.d + j, lane, x);
}

// Halton: a block takes 64 P consecutive indices of one replication, P per
// lane (the rows of S and the permutations are fetched once for them); its
// eight waves split the dimensions (a balanced order from the host) and write
// into an LDS tile of whole rows, which the block then stores as one
// contiguous run (d <= 54 fits one tile).  Bound by VALU issue and, with
// permutations, by the gathers of their bytes.  R = 16, n = 2^15, d = 52 (us):
// no scrambles 106 -> 56, LMS + DP 196 -> 138, LMS + DS 175 -> 125.  Three
// points a lane: 148 (two blocks a CU).  Staging S and the permutations in LDS
// for longer spans of points measured no better than one point a lane (175 to
// 185) and loses on small sets.
template <int F, int P>
__global__ __launch_bounds__(BP_TT) void k_gen_halton(BpArgs a, const uint32_t *__restrict__ lmsw,
                                                      const uint8_t *__restrict__ shift,
                                                      const uint8_t *__restrict__ perm,
                                                      double *__restrict__ out)
{
    double *tile = reinterpret_cast<double *>(g_bp_lds);  // [64 P][d]
    const int tid = threadIdx.x, lane = tid & 63, r = blockIdx.y;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int64_t i0 = (int64_t)blockIdx.x * (BP_P * P);
    uint32_t i[P];
#pragma unroll
    for (int p = 0; p < P; ++p) {
        const int64_t ii = i0 + 64 * p + lane;
        i[p] = (uint32_t)(a.n_min + (ii < a.cnt ? ii : 0));
    }
    for (int q = a.wbeg[wave]; q < (int)a.wbeg[wave + 1]; ++q) {
        const int j = a.ord[q];
        const int mq = (a.M[j] + 3) >> 2;
        double x[P];
        switch (mq) {
        case 1: halton_coordinate<1, F, P>(a, lmsw, shift, perm, i, r, j, lane, x); break;
        case 2: halton_coordinate<2, F, P>(a, lmsw, shift, perm, i, r, j, lane, x); break;
        case 3: halton_coordinate<3, F, P>(a, lmsw, shift, perm, i, r, j, lane, x); break;
        case 4: halton_coordinate<4, F, P>(a, lmsw, shift, perm, i, r, j, lane, x); break;
        case 5: halton_coordinate<5, F, P>(a, lmsw, shift, perm, i, r, j, lane, x); break;
        case 6: halton_coordinate<6, F, P>(a, lmsw, shift, perm, i, r, j, lane, x); break;
        case 7: halton_coordinate<7, F, P>(a, lmsw, shift, perm, i, r, j, lane, x); break;
        default: halton_coordinate<8, F, P>(a, lmsw, shift, perm, i, r, j, lane, x); break;
        }
#pragma unroll
        for (int p = 0; p < P; ++p) tile[(64 * p + lane) * a.d + j] = x[p];
    }
    __syncthreads();
    flush_tile<BP_P * P>(out, tile, a.cnt, a.d, r, i0, 0, a.d, tid);
}

// Faure: one base for every dimension, so a lane forms its index digits (MJ
// words) once; dimension j takes z = C_j a mod b from its packed matrix
// rows.  Tiles of up to 64 dimensions (d may reach 251).
template <int MJ, int F, int P>
__global__ __launch_bounds__(BP_TT) void k_gen_faure(BpArgs a, const uint32_t *__restrict__ lmsw,
                                                     const uint8_t *__restrict__ shift,
                                                     const uint8_t *__restrict__ perm,
                                                          const uint32_t *__restrict__ cmat,
                                                          double *__restrict__ out)
{
    double *tile = reinterpret_cast<double *>(g_bp_lds);  // [64 P][min(d, 64)]
    const int tid = threadIdx.x, lane = tid & 63, r = blockIdx.y;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int64_t i0 = (int64_t)blockIdx.x * (BP_P * P);
    const uint32_t b = a.base[0], inv = a.inv[0];
    uint32_t ad[P][MJ];
#pragma unroll
    for (int p = 0; p < P; ++p) {
        const int64_t ii = i0 + 64 * p + lane;
        index_digits_packed<MJ>(a, 0, (uint32_t)(a.n_min + (ii < a.cnt ? ii : 0)), ad[p]);
    }
    for (int j0 = 0; j0 < a.d; j0 += BP_DCH) {
        const int dch = a.d - j0 < BP_DCH ? a.d - j0 : BP_DCH;
        for (int jj = wave; jj < dch; jj += BP_WAVES) {
            const int j = j0 + jj;
            // z_t = sum_{k >= t} C[t][k] a_k mod b (zero for t >= M: a_k = 0 there)
            const uint32_t *cj = cmat + (size_t)j * (4 * MJ * MJ);
            uint32_t z[P][MJ] = {};
#pragma unroll
            for (int t = 0; t < 4 * MJ; ++t) {
#pragma unroll
                for (int p = 0; p < P; ++p) {
                    uint32_t s = 0;
#pragma unroll
                    for (int q = 0; q < MJ; ++q) s = __builtin_amdgcn_udot4(cj[t * MJ + q], ad[p][q], s, false);
                    z[p][t >> 2] |= mod_b(s, b, inv) << (8 * (t & 3));
                }
            }
            double x[P];
            coordinate<MJ, F, P>(a, 0, lmsw, shift, perm, z, (size_t)r * a.d + j, lane, x);
#pragma unroll
            for (int p = 0; p < P; ++p) tile[(64 * p + lane) * dch + jj] = x[p];
        }
        __syncthreads();
        flush_tile<BP_P * P>(out, tile, a.cnt, a.d, r, i0, j0, dch, tid);
        __syncthreads();  // the tile is free for the next dimensions
    }
}

__device__ __forceinline__ uint64_t mix64(uint64_t z)
{
    z = (z ^ (z >> 30)) * 0xbf58476d1ce4e5b9ull;
    z = (z ^ (z >> 27)) * 0x94d049bb133111ebull;
    return z ^ (z >> 31);
}

// The word whose top bit says whether digit t of a point is flipped: the high
// half of mix64(key XOR seed) (its last step leaves the top bit alone).  With
// key = 2^(t-1) + (z >> (65 - t)), z the unscrambled word, the first step
// w ^ (w >> 30) is linear and commutes with the shift, so zz = z ^ (z >> 30)
// is formed once per point and c = seed ^ (seed >> 30) once per dimension:
// 13 to 15 instructions a digit (23 with the key put together each time).
__device__ __forceinline__ uint64_t mix_first(uint64_t v) { return v ^ (v >> 30); }
__device__ __forceinline__ uint32_t nus_flip_word(uint64_t zz, uint64_t c, int t)
{
    uint64_t w = (t > 1 ? zz >> (65 - t) : 0) ^ (c ^ mix_first(1ull << (t - 1)));
    w *= 0xbf58476d1ce4e5b9ull;
    w = (w ^ (w >> 27)) * 0x94d049bb133111ebull;
    return (uint32_t)(w >> 32);
}
// f with the top bit of w shifted in.
__device__ __forceinline__ uint32_t shift_in(uint32_t f, uint32_t w) { return __builtin_amdgcn_alignbit(f, w, 31); }

// NUS.  Bound by the 64 mixing functions a coordinate (VALU): the first
// NUS_B digits have at most 2^NUS_B prefixes, so a block forms their flips
// once per dimension, as a table over the top NUS_B digits, and a point mixes
// the remaining 64 - NUS_B.  Block: up to NUS_D dimensions (a wave each; the
// dimensions go to the blocks as evenly as they can), one replication, `span`
// consecutive indices (a multiple of 64), 64 at a time, one per lane; the word
// of an index is a lane word (its low 6 bits) XOR a wave-uniform one.  The
// tile's coordinates go out in runs of up to 8 NUS_D bytes per point (less than
// a tenth of the store bandwidth is in use).  Measured: R = 16, n = 2^16, d = 52
// 2.00 -> 1.13 ms; d = 1 90 -> 36 us (always four waves a block: 114), d = 5
// 206 -> 169 (199).
constexpr int NUS_B = 12;  // table digits: 8 KiB per dimension, 2^12 mixing functions per block
constexpr int NUS_D = 4;
constexpr int NUS_T = 64 * NUS_D;
// Orders a wave's own LDS accesses (they complete in order in the hardware).
__device__ __forceinline__ void wave_lds_fence() { __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront"); }
__global__ __launch_bounds__(NUS_T) void k_gen_nus(int d, int m, int B, int span, int64_t n_min, int64_t cnt,
                                                   const uint64_t *__restrict__ gen,
                                                   const uint64_t *__restrict__ seed,
                                                   double *__restrict__ out)
{
    uint16_t *const table = reinterpret_cast<uint16_t *>(g_bp_lds);  // [NUS_D][top B digits] -> their flips
    __shared__ double tile[64][NUS_D + 1];
    const int tid = threadIdx.x, lane = tid & 63, r = blockIdx.y;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    // blocks of the same points are neighbours: their runs share cache lines
    const int groups = (d + NUS_D - 1) / NUS_D;
    const int gj = (int)(blockIdx.x % groups);
    const int j0 = gj * d / groups, dims = (gj + 1) * d / groups - j0;  // as even as they go
    const int W = blockDim.x >> 6;       // waves: the most dimensions of a group
    const bool live = wave < dims;       // the last wave of a smaller group only stores
    const int j = j0 + (live ? wave : 0);
    const uint64_t s = seed[(size_t)r * d + j];
    const uint64_t *__restrict__ col = gen + (size_t)j * m;
    uint16_t *const tab = table + (wave << B);
    const uint64_t cs = mix_first(s);
    // flips of the top b digits from those of the top b - 1: entry q becomes
    // 2 q and 2 q + 1.  The wave goes from the last entries down, so that an
    // entry is read before it is overwritten: a step reads entries q0 .. q0 +
    // 63 and then writes 2 q0 .. 2 q0 + 127.
    if (lane == 0) tab[0] = 0;
    for (int b = 1; b <= B && live; ++b) {
        const int half = 1 << (b - 1);
        for (int q0 = (half - 1) & ~63; q0 >= 0; q0 -= 64) {
            const int q = q0 + lane;
            wave_lds_fence();
            const uint32_t up = q < half ? tab[q] : 0;
            wave_lds_fence();
            if (q < half) {
                const uint64_t zq = b > 1 ? (uint64_t)q << (65 - b) : 0;
                const uint16_t v = (uint16_t)shift_in(up, nus_flip_word(mix_first(zq), cs, b));
                tab[2 * q] = v;
                tab[2 * q + 1] = v;
            }
        }
    }
    wave_lds_fence();
    // word of the low 6 index bits, and of the tile's
    const int64_t first = n_min + (int64_t)(blockIdx.x / groups) * span;
    const int64_t lo = first & ~(int64_t)63;  // tiles at multiples of 64
    uint64_t zl = 0, zu = 0;
    for (int k = 0; k < 6 && k < m; ++k)
        if ((lane >> k) & 1) zl ^= col[k];
    for (int k = 6; k < m; ++k) zu ^= col[k] & -(uint64_t)((lo >> k) & 1);
    const int64_t end = first + span < n_min + cnt ? first + span : n_min + cnt;
    for (int64_t i0 = lo; i0 < end; i0 += 64) {
        uint64_t z = zl ^ zu;
        if (live) {
            const uint64_t zz = mix_first(z);
            // c's XORs with the 52 constants stay in the loop, on the scalar unit
            // (hoisted, they spill the scalar registers)
            uint64_t c = cs;
            asm volatile("" : "+s"(c));
            uint32_t fh = B ? tab[z >> (64 - B)] : 0, fl = 0;
            for (int t = B + 1; t <= NUS_B; ++t) fh = shift_in(fh, nus_flip_word(zz, c, t));
#pragma unroll
            for (int t = NUS_B + 1; t <= 32; ++t) fh = shift_in(fh, nus_flip_word(zz, c, t));
#pragma unroll
            for (int t = 33; t <= 64; ++t) fl = shift_in(fl, nus_flip_word(zz, c, t));
            z ^= ((uint64_t)fh << 32) | fl;
        }
        __syncthreads();  // the previous tile is out
        if (live) tile[lane][wave] = unit_f64(z);
        __syncthreads();
        const int p = tid / W, q = tid % W;
        const int64_t i = i0 + p;
        if (q < dims && i >= first && i < end)
            out[((size_t)r * cnt + (i - n_min)) * d + j0 + q] = tile[p][q];
        // the next tile flips the index bits from 6 up to its lowest zero one
        for (int k = 6; k < m; ++k) {
            zu ^= col[k];
            if (!((i0 >> k) & 1)) break;
        }
    }
}

// Indices per NUS block and table digits: the longest span that leaves about
// ten blocks per compute unit (the tail of the last round of blocks is a
// tenth of the launch), 64 at least, and a table of at most half the span's
// points, so that forming it (2^B - 1 mixing functions) costs 4 % (a span of
// 8192) to 10 % (64) of the B span that it saves.
struct NusSplit {
    int span, B;
};
NusSplit nus_split(int64_t cnt, int64_t columns)
{
    int span = 64;
    while (span < 8192 && (cnt + 2 * span - 1) / (2 * span) * columns >= 2560) span *= 2;
    NusSplit s{span, 0};
    while (s.B < NUS_B && (2 << s.B) <= span / 2) ++s.B;
    return s;
}

bool is_prime(int v)
{
    if (v < 2) return false;
    for (int q = 2; q * q <= v; ++q)
        if (v % q == 0) return false;
    return true;
}

int digits_kept(int b)
{
    int T = 0;
    uint64_t p = 1;
    while (p <= ((uint64_t)1 << 53) / (uint64_t)b) {
        p *= (uint64_t)b;
        ++T;
    }
    return T;
}

// Digits needed for the indices below n_max (at least 1).
int index_digits(int b, int64_t n_max)
{
    int M = 1;
    uint64_t p = (uint64_t)b;
    while (p < (uint64_t)n_max) {
        p *= (uint64_t)b;
        ++M;
    }
    return M;
}

int validate_bpointset(const ldk_bpointset *ps, int64_t n_min, int64_t n_max)
{
    if (!ps) return LDK_EINVAL;
    if (ps->R < 1 || ps->R > 65535 || ps->d < 1 || n_min < 0 || n_max < n_min) return LDK_EINVAL;
    if (n_max > ((int64_t)1 << 32)) return LDK_ENOTSUP;
    switch (ps->kind) {
    case LDK_HALTON:
        if (ps->d > BP_MAX_D) return LDK_EINVAL;
        break;
    case LDK_FAURE:
        if (!is_prime(ps->base) || ps->base < ps->d || ps->base > 251) return LDK_EINVAL;
        break;
    case LDK_DNET_NUS:
        if (ps->m < 0 || ps->m > 32 || n_max > ((int64_t)1 << ps->m)) return LDK_EINVAL;
        if (!ps->gen || !ps->seed) return LDK_EINVAL;
        return LDK_OK;
    default:
        return LDK_EINVAL;
    }
    if (ps->flags & ~(LDK_BR_LMS | LDK_BR_DP | LDK_BR_DS)) return LDK_EINVAL;
    if (((ps->flags & LDK_BR_LMS) && !ps->lms) || ((ps->flags & LDK_BR_DP) && !ps->perm) ||
        ((ps->flags & LDK_BR_DS) && !ps->shift))
        return LDK_EINVAL;
    return LDK_OK;
}

}  // namespace

}  // namespace ldk

using namespace ldk;

extern "C" size_t ldk_bpoints_workspace_bytes(const ldk_bpointset *ps)
{
    if (!ps || ps->kind != LDK_FAURE || ps->d < 1) return 0;
    return (size_t)ps->d * BP_KMAX * BP_QW * sizeof(uint32_t);
}

extern "C" int ldk_gen_bpoints(const ldk_bpointset *ps, int64_t n_min, int64_t n_max, double *out,
                               void *ws, ldk_stream stream)
{
    int st = validate_bpointset(ps, n_min, n_max);
    if (st) return st;
    const int64_t cnt = n_max - n_min;
    if (cnt == 0) return LDK_OK;
    if (!out) return LDK_EINVAL;
    if (ps->kind == LDK_FAURE && !ws) return LDK_EINVAL;
    st = ensure_init();
    if (st) return st;
    hipStream_t s = as_stream(stream);
    if (ps->kind == LDK_DNET_NUS) {
        const int64_t groups = (ps->d + NUS_D - 1) / NUS_D;
        const unsigned waves = (unsigned)((ps->d + groups - 1) / groups);
        const NusSplit sp = nus_split(cnt, groups * ps->R);
        const int64_t blocks = (cnt + sp.span - 1) / sp.span * groups;
        if ((uint64_t)blocks * waves * 64 > 0xffffffffull) return LDK_ENOTSUP;
        // (the table's size in LDS by its digits: short spans keep eight blocks a CU)
        const size_t lds = (size_t)waves * sizeof(uint16_t) << sp.B;
        hipLaunchKernelGGL(k_gen_nus, dim3((unsigned)blocks, (unsigned)ps->R), dim3(64 * waves),
                           lds, s, ps->d, ps->m, sp.B, sp.span, n_min, cnt, ps->gen, ps->seed, out);
        LDK_LAUNCH_CHECK();
        return LDK_OK;
    }
    const int64_t blocks = (cnt + BP_P - 1) / BP_P;
    if (blocks > 0x7fffffff) return LDK_ENOTSUP;
    const dim3 grid((unsigned)blocks, (unsigned)ps->R);
    BpArgs a{};
    a.d = ps->d;
    a.flags = ps->flags;
    a.n_min = n_min;
    a.cnt = cnt;
    a.small = n_max <= (1 << 24);
    // lms is read as 32-bit words from the word boundary at or below its
    // first byte (the same word, so within the allocation's page)
    const uintptr_t lp = reinterpret_cast<uintptr_t>(ps->lms);
    a.lms_off = (uint32_t)(lp & 3);
    const uint32_t *lmsw = reinterpret_cast<const uint32_t *>(lp & ~(uintptr_t)3);
    int prime = 1, m_max = 1;
    const int dims = ps->kind == LDK_FAURE ? 1 : ps->d;  // Faure: one base for all dimensions
    double cost[BP_MAX_D];
    for (int j = 0; j < dims; ++j) {
        int b = ps->base;
        if (ps->kind == LDK_HALTON) {
            do ++prime;
            while (!is_prime(prime));
            b = prime;
        }
        const int T = digits_kept(b), M = index_digits(b, n_max);
        if (M > BP_KMAX) return LDK_EINVAL;  // not reached for i < 2^32
        a.base[j] = (uint32_t)b;
        a.T[j] = (uint32_t)T;
        a.M[j] = (uint32_t)M;
        a.inv[j] = (uint32_t)((((uint64_t)1 << 32) + (uint64_t)b - 1) / (uint64_t)b);
        a.rb[j] = 1.0 / (double)b;
        double p = 1.0;
        for (int t = 0; t < T; ++t) p *= (double)b;
        a.bT[j] = p;
        a.ibT[j] = 1.0 / p;
        a.bTM[j] = 1.0;
        for (int t = M; t < T; ++t) a.bTM[j] *= (double)b;
        m_max = M > m_max ? M : m_max;
        cost[j] = (double)T * (((M + 3) / 4) + 12) + 10.0 * M;  // VALU work per coordinate, roughly
    }
    if (ps->kind == LDK_HALTON) {
        // longest processing time first: dimensions by decreasing cost, each
        // to the wave with the least work so far; then each wave's list in turn
        int idx[BP_MAX_D], owner[BP_MAX_D];
        for (int j = 0; j < ps->d; ++j) idx[j] = j;
        for (int x = 1; x < ps->d; ++x)
            for (int y = x; y > 0 && cost[idx[y]] > cost[idx[y - 1]]; --y) {
                const int tmp = idx[y];
                idx[y] = idx[y - 1];
                idx[y - 1] = tmp;
            }
        double load[BP_WAVES] = {};
        for (int k = 0; k < ps->d; ++k) {
            int w = 0;
            for (int x = 1; x < BP_WAVES; ++x)
                if (load[x] < load[w]) w = x;
            owner[k] = w;
            load[w] += cost[idx[k]];
        }
        int q = 0;
        for (int w = 0; w < BP_WAVES; ++w) {
            a.wbeg[w] = (uint32_t)q;
            for (int k = 0; k < ps->d; ++k)
                if (owner[k] == w) a.ord[q++] = (uint32_t)idx[k];
        }
        a.wbeg[BP_WAVES] = (uint32_t)q;
    }
    const int mq = (m_max + 3) / 4;
    const int F = ps->flags & (LDK_BR_LMS | LDK_BR_DP | LDK_BR_DS);
    const int dmax = ps->kind == LDK_FAURE && ps->d > BP_DCH ? BP_DCH : ps->d;
    const size_t lds = (size_t)BP_P * dmax * sizeof(double);
    // Two points a lane where that leaves two blocks a CU (four for Faure) and
    // the tile lets three share one.  R = 16, n = 2^15, LMS + DP (us): Halton d =
    // 52 175 -> 138, Faure b = 53, d = 52 135 -> 129; below the line, R = 2, n =
    // 2^14: 17.7 -> 19.4 and 18.1 -> 18.9; Faure b = 127, d = 100 (64 KiB): 353 -> 361.
    const bool two = blocks * ps->R >= (ps->kind == LDK_HALTON ? 1024 : 2048) && 3 * 2 * lds <= LDS_PER_CU;
    const dim3 grid2((unsigned)((blocks + 1) / 2), (unsigned)ps->R);
    if (ps->kind == LDK_FAURE) {
        hipLaunchKernelGGL(k_faure_cmat, dim3((unsigned)ps->d), dim3(64), 0, s, ps->base,
                           digits_kept(ps->base), mq, static_cast<uint32_t *>(ws));
        LDK_LAUNCH_CHECK();
        const uint32_t *cm = static_cast<const uint32_t *>(ws);
#define BP_FAURE_F(MJ, FL)                                                                              \
    case FL:                                                                                            \
        if (two)                                                                                        \
            hipLaunchKernelGGL((k_gen_faure<MJ, FL, 2>), grid2, dim3(BP_TT), 2 * lds, s, a, lmsw, ps->shift, \
                               ps->perm, cm, out);                                                      \
        else                                                                                            \
            hipLaunchKernelGGL((k_gen_faure<MJ, FL, 1>), grid, dim3(BP_TT), lds, s, a, lmsw, ps->shift, \
                               ps->perm, cm, out);                                                      \
        break;
#define BP_FAURE(MJ)                                                                                    \
    case MJ:                                                                                            \
        switch (F) {                                                                                    \
            BP_FAURE_F(MJ, 0) BP_FAURE_F(MJ, 1) BP_FAURE_F(MJ, 2) BP_FAURE_F(MJ, 3)                     \
            BP_FAURE_F(MJ, 4) BP_FAURE_F(MJ, 5) BP_FAURE_F(MJ, 6) BP_FAURE_F(MJ, 7)                     \
        }                                                                                               \
        break;
        switch (mq) {
            BP_FAURE(1) BP_FAURE(2) BP_FAURE(3) BP_FAURE(4) BP_FAURE(5) BP_FAURE(6) BP_FAURE(7) BP_FAURE(8)
        default: return LDK_EINVAL;
        }
#undef BP_FAURE
#undef BP_FAURE_F
    } else {
#define BP_HALTON(FL)                                                                                   \
    case FL:                                                                                            \
        if (two)                                                                                        \
            hipLaunchKernelGGL((k_gen_halton<FL, 2>), grid2, dim3(BP_TT), 2 * lds, s, a, lmsw, ps->shift, \
                               ps->perm, out);                                                          \
        else                                                                                            \
            hipLaunchKernelGGL((k_gen_halton<FL, 1>), grid, dim3(BP_TT), lds, s, a, lmsw, ps->shift,    \
                               ps->perm, out);                                                          \
        break;
        switch (F) {
            BP_HALTON(0) BP_HALTON(1) BP_HALTON(2) BP_HALTON(3) BP_HALTON(4) BP_HALTON(5) BP_HALTON(6)
            BP_HALTON(7)
        }
#undef BP_HALTON
    }
    LDK_LAUNCH_CHECK();
    return LDK_OK;
}
