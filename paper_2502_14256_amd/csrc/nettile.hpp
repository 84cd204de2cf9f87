// Net points of a tile of consecutive indices, regenerated in registers: the
// part shared by the kernel column, its parameter gradient and the RQMC sums.
//
// A block of KC_THREADS threads takes KC_THREADS IT indices from tile0 (a
// multiple of that); thread t has the points tile0 + t + KC_THREADS l, l < IT.
// The index bits of tile0, l and t are disjoint and the point is GF(2)-linear
// in the index (Gray order too: the Gray code is linear), so
//   z(tile0 + t + KC_THREADS l) = z(tile0) ^ z(KC_THREADS l) ^ z(t),
// i.e. one base word per tile, log2 IT step words and two 16-entry nibble
// tables of z over the low 8 index bits, per dimension.
#pragma once

#include <type_traits>

#include "kfactor.hpp"

namespace ldk {

namespace {

// The word a kernel needs of a point: FP32 factors see the top 32 digits only.
template <typename R>
struct net_word {
    using type = uint64_t;
    static __device__ __forceinline__ type cut(uint64_t z) { return z; }
};
template <>
struct net_word<float> {
    using type = uint32_t;
    static __device__ __forceinline__ type cut(uint64_t z) { return (uint32_t)(z >> 32); }
};
__device__ __forceinline__ uint32_t top_word(uint64_t z) { return (uint32_t)(z >> 32); }
__device__ __forceinline__ uint32_t top_word(uint32_t z) { return z; }

constexpr int log2_of(int v) { return v <= 1 ? 0 : 1 + log2_of(v / 2); }
constexpr uint32_t brev_const(uint32_t v, int bits)
{
    uint32_t r = 0;
    for (int b = 0; b < bits; ++b) r |= ((v >> b) & 1u) << (bits - 1 - b);
    return r;
}

// Tables of a chunk of dimensions.  w[jj][q]: z of index bit q for
// q < NW - 1, then z(tile0).
template <typename Z, int NW>
struct NetTables {
    Z w[NT_DIMS][NW];
    Z nib[NT_DIMS][2][16];  // z of (nibble h of the low index byte)
    // the columns and scrambles the words are formed from; rows padded:
    // lanes of a wave read rows of different dimensions
    uint64_t col[NT_DIMS][65];
    uint64_t srow[NT_DIMS][sizeof(Z) * 8 + 1];
};

// Effective column of index bit k: the change of the point when the bit
// flips (Gray order: the bit is in code bits k and k - 1).
__device__ __forceinline__ uint64_t index_column(const uint64_t *col, int m, bool gray, int k)
{
    if (k >= m) return 0;
    return col[k] ^ (gray && k > 0 ? col[k - 1] : 0);
}

// Forms the tables of dimensions jc .. jc + DB - 1 (DB <= NT_DIMS) of
// replication r for the tile at tile0 (a multiple of 2^(NW - 1)).
// Scrambling acts on words, not on generating columns: S (C_a ^ C_b) =
// S C_a ^ S C_b, so the base word is scrambled once, whatever its number of
// set index bits.  A scrambled word is split over several threads (16 digits
// each): 64 parities one after the other in one thread per word left half
// the block idle and set the latency of small problems (a 16-dimension
// chunk: about 10 us before, 2 us now).  Every thread of the block calls it.
// `stage` runs in each thread between the build's first two barriers (for
// per-chunk words of the caller's own).
template <typename Z, int NW, typename Stage>
__device__ __forceinline__ void build_net_tables(const PointsetArgs &ps, NetTables<Z, NW> &L, int r,
                                                 int jc, int DB, uint64_t tile0, Stage &&stage)
{
    constexpr int DIGITS = sizeof(Z) * 8, PARTS = DIGITS / 16;
    const int d = ps.d, m = ps.m_max, t = threadIdx.x;
    const bool gray = ps.order == LDK_GRAY, lms = ps.lms != nullptr;
    __syncthreads();  // tables of the previous chunk are no longer read
    stage();
    for (int w = t; w < DB * m; w += KC_THREADS) {
        const int jj = w / m, k = w - jj * m;
        L.col[jj][k] = net_gen_column(ps, r, jc + jj, k);
    }
    if (lms)
        for (int w = t; w < DB * DIGITS; w += KC_THREADS)
            L.srow[w / DIGITS][w % DIGITS] =
                ps.lms[((size_t)r * d + jc + w / DIGITS) * 64 + w % DIGITS];
    __syncthreads();
    const int items = DB * NW * (lms ? PARTS : 1);
    for (int it = t; it < items; it += KC_THREADS) {
        const int q = it % NW, rest = it / NW;
        const int part = lms ? rest % PARTS : 0, jj = lms ? rest / PARTS : rest;
        uint64_t c = 0;
        if (q == NW - 1) {
            for (int k = NW - 1; k < m; ++k)
                c ^= index_column(L.col[jj], m, gray, k) & -(uint64_t)((tile0 >> k) & 1);
        } else {
            c = index_column(L.col[jj], m, gray, q);
        }
        if (!lms) {
            L.w[jj][q] = sizeof(Z) == 8 ? (Z)c : (Z)(c >> 32);
            continue;
        }
        // digits 16 part + 15 down to 16 part: each parity enters at the top
        // of acc, so the last one (the most significant digit) ends on top
        const uint32_t clo = (uint32_t)c, chi = (uint32_t)(c >> 32);
        uint32_t acc = 0;
#pragma unroll
        for (int x = 15; x >= 0; --x) {
            const uint64_t row = L.srow[jj][16 * part + x];
            const uint32_t f = ((uint32_t)row & clo) ^ ((uint32_t)(row >> 32) & chi);
            acc = __builtin_amdgcn_alignbit((uint32_t)__popc(f), acc, 1);
        }
        reinterpret_cast<uint16_t *>(&L.w[jj][q])[PARTS - 1 - part] = (uint16_t)(acc >> 16);
    }
    __syncthreads();
    for (int w = t; w < DB * 32; w += KC_THREADS) {
        const int jj = w >> 5, h = (w >> 4) & 1, v = w & 15;
        Z z = 0;
#pragma unroll
        for (int k = 0; k < 4; ++k) z ^= L.w[jj][4 * h + k] & -(Z)((v >> k) & 1);
        L.nib[jj][h][v] = z;
    }
    __syncthreads();
}

// The thread's points of dimension jj from its tables: base word zb, z(t),
// then the step words.
template <int IT, typename Z, int NW>
__device__ __forceinline__ void net_points(const NetTables<Z, NW> &L, int jj, Z zb, Z (&z)[IT])
{
    const int t = threadIdx.x;
    z[0] = zb ^ L.nib[jj][0][t & 15] ^ L.nib[jj][1][t >> 4];
#pragma unroll
    for (int h = 1; h < IT; h <<= 1) {
        const Z st = L.w[jj][KC_LOG_THREADS + log2_of(h)];
#pragma unroll
        for (int l = h; l < 2 * h; ++l) z[l] = z[l - h] ^ st;
    }
}

// ---- DSI factors of a point word through a table over the leading zeros ----
// beta (1 + leading zeros) and t1 = 2^-beta take at most 65 values, so what
// depends on them alone is read from LDS: one leading-zero count and one
// table read per factor instead of a count, a test for zero, two selections,
// a conversion and the exponent arithmetic (FP32 order 2: 18.6 -> 8
// instructions per factor, FP64: 29 -> 11).
//   order 2:  {1.5 - 2.5 t1, -beta 2^-32}: K = fma(-beta 2^-32, 2^32 x,
//             1.5 - 2.5 t1), the power of two kept in the entry;
//   order 1:  {1 - 3 t1, unused};
//   others:   {beta, t1}.
// Entry 0 is the point 0 (beta = t1 = 0), entry 1 + c has c leading zeros.
// FP32 sees the top 32 digits only; where they are all zero, x = 0 and
// t_nu <= 2^-33 is below half an ulp of every term it enters.
template <typename R>
struct alignas(2 * sizeof(R)) DsiEntry {
    R a, b;
};
template <typename R>
struct DsiLead {
    DsiEntry<R> e[8 * sizeof(R) + 1];  // 33 (FP32) or 65 (FP64)
};
template <typename R, int ALPHA>
__device__ __forceinline__ void fill_dsi_lead(DsiLead<R> &L, int t, int nthreads)
{
    constexpr int N = 8 * sizeof(R) + 1;
    for (int i = t; i < N; i += nthreads) {
        const R t1 = i ? pow2_neg_r<R>(i) : (R)0;
        if constexpr (ALPHA == 1)
            L.e[i] = {(R)1 - (R)3 * t1, (R)0};
        else if constexpr (ALPHA == 2)
            L.e[i] = {(R)1.5 - (R)2.5 * t1, -(R)i * (R)0x1p-32};
        else
            L.e[i] = {(R)i, t1};
    }
}

// Leading zeros of v as the hardware counts them (-1 for v = 0).
__device__ __forceinline__ int lead32(uint32_t v)
{
    int c;
    asm("v_ffbh_u32 %0, %1" : "=v"(c) : "v"(v));
    return c;
}

// Table index (leading zeros, -1 for the point 0) of each word.  FP64 counts
// the high half and corrects the words whose high half is zero (the point 0,
// otherwise one in 2^32) where a lane of the wave has one.
template <int IT>
__device__ __forceinline__ void lead_index(const uint32_t (&z)[IT], int (&c)[IT])
{
#pragma unroll
    for (int l = 0; l < IT; ++l) c[l] = lead32(z[l]);
}
template <int IT>
__device__ __forceinline__ void lead_index(const uint64_t (&z)[IT], int (&c)[IT])
{
    uint32_t least = 0xffffffffu;
#pragma unroll
    for (int l = 0; l < IT; ++l) {
        c[l] = lead32(top_word(z[l]));
        least = min(least, top_word(z[l]));
    }
    if (__builtin_amdgcn_ballot_w64(least == 0)) {
#pragma unroll
        for (int l = 0; l < IT; ++l)
            c[l] = top_word(z[l]) ? c[l] : z[l] ? clz64(z[l]) : -1;
    }
}

// 2^32 x of a point word, rounded once (unit<R> returns the same value scaled
// by the power of two).  FP64: hi + lo 2^-32, both terms exact.
__device__ __forceinline__ float word_scaled(uint32_t z) { return (float)opaque32(z); }
__device__ __forceinline__ double word_scaled(uint64_t z)
{
    return __builtin_fma((double)opaque32((uint32_t)z), scalar_const(0x1p-32),
                         (double)opaque32((uint32_t)(z >> 32)));
}

// LDS of a kernel that forms net factors of IT points per thread.
template <typename R, int IT>
struct NetLds {
    static constexpr int NW = KC_LOG_THREADS + log2_of(IT) + 1;
    NetTables<typename net_word<R>::type, NW> t;
    R gam[NT_DIMS];
    DsiLead<R> lead;
    DsiTables tab;  // order 4 and mixed orders
};
template <typename R, int ALPHA, int IT>
__device__ __forceinline__ void fill_net_lds(NetLds<R, IT> &L)
{
    if constexpr (ALPHA == 0 || ALPHA == 4) fill_dsi_tables(L.tab, threadIdx.x, KC_THREADS);
    fill_dsi_lead<R, ALPHA>(L.lead, threadIdx.x, KC_THREADS);
}
template <typename R, int IT>
__device__ __forceinline__ void build_net_lds(const KcolArgs &a, NetLds<R, IT> &L, int r, int jc, int DB,
                                              int64_t tile0)
{
    build_net_tables(a.ps, L.t, r, jc, DB, (uint64_t)tile0, [&] {
        if ((int)threadIdx.x < DB) L.gam[threadIdx.x] = (R)a.gamma[jc + threadIdx.x];
    });
}

// K of one point word; c = its table index (lead_index).
template <typename R, int ALPHA, typename Z>
__device__ __forceinline__ R dsi_word(Z z, int c, int alpha, const DsiLead<R> &lead, const DsiTables &tab)
{
    const DsiEntry<R> e = lead.e[c + 1];
    if constexpr (ALPHA == 1) {
        return e.a;
    } else if constexpr (ALPHA == 2) {
        return fma_r(e.b, word_scaled(z), e.a);
    } else {
        return dsi_from_lead<R, ALPHA>(top_word(z), word_scaled(z) * (R)0x1p-32, e.a, e.b, alpha,
                                       tab);
    }
}

}  // namespace

}  // namespace ldk
