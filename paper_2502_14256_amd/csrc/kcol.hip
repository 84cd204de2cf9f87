// First column of the product-weight Gram matrix,
//   k1_i = zeta prod_j (1 + gamma_j K_{alpha_j}(x_ij (-) x0_j)),
// with SI factors (Sec. 5.2, Bernoulli polynomials) for lattices and DSI
// factors (Sec. 5.3, Theorem 1) for base-2 digital nets.  This op is
// ALU-bound: the points are either read once or regenerated in registers.
#include <type_traits>

#include "nettile.hpp"

namespace ldk {

// ---------------------------------------------------------------------------
// Regenerating lattice variant.  Block: replication r = blockIdx.y; points
// i = tile0 + t + KC_THREADS l (l < IT), tile0 a multiple of KC_THREADS IT,
// so the bits of t, l and tile0 are disjoint and (LI = log2 IT)
//   natural: bitreverse(i) g = bitreverse(tile0 + t) g + bitreverse_LI(l) (g << (56 - LI)),
//   linear:  (i g) << (64-m) = ((tile0 + t) g) << (64-m) + l ((g << 8) << (64-m)).
// The anchor is point 0, so delta = z(i) - z(0) = z(i): the shift cancels.
// ---------------------------------------------------------------------------
template <typename R, int ALPHA, int ORDER, int IT>
__device__ __forceinline__ void lattice_tile(const KcolArgs &a, int64_t first, R (&prod)[IT])
{
    constexpr int LI = log2_of(IT);
    const int d = a.ps.d, m = a.ps.m_max;
    const uint64_t bfirst = ORDER == LDK_NATURAL ? brev64((uint64_t)first) : (uint64_t)first;
    for (int j = 0; j < d; ++j) {
        const uint64_t g = a.ps.gen[j];
        const int alpha = ALPHA ? ALPHA : alpha_of(a, j);
        const SiPoly cf = si_poly(alpha, a.gamma[j]);
        const R c0 = (R)cf.c0, c1 = (R)cf.c1, c2 = (R)cf.c2, c3 = (R)cf.c3;
        uint64_t base, G;
        if constexpr (ORDER == LDK_NATURAL) {
            base = bfirst * g;
            G = g << (56 - LI);
        } else {
            base = m == 0 ? 0 : ((bfirst * g) << (64 - m));
            G = m <= 8 ? 0 : ((g << 8) << (64 - m));
        }
        // natural order: G has no low-half bits, so the points of a thread
        // share the low half of delta and differ in the high half only
        const R lo_p = lo_part<R>((uint32_t)base);
#pragma unroll
        for (int l = 0; l < IT; ++l) {
            R x;
            if constexpr (ORDER == LDK_NATURAL)
                x = unit_hl<R>((uint32_t)(base >> 32) +
                                   brev_const((uint32_t)l, LI) * (uint32_t)(G >> 32),
                               lo_p);
            else
                x = unit<R>(base + (uint64_t)l * G);
            prod[l] *= si_weighted<R, ALPHA>(x, c0, c1, c2, c3);
        }
    }
}

// Column tile bx of replication r (KC_THREADS IT points from tile_base +
// bx KC_THREADS IT).  Points outside the window are formed and not stored.
template <typename R, int IT>
__device__ __forceinline__ void store_column(const KcolArgs &a, int64_t first, int r, const R (&prod)[IT],
                                             R *__restrict__ out)
{
    const int64_t cnt = a.n_max - a.n_min;
#pragma unroll
    for (int l = 0; l < IT; ++l) {
        const int64_t i = first + (int64_t)l * KC_THREADS;
        if (i >= a.n_min && i < a.n_max) out[(size_t)r * cnt + (i - a.n_min)] = prod[l];
    }
}
template <typename R, int ALPHA, int ORDER, int IT>
__device__ __forceinline__ void kcol_lattice_block(const KcolArgs &a, int64_t tile_base,
                                                   R *__restrict__ out, int64_t bx, int r)
{
    const int64_t first = tile_base + bx * (KC_THREADS * IT) + threadIdx.x;
    R prod[IT];
#pragma unroll
    for (int l = 0; l < IT; ++l) prod[l] = (R)a.zeta;
    lattice_tile<R, ALPHA, ORDER, IT>(a, first, prod);
    store_column<R, IT>(a, first, r, prod, out);
}

template <typename R, int ALPHA, int ORDER, int IT>
__global__ __launch_bounds__(KC_THREADS) void k_kcol_lattice(KcolArgs a, int64_t tile_base,
                                                            R *__restrict__ out)
{
    kcol_lattice_block<R, ALPHA, ORDER, IT>(a, tile_base, out, blockIdx.x, blockIdx.y);
}

// Point words and first column of a lattice in one launch.  The column
// regenerates the points in registers and never reads the words, so the
// two halves are independent: column tiles (VALU bound) and point-word
// tiles (store bound).  The column tiles are spread evenly over the block
// indices (one per ~8 point tiles at n = 2^20, d = 32), so every stretch of
// the launch mixes the two and the column's arithmetic runs beside the
// stores, instead of after 256 MiB of stores (two launches), before them
// (column blocks first: 52 us against 48 here), or not at all beside them
// (two streams: the point launch takes every slot).
static_assert(GEN_THREADS == KC_THREADS, "one block shape for both halves");
template <typename R, int ALPHA, int ORDER, int IT>
__global__ __launch_bounds__(KC_THREADS) void k_points_kcol_lattice(KcolArgs a, int64_t tile_base,
                                                                   int64_t kc_tiles,
                                                                   R *__restrict__ k1, GenGrid g,
                                                                   uint64_t *__restrict__ pts)
{
    const int64_t b = blockIdx.x;
    const int64_t kc_blocks = kc_tiles * a.ps.R;
    const int64_t total = kc_blocks + g.tiles * g.chunks * g.R;
    // column blocks spread evenly over the grid: block b is one iff the
    // count floor((b+1) kc / total) of column blocks up to b steps at b
    const int64_t before = b * kc_blocks / total, upto = (b + 1) * kc_blocks / total;
    if (upto != before) {
        kcol_lattice_block<R, ALPHA, ORDER, IT>(a, tile_base, k1, before % kc_tiles,
                                                (int)(before / kc_tiles));
        return;
    }
    const int64_t q = b - upto;
    gen_lattice_block<ORDER>(a.ps, a.n_min, a.n_max, g.P, g.pairs != 0, pts, q % g.tiles,
                             (int)((q / g.tiles) % g.chunks), (int)(q / (g.tiles * g.chunks)),
                             threadIdx.x);
}

// ---------------------------------------------------------------------------
// Regenerating net variant (see nettile.hpp): per chunk of dimensions the
// block forms the tables, then every thread its IT points per dimension.  The
// anchor is point 0 (z = 0), so delta = z(i).
// ---------------------------------------------------------------------------
template <typename R, int ALPHA, int IT>
__device__ __forceinline__ void kcol_net_block(const KcolArgs &a, NetLds<R, IT> &L, int64_t tile_base,
                                               R *__restrict__ out, int64_t bx, int r)
{
    using Z = typename net_word<R>::type;
    const int t = threadIdx.x, d = a.ps.d;
    const int64_t tile0 = tile_base + bx * (KC_THREADS * IT);
    fill_net_lds<R, ALPHA>(L);
    R prod[IT];
#pragma unroll
    for (int l = 0; l < IT; ++l) prod[l] = (R)a.zeta;
    for (int jc = 0; jc < d; jc += NT_DIMS) {
        const int DB = min(NT_DIMS, d - jc);
        build_net_lds(a, L, r, jc, DB, tile0);
        for (int jj = 0; jj < DB; ++jj) {
            const R gam = L.gam[jj];
            Z z[IT];
            int c[IT];
            net_points<IT>(L.t, jj, L.t.w[jj][L.NW - 1], z);
            lead_index(z, c);
            const int alpha = ALPHA ? ALPHA : alpha_of(a, jc + jj);
#pragma unroll
            for (int l = 0; l < IT; ++l)
                prod[l] *= dsi_weighted(gam, dsi_word<R, ALPHA>(z[l], c[l], alpha, L.lead, L.tab));
        }
    }
    store_column<R, IT>(a, tile0 + t, r, prod, out);
}

template <typename R, int ALPHA, int IT>
__global__ __launch_bounds__(KC_THREADS) void k_kcol_net(KcolArgs a, int64_t tile_base,
                                                        R *__restrict__ out)
{
    __shared__ NetLds<R, IT> L;
    kcol_net_block<R, ALPHA, IT>(a, L, tile_base, out, blockIdx.x, blockIdx.y);
}

// Point words and first column of a net in one launch: column blocks and
// point-word blocks interleaved as for lattices (the column regenerates the
// points and never reads the words), one LDS region shared by the two
// block kinds.
template <typename R, int ALPHA, int IT>
__global__ __launch_bounds__(KC_THREADS) void k_points_kcol_net(KcolArgs a, int64_t tile_base,
                                                               int64_t kc_tiles, R *__restrict__ k1,
                                                               GenGrid g, uint64_t *__restrict__ pts)
{
    __shared__ union {
        NetLds<R, IT> k;
        GenNetLds g;
    } L;
    const int64_t b = blockIdx.x;
    const int64_t kc_blocks = kc_tiles * a.ps.R;
    const int64_t total = kc_blocks + g.tiles * g.chunks * g.R;
    const int64_t before = b * kc_blocks / total, upto = (b + 1) * kc_blocks / total;
    if (upto != before) {
        kcol_net_block<R, ALPHA, IT>(a, L.k, tile_base, k1, before % kc_tiles, (int)(before / kc_tiles));
        return;
    }
    const int64_t q = b - upto;
    gen_net_block(a.ps, a.n_min, a.n_max, g.tile_base, g.P, g.logP, g.pairs, pts, q % g.tiles,
                  (int)((q / g.tiles) % g.chunks), (int)(q / (g.tiles * g.chunks)), threadIdx.x, L.g);
}

// ---------------------------------------------------------------------------
// Points given (any order; anchor rows x0).  Thread per point.
// ---------------------------------------------------------------------------
template <typename R, bool NET>
__global__ __launch_bounds__(KC_THREADS) void k_kcol_points(KcolArgs a, R *__restrict__ out)
{
    __shared__ DsiTables tab;
    if constexpr (NET) {
        fill_dsi_tables(tab, threadIdx.x, KC_THREADS);
        __syncthreads();
    }
    const int r = blockIdx.y;
    const int d = a.ps.d;
    const int64_t cnt = a.n_max - a.n_min;
    const int64_t i = a.n_min + (int64_t)blockIdx.x * KC_THREADS + threadIdx.x;
    if (i >= a.n_max) return;
    const uint64_t *row = a.pts + ((size_t)r * cnt + (i - a.n_min)) * d;
    R prod = (R)a.zeta;
    for (int j = 0; j < d; ++j) {
        const uint64_t u0 = a.x0 ? a.x0[(size_t)r * d + j] : a.pts[(size_t)r * cnt * d + j];
        const int alpha = alpha_of(a, j);
        if constexpr (NET) {
            prod *= dsi_weighted((R)a.gamma[j], dsi_factor_any<R>(alpha, row[j] ^ u0, tab));
        } else {
            const SiPoly cf = si_poly(alpha, a.gamma[j]);
            prod *= si_weighted<R, 0>(unit<R>(row[j] - u0), (R)cf.c0, (R)cf.c1, (R)cf.c2, (R)cf.c3);
        }
    }
    out[(size_t)r * cnt + (i - a.n_min)] = prod;
}

template <typename R, int ALPHA, int IT>
void launch_column(const KcolArgs &a, int64_t tile_base, int64_t tiles, hipStream_t s, void *k1)
{
    const dim3 grid((unsigned)tiles, (unsigned)a.ps.R), block(KC_THREADS);
    if (a.ps.kind == LDK_DNET_B2)
        hipLaunchKernelGGL((k_kcol_net<R, ALPHA, IT>), grid, block, 0, s, a, tile_base, (R *)k1);
    else if constexpr (ALPHA < 4) {
        if (a.ps.order == LDK_LINEAR)
            hipLaunchKernelGGL((k_kcol_lattice<R, ALPHA, LDK_LINEAR, IT>), grid, block, 0, s, a,
                               tile_base, (R *)k1);
        else
            hipLaunchKernelGGL((k_kcol_lattice<R, ALPHA, LDK_NATURAL, IT>), grid, block, 0, s, a,
                               tile_base, (R *)k1);
    }
}

template <typename R, int ALPHA, int IT>
void launch_points_column(const KcolArgs &a, int64_t tile_base, int64_t tiles, const GenGrid &g,
                          hipStream_t s, void *k1, uint64_t *pts)
{
    const dim3 grid((unsigned)(tiles * a.ps.R + g.tiles * g.chunks * g.R)), block(KC_THREADS);
    if (a.ps.kind == LDK_DNET_B2)
        hipLaunchKernelGGL((k_points_kcol_net<R, ALPHA, IT>), grid, block, 0, s, a, tile_base, tiles,
                           (R *)k1, g, pts);
    else if constexpr (ALPHA < 4) {
        if (a.ps.order == LDK_LINEAR)
            hipLaunchKernelGGL((k_points_kcol_lattice<R, ALPHA, LDK_LINEAR, IT>), grid, block, 0, s, a,
                               tile_base, tiles, (R *)k1, g, pts);
        else
            hipLaunchKernelGGL((k_points_kcol_lattice<R, ALPHA, LDK_NATURAL, IT>), grid, block, 0, s,
                               a, tile_base, tiles, (R *)k1, g, pts);
    }
}

// Calls f with the order as a compile-time constant: lattice orders 1..3 and
// net orders 1..4 get specialised kernels, mixed orders (0) read the
// per-dimension code.
template <typename F>
void with_alpha(int alpha, F &&f)
{
    switch (alpha) {
    case 1: f(std::integral_constant<int, 1>()); break;
    case 2: f(std::integral_constant<int, 2>()); break;
    case 3: f(std::integral_constant<int, 3>()); break;
    case 4: f(std::integral_constant<int, 4>()); break;
    default: f(std::integral_constant<int, 0>()); break;
    }
}
template <typename F>
void with_iters(int it, F &&f)
{
    switch (it) {
    case 1: f(std::integral_constant<int, 1>()); break;
    case 4: f(std::integral_constant<int, 4>()); break;
    case 8: f(std::integral_constant<int, 8>()); break;
    default: f(std::integral_constant<int, 16>()); break;
    }
}

}  // namespace ldk

using namespace ldk;

namespace ldk {

int prepare_kernel_args(const ldk_kernel *k, const ldk_pointset *ps, const uint64_t *pts,
                        const uint64_t *x0, int64_t n_min, int64_t n_max, int dtype, KcolArgs *out,
                        int *uniform_alpha)
{
    PointsetArgs p;
    int st = validate_pointset(ps, &p);
    if (st) return st;
    if (!k || k->kind != p.kind || k->d != p.d || !k->alpha || !k->gamma) return LDK_EINVAL;
    if (!(k->zeta > 0.0)) return LDK_EINVAL;
    if (dtype != LDK_F64 && dtype != LDK_F32) return LDK_EINVAL;
    if (n_min < 0 || n_max < n_min) return LDK_EINVAL;
    KcolArgs a{};
    a.ps = p;
    a.gamma = k->gamma;
    a.zeta = k->zeta;
    a.n_min = n_min;
    a.n_max = n_max;
    a.pts = pts;
    a.x0 = x0;
    // orders live on the host: validate, pack 2-bit codes, detect a uniform order
    const int amax = p.kind == LDK_LATTICE ? 3 : 4;
    int uniform = k->alpha[0];
    for (int j = 0; j < p.d; ++j) {
        const int al = k->alpha[j];
        if (al < 1 || al > amax) return LDK_EINVAL;
        if (al != uniform) uniform = 0;
        a.acode[j >> 5] |= (uint64_t)(al - 1) << (2 * (j & 31));
    }
    if (pts == nullptr) {
        const int64_t lim = (p.kind == LDK_LATTICE && p.order == LDK_NATURAL)
                                ? ((int64_t)1 << 62)
                                : ((int64_t)1 << p.m_max);
        if (n_max > lim) return LDK_EINVAL;
    } else if (x0 == nullptr && n_min != 0) {
        return LDK_EINVAL;  // the anchor must be given when row 0 is not point 0
    }
    *out = a;
    *uniform_alpha = uniform;
    return LDK_OK;
}

}  // namespace ldk

extern "C" int ldk_kernel_column(const ldk_kernel *k, const ldk_pointset *ps, const uint64_t *pts,
                                 const uint64_t *x0, int64_t n_min, int64_t n_max, int dtype,
                                 void *out, ldk_stream stream)
{
    KcolArgs a;
    int uniform = 0;
    const int st = prepare_kernel_args(k, ps, pts, x0, n_min, n_max, dtype, &a, &uniform);
    if (st) return st;
    const PointsetArgs &p = a.ps;
    if (n_max == n_min) return LDK_OK;  // empty window: out may be NULL
    if (!out) return LDK_EINVAL;
    hipStream_t s = as_stream(stream);
    if (pts != nullptr) {
        const int64_t blocks = (n_max - n_min + KC_THREADS - 1) / KC_THREADS;
        if (blocks > 0x7fffffff) return LDK_ENOTSUP;
        dim3 grid((unsigned)blocks, (unsigned)p.R);
        const bool net = p.kind == LDK_DNET_B2;
        if (dtype == LDK_F64) {
            if (net) hipLaunchKernelGGL((k_kcol_points<double, true>), grid, dim3(KC_THREADS), 0, s, a, (double *)out);
            else hipLaunchKernelGGL((k_kcol_points<double, false>), grid, dim3(KC_THREADS), 0, s, a, (double *)out);
        } else {
            if (net) hipLaunchKernelGGL((k_kcol_points<float, true>), grid, dim3(KC_THREADS), 0, s, a, (float *)out);
            else hipLaunchKernelGGL((k_kcol_points<float, false>), grid, dim3(KC_THREADS), 0, s, a, (float *)out);
        }
        LDK_LAUNCH_CHECK();
        return LDK_OK;
    }
    // tiles aligned to absolute multiples of their size
    const int it = column_iters(p.kind == LDK_LATTICE, p.R, n_min, n_max);
    const int64_t tile = (int64_t)KC_THREADS * it;
    const int64_t tile_base = (n_min / tile) * tile;
    const int64_t tiles = window_tiles(n_min, n_max, it);
    if (tiles > 0x7fffffff) return LDK_ENOTSUP;
    with_alpha(uniform, [&](auto al) {
        with_iters(it, [&](auto n) {
            if (dtype == LDK_F64) launch_column<double, al(), n()>(a, tile_base, tiles, s, out);
            else launch_column<float, al(), n()>(a, tile_base, tiles, s, out);
        });
    });
    LDK_LAUNCH_CHECK();
    return LDK_OK;
}

extern "C" int ldk_points_column(const ldk_kernel *k, const ldk_pointset *ps, int64_t n_min,
                                 int64_t n_max, uint64_t *pts, int dtype, void *k1,
                                 ldk_stream stream)
{
    KcolArgs a;
    int uniform = 0;
    int st = prepare_kernel_args(k, ps, nullptr, nullptr, n_min, n_max, dtype, &a, &uniform);
    if (st) return st;
    const PointsetArgs &p = a.ps;
    const int64_t lim = (p.kind == LDK_LATTICE && p.order == LDK_NATURAL) ? ((int64_t)1 << 62)
                                                                          : ((int64_t)1 << p.m_max);
    if (n_min < 0 || n_max < n_min || n_max > lim) return LDK_EINVAL;
    if (n_max == n_min) return LDK_OK;  // empty window: the outputs may be NULL
    if (!pts || !k1) return LDK_EINVAL;
    const int it = points_column_iters(p.kind == LDK_LATTICE, p.R, p.d, n_min, n_max);
    const int64_t tile = (int64_t)KC_THREADS * it;
    const int64_t tile_base = (n_min / tile) * tile;
    const int64_t kc_tiles = window_tiles(n_min, n_max, it);
    const GenGrid g = gen_grid(p, n_min, n_max, pts);
    const int64_t blocks = kc_tiles * p.R + g.tiles * g.chunks * g.R;
    if (blocks > 0x7fffffff) return LDK_ENOTSUP;
    hipStream_t s = as_stream(stream);
    with_alpha(uniform, [&](auto al) {
        with_iters(it, [&](auto n) {
            if (dtype == LDK_F64)
                launch_points_column<double, al(), n()>(a, tile_base, kc_tiles, g, s, k1, pts);
            else
                launch_points_column<float, al(), n()>(a, tile_base, kc_tiles, g, s, k1, pts);
        });
    });
    LDK_LAUNCH_CHECK();
    return LDK_OK;
}
