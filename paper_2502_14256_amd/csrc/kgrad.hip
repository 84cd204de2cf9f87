// Gradient of sum_i a_i k1_i in the kernel's parameters, the last step of the
// marginal-likelihood gradient (a = dL/dk1):
//   d k1_i / d log gamma_j = zeta t_ij prod_{l != j} f_il,   t = gamma K, f = 1 + t,
//   d k1_i / d log zeta    = k1_i = zeta prod_l f_il.
// ALU-bound like the kernel column.  Two sweeps over the dimensions in
// general: the first forms every point's product of nonzero factors P and
// counts its exact zeros; the second re-evaluates t_ij and takes the product
// of the other factors as P / f_ij (no zero), P (the one zero is f_ij) or 0.
// Given the forward column k1 (formed by the kernel column from bit-identical
// factors), the product of the other factors is k1_i / f_ij, so a dimension
// needs nothing of the others: the work is split over groups of dimensions as
// well as over the points.  The sums over points are FP64: per tile a thread
// adds its points' terms, KC_ITERS at a time, in the factor precision, the rest
// in FP64 in a fixed order.
#include <type_traits>

#include "nettile.hpp"

namespace ldk {

namespace {
constexpr int KG_WAVES = KC_THREADS / 64;

struct KgradArgs {
    KcolArgs k;
    const double *a;  // [R][cnt], dL/dk1
    const void *k1;   // [R][cnt] forward column (kernel-column dtype), or nullptr
    double *part;     // [R][parts][d + 1]
    int64_t tile_base;
    int64_t tiles;
    int dims_per_block;  // given the forward column
};

// One DPP lane move of a double (both halves), lanes the control leaves
// unwritten read 0.
template <int CTRL, int ROW_MASK = 0xf>
__device__ __forceinline__ double dpp_move(double v)
{
    const uint64_t u = (uint64_t)__double_as_longlong(v);
    const int lo = __builtin_amdgcn_update_dpp(0, (int)(uint32_t)u, CTRL, ROW_MASK, 0xf, false);
    const int hi = __builtin_amdgcn_update_dpp(0, (int)(uint32_t)(u >> 32), CTRL, ROW_MASK, 0xf,
                                               false);
    return __longlong_as_double((long long)(((uint64_t)(uint32_t)hi << 32) | (uint32_t)lo));
}

// Sum of v over the wavefront in a fixed order, returned in every lane.
// Lane moves go through DPP (no LDS round trips): swap neighbours, swap
// pairs, mirror within 8 and within 16 lanes (every lane of a row of 16 then
// holds the row's sum), then lane 15 of a row is added into the next row and
// lane 31 into the upper half; lane 63 ends with the total.
__device__ __forceinline__ double wave_sum(double v)
{
    v += dpp_move<0xb1>(v);        // quad_perm [1,0,3,2]
    v += dpp_move<0x4e>(v);        // quad_perm [2,3,0,1]
    v += dpp_move<0x141>(v);       // row_half_mirror
    v += dpp_move<0x140>(v);       // row_mirror
    v += dpp_move<0x142, 0xa>(v);  // row_bcast15 into rows 1 and 3
    v += dpp_move<0x143, 0xc>(v);  // row_bcast31 into rows 2 and 3
    const uint64_t u = (uint64_t)__double_as_longlong(v);
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)u, 63);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(u >> 32), 63);
    return __longlong_as_double((long long)(((uint64_t)hi << 32) | lo));
}

// Product of the other factors, P / f, f not 0 (the callers' case).  FP32
// multiplies by the hardware reciprocal (1 ulp; |f| is far above the range
// where it overflows).
__device__ __forceinline__ float quot(float p, float f) { return p * __builtin_amdgcn_rcpf(f); }
// FP64: the hardware's estimate of 1 / f (2^-24 relative), one Newton step
// (2^-48), and one correction of the quotient from its exact remainder, which
// leaves half an ulp and a term of 2^-96.  Where P is infinite or P / f
// overflows the correction is inf - inf: NaN, for which sum_terms below asks.
__device__ __forceinline__ double quot(double p, double f)
{
    double r = __builtin_amdgcn_rcp(f);
    r = fma_r(r, fma_r(-f, r, 1.0), r);
    const double q = p * r;
    return fma_r(fma_r(-f, q, p), r, q);
}
// Sum of a thread's KC_ITERS terms, term(l, divide), by quot; an FP64 sum that
// is NaN is formed again with the full division (one test per KC_ITERS
// quotients, and the branch is not taken for finite data).
template <typename R, typename Term>
__device__ __forceinline__ R sum_terms(Term &&term)
{
    R ps = (R)0;
#pragma unroll
    for (int l = 0; l < KC_ITERS; ++l) ps += term(l, [](R p, R f) { return quot(p, f); });
    if constexpr (std::is_same<R, double>::value) {
        if (__builtin_expect(ps != ps, 0)) {
            ps = 0.0;
#pragma unroll
            for (int l = 0; l < KC_ITERS; ++l) ps += term(l, [](double p, double f) { return p / f; });
        }
    }
    return ps;
}

// ---- dimension sweeps: call visit(j, l0, t[KC_ITERS], f[KC_ITERS]) for the
// dimensions ja .. jb - 1 in order and l0 = 0, KC_ITERS, .. below IT, t[l] =
// gamma_j K_j(delta) and f[l] = 1 + t[l] of point tile0 + threadIdx.x +
// KC_THREADS (l0 + l), f formed exactly as the kernel column forms it ----

// t and f of the KC_ITERS points l0 .. l0 + KC_ITERS - 1 of a thread (its
// points are first + KC_THREADS l, l < IT, first = tile0 + threadIdx.x with
// tile0 a multiple of KC_THREADS IT).
template <typename R, int ALPHA, int ORDER, int IT>
struct LatticeDim {
    R e0, c0, c1, c2, c3, lo_p;
    uint64_t base, G;
    __device__ __forceinline__ LatticeDim(const KcolArgs &a, uint64_t bfirst, int j)
    {
        const int m = a.ps.m_max;
        const uint64_t g = a.ps.gen[j];
        const int alpha = ALPHA ? ALPHA : alpha_of(a, j);
        const SiPoly cf = si_tpoly(alpha, a.gamma[j]);
        e0 = (R)cf.c0, c1 = (R)cf.c1, c2 = (R)cf.c2, c3 = (R)cf.c3;
        c0 = (R)si_poly(alpha, a.gamma[j]).c0;
        if constexpr (ORDER == LDK_NATURAL) {
            base = bfirst * g;
            G = g << (56 - log2_of(IT));
        } else {
            base = m == 0 ? 0 : ((bfirst * g) << (64 - m));
            G = m <= 8 ? 0 : ((g << 8) << (64 - m));
        }
        lo_p = lo_part<R>((uint32_t)base);  // shared low half (natural order)
    }
    __device__ __forceinline__ void factors(int l0, R (&t)[KC_ITERS], R (&f)[KC_ITERS]) const
    {
#pragma unroll
        for (int l = 0; l < KC_ITERS; ++l) {
            R x;
            if constexpr (ORDER == LDK_NATURAL)
                x = unit_hl<R>((uint32_t)(base >> 32) +
                                   brev_const((uint32_t)(l0 + l), log2_of(IT)) * (uint32_t)(G >> 32),
                               lo_p);
            else
                x = unit<R>(base + (uint64_t)(l0 + l) * G);
            t[l] = si_weighted<R, ALPHA>(x, e0, c1, c2, c3);
            f[l] = si_weighted<R, ALPHA>(x, c0, c1, c2, c3);
        }
    }
};

// The same for dimension jc + jj of net tables in LDS.
template <typename R, int ALPHA, int IT>
struct NetDim {
    using Z = typename net_word<R>::type;
    const NetLds<R, IT> &L;
    R gam;
    int alpha;
    Z z[IT];
    __device__ __forceinline__ NetDim(const KcolArgs &a, const NetLds<R, IT> &L_, int jc, int jj) : L(L_)
    {
        gam = L.gam[jj];
        alpha = ALPHA ? ALPHA : alpha_of(a, jc + jj);
        net_points<IT>(L.t, jj, L.t.w[jj][L.NW - 1], z);
    }
    __device__ __forceinline__ void factors(int l0, R (&t)[KC_ITERS], R (&f)[KC_ITERS]) const
    {
        Z zl[KC_ITERS];
        int c[KC_ITERS];
#pragma unroll
        for (int l = 0; l < KC_ITERS; ++l) zl[l] = z[l0 + l];
        lead_index(zl, c);
#pragma unroll
        for (int l = 0; l < KC_ITERS; ++l) {
            const R k = dsi_word<R, ALPHA>(zl[l], c[l], alpha, L.lead, L.tab);
            t[l] = gam * k;
            f[l] = dsi_weighted(gam, k);
        }
    }
};

// Points read from memory (any order; anchors x0 or row 0).
template <typename R, bool NET, typename Visit>
__device__ __forceinline__ void points_sweep(const KcolArgs &a, const DsiTables &tab, int r, int ja,
                                             int jb, int64_t first, Visit &&visit)
{
    const int d = a.ps.d;
    const int64_t cnt = a.n_max - a.n_min;
    for (int j = ja; j < jb; ++j) {
        const uint64_t u0 = a.x0 ? a.x0[(size_t)r * d + j] : a.pts[(size_t)r * cnt * d + j];
        const int alpha = alpha_of(a, j);
        const SiPoly cf = NET ? SiPoly{} : si_tpoly(alpha, a.gamma[j]);
        const R c0 = NET ? (R)1 : (R)si_poly(alpha, a.gamma[j]).c0;
        R t[KC_ITERS], f[KC_ITERS];
#pragma unroll
        for (int l = 0; l < KC_ITERS; ++l) {
            int64_t i = first + (int64_t)l * KC_THREADS;
            if (i >= a.n_max) i = a.n_max - 1;  // any valid row; masked out later
            const uint64_t u = a.pts[((size_t)r * cnt + (i - a.n_min)) * d + j];
            if constexpr (NET) {
                const R gam = (R)a.gamma[j];
                const R k = dsi_factor_any<R>(alpha, u ^ u0, tab);
                t[l] = gam * k;
                f[l] = dsi_weighted(gam, k);
            } else {
                const R x = unit<R>(u - u0);
                t[l] = si_weighted<R, 0>(x, (R)cf.c0, (R)cf.c1, (R)cf.c2, (R)cf.c3);
                f[l] = si_weighted<R, 0>(x, c0, (R)cf.c1, (R)cf.c2, (R)cf.c3);
            }
        }
        visit(j, 0, t, f);
    }
}

// Source selector: SRC 0 lattice natural, 1 lattice linear, 2 net, 3 points
// (lattice), 4 points (net).  Net tables are formed per chunk of NT_DIMS.
template <typename R, int ALPHA, int SRC, int IT, typename Visit>
__device__ __forceinline__ void sweep(const KcolArgs &a, NetLds<R, IT> &L, int r, int ja, int jb,
                                      int64_t tile0, Visit &&visit)
{
    const int64_t first = tile0 + threadIdx.x;
    if constexpr (SRC >= 3) {
        static_assert(IT == KC_ITERS, "given points: one group of points per thread");
        points_sweep<R, SRC == 4>(a, L.tab, r, ja, jb, first, visit);
    } else if constexpr (SRC == 2) {
        for (int jc = ja; jc < jb; jc += NT_DIMS) {
            const int DB = min(NT_DIMS, jb - jc);
            build_net_lds(a, L, r, jc, DB, tile0);
            for (int jj = 0; jj < DB; ++jj) {
                const NetDim<R, ALPHA, IT> dim(a, L, jc, jj);
#pragma unroll
                for (int l0 = 0; l0 < IT; l0 += KC_ITERS) {
                    R t[KC_ITERS], f[KC_ITERS];
                    dim.factors(l0, t, f);
                    visit(jc + jj, l0, t, f);
                }
            }
        }
    } else {
        constexpr int ORDER = SRC == 1 ? LDK_LINEAR : LDK_NATURAL;
        const uint64_t bfirst = ORDER == LDK_NATURAL ? brev64((uint64_t)first) : (uint64_t)first;
        for (int j = ja; j < jb; ++j) {
            const LatticeDim<R, ALPHA, ORDER, IT> dim(a, bfirst, j);
#pragma unroll
            for (int l0 = 0; l0 < IT; l0 += KC_ITERS) {
                R t[KC_ITERS], f[KC_ITERS];
                dim.factors(l0, t, f);
                visit(j, l0, t, f);
            }
        }
    }
}

// One block: the tile of KC_THREADS IT points blockIdx.x of replication
// blockIdx.y, dimensions z D .. z D + D - 1 (z = blockIdx.z, D =
// dims_per_block; every dimension when K1 is false); block z = 0 also sums
// the log zeta term.  The wavefront reduction of a dimension's sum (22
// instructions) is paid once per IT points of a thread.
template <typename R, int ALPHA, int SRC, bool K1, int IT>
__global__ __launch_bounds__(KC_THREADS) void k_kernel_grad(KgradArgs g)
{
    __shared__ NetLds<R, IT> L;
    __shared__ double red[KG_WAVES][64];
    const KcolArgs &a = g.k;
    const int r = blockIdx.y, d = a.ps.d;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int64_t cnt = a.n_max - a.n_min;
    const int64_t tile0 = g.tile_base + (int64_t)blockIdx.x * (KC_THREADS * IT);
    const int64_t first = tile0 + threadIdx.x;
    const int ja = K1 ? (int)blockIdx.z * g.dims_per_block : 0;
    const int jb = K1 ? min(ja + g.dims_per_block, d) : d;
    if constexpr (SRC == 2) {
        fill_net_lds<R, ALPHA>(L);
    } else if constexpr (SRC == 4) {
        fill_dsi_tables(L.tab, threadIdx.x, KC_THREADS);
        __syncthreads();
    }
    R pnz[IT], av[IT];
    int nz[IT];
    uint32_t valid = 0;
    int zero = 0;
#pragma unroll
    for (int l = 0; l < IT; ++l) {
        const int64_t i = first + (int64_t)l * KC_THREADS;
        const bool in = i >= a.n_min && i < a.n_max;
        const size_t at = (size_t)r * cnt + (i - a.n_min);
        valid |= (uint32_t)in << l;
        av[l] = in ? (R)g.a[at] : (R)0;
        pnz[l] = (R)1;
        if constexpr (K1) pnz[l] = in ? static_cast<const R *>(g.k1)[at] : (R)1;
        zero |= pnz[l] == (R)0;
        nz[l] = 0;
    }
    // With the forward column given, k1_i = zeta prod_l f_il already holds
    // the product, formed from the same factors bit for bit, so one sweep
    // over the block's own dimensions suffices: zeta t_ij prod_{l != j} f_il
    // = t_ij (k1_i / f_ij).  A block with a zero k1_i (a zero factor, or
    // underflow) forms the products itself.
    const bool from_k1 = K1 && !__syncthreads_or(zero);
    if (!from_k1) {
        // product of the nonzero factors and the number of zero factors
#pragma unroll
        for (int l = 0; l < IT; ++l) pnz[l] = (R)1;
        sweep<R, ALPHA, SRC, IT>(a, L, r, 0, d, tile0,
                                 [&](int, int l0, const R(&)[KC_ITERS], const R(&f)[KC_ITERS]) {
#pragma unroll
            for (int l = 0; l < KC_ITERS; ++l) {
                if (f[l] == (R)0) ++nz[l0 + l];
                else pnz[l0 + l] *= f[l];
            }
        });
    }
    // pnz already carries zeta when it came from k1
    const double zf = from_k1 ? 1.0 : a.zeta;
    double *part = g.part + ((size_t)r * g.tiles + blockIdx.x) * (d + 1);
    if (!K1 || blockIdx.z == 0) {
        // d/dlog zeta: sum_i a_i k1_i
        double zt = 0.0;
#pragma unroll
        for (int l0 = 0; l0 < IT; l0 += KC_ITERS) {
            R zs = (R)0;
#pragma unroll
            for (int l = l0; l < l0 + KC_ITERS; ++l)
                if (((valid >> l) & 1u) && nz[l] == 0) zs += av[l] * pnz[l];
            zt += (double)zs;
        }
        const double w = wave_sum(zt * zf);
        if (lane == 0) red[wave][0] = w;
        __syncthreads();
        if (threadIdx.x == 0) {
            double s = 0.0;
            for (int q = 0; q < KG_WAVES; ++q) s += red[q][0];
            part[d] = s;
        }
        __syncthreads();
    }
    // t_ij times the product of the other factors
    double acc = 0.0, sum = 0.0;
    auto emit = [&](int j, int l0, R ps) {
        sum = l0 == 0 ? (double)ps : sum + (double)ps;
        if (l0 + KC_ITERS < IT) return;
        const double w = wave_sum(sum * zf);
        const int at = (j - ja) & 63;
        if (at == lane) acc = w;
        if (at == 63 || j == jb - 1) {
            // block-uniform: every thread reaches these barriers
            const int j0 = j - at;
            red[wave][lane] = acc;
            __syncthreads();
            if ((int)threadIdx.x <= at) {
                double s = 0.0;
                for (int q = 0; q < KG_WAVES; ++q) s += red[q][threadIdx.x];
                part[j0 + threadIdx.x] = s;
            }
            __syncthreads();
        }
    };
    if (from_k1) {
        // no zero factor at any valid point of the tile
        sweep<R, ALPHA, SRC, IT>(a, L, r, ja, jb, tile0,
                                 [&](int j, int l0, const R(&t)[KC_ITERS], const R(&f)[KC_ITERS]) {
            emit(j, l0, sum_terms<R>([&](int l, auto &&divide) {
                const R c = av[l0 + l] * (t[l] * divide(pnz[l0 + l], f[l]));
                return ((valid >> (l0 + l)) & 1u) ? c : (R)0;
            }));
        });
    } else {
        sweep<R, ALPHA, SRC, IT>(a, L, r, ja, jb, tile0,
                                 [&](int j, int l0, const R(&t)[KC_ITERS], const R(&f)[KC_ITERS]) {
            emit(j, l0, sum_terms<R>([&](int l, auto &&divide) {
                const int k = l0 + l;
                const R q = divide(pnz[k], f[l]);
                const R one_zero = (nz[k] == 1 && f[l] == (R)0) ? pnz[k] : (R)0;
                const R other = nz[k] == 0 ? q : one_zero;
                const R c = av[k] * (t[l] * other);
                return ((valid >> k) & 1u) ? c : (R)0;
            }));
        });
    }
}

// grad[r][j] = sum over tiles of the partials in a fixed order: four
// interleaved sums, tile by tile, then (s0 + s1) + (s2 + s3).  A block takes 64
// components: its threads bring KG_FINAL_TILES tiles' partials into LDS
// together, then four threads per component add them in turn.  (One thread
// per component walking the tiles in memory was a chain of latencies: 60 us
// of the 75 us of a gradient of 512 tiles.)
constexpr int KG_FINAL_TILES = 64;
constexpr int KG_FINAL_THREADS = 1024;
__global__ __launch_bounds__(KG_FINAL_THREADS) void k_grad_final(const double *__restrict__ part, int64_t tiles,
                                                                 int d, double *__restrict__ grad)
{
    __shared__ double v[KG_FINAL_TILES][65];
    const int r = blockIdx.y, t = threadIdx.x, lane = t & 63, wave = t >> 6;
    const int j = blockIdx.x * 64 + lane;
    const double *p = part + (size_t)r * tiles * (d + 1) + (j <= d ? j : d);
    double s = 0.0;  // threads 0 .. 255: sum `wave` of component j
    for (int64_t q0 = 0; q0 < tiles; q0 += KG_FINAL_TILES) {
        const int n = (int)(tiles - q0 < KG_FINAL_TILES ? tiles - q0 : KG_FINAL_TILES);
        __syncthreads();
#pragma unroll
        for (int k = 0; k < KG_FINAL_TILES / (KG_FINAL_THREADS / 64); ++k) {
            const int q = wave + k * (KG_FINAL_THREADS / 64);
            if (q < n) v[q][lane] = p[(size_t)(q0 + q) * (d + 1)];
        }
        __syncthreads();
        if (wave < 4) {
            // the tiles past the last multiple of four belong to sum 0
            const int whole = q0 + n == tiles ? n & ~3 : n;
            for (int q = wave; q < whole; q += 4) s += v[q][lane];
            if (wave == 0)
                for (int q = whole; q < n; ++q) s += v[q][lane];
        }
    }
    __syncthreads();
    if (wave < 4) v[wave][lane] = s;
    __syncthreads();
    if (wave == 0 && j <= d)
        grad[(size_t)r * (d + 1) + j] = (v[0][lane] + v[1][lane]) + (v[2][lane] + v[3][lane]);
}

// The same sums for up to FEW tiles: a thread per component of every
// replication, its partials loaded before any is added.  Gradients of 2000
// lattices, n = 32, d = 2, FP64: 21.4 us with a block of 1024 threads per
// replication, 17.7 here.
template <int FEW>
__global__ __launch_bounds__(KC_THREADS) void k_grad_few(const double *__restrict__ part, int tiles, int d,
                                                         uint32_t count, double *__restrict__ grad)
{
    const uint32_t id = blockIdx.x * KC_THREADS + threadIdx.x;
    if (id >= count) return;
    const uint32_t r = id / (uint32_t)(d + 1), j = id % (uint32_t)(d + 1);
    const double *p = part + (size_t)r * tiles * (d + 1) + j;
    double v[FEW], s[4] = {};
#pragma unroll
    for (int q = 0; q < FEW; ++q)
        if (q < tiles) v[q] = p[(size_t)q * (d + 1)];
    const int whole = tiles & ~3;
#pragma unroll
    for (int q = 0; q < FEW; ++q)
        if (q < whole) s[q & 3] += v[q];
        else if (q < tiles) s[0] += v[q];
    grad[id] = (s[0] + s[1]) + (s[2] + s[3]);
}

int launch_grad_final(const double *part, int64_t tiles, int R, int d, double *grad, hipStream_t s)
{
    static_assert(65536ull * (LDK_MAX_D + 1) < 0x100000000ull, "R is a grid's y extent: 32-bit components");
    const uint32_t count = (uint32_t)R * (uint32_t)(d + 1);
    const dim3 few((count + KC_THREADS - 1) / KC_THREADS);
    if (tiles <= 4)
        hipLaunchKernelGGL(k_grad_few<4>, few, dim3(KC_THREADS), 0, s, part, (int)tiles, d, count, grad);
    else if (tiles <= 16)
        hipLaunchKernelGGL(k_grad_few<16>, few, dim3(KC_THREADS), 0, s, part, (int)tiles, d, count, grad);
    else
        hipLaunchKernelGGL(k_grad_final, dim3((d + 1 + 63) / 64, R), dim3(KG_FINAL_THREADS), 0, s, part, tiles, d,
                           grad);
    LDK_LAUNCH_CHECK();
    return LDK_OK;
}

template <typename R, int ALPHA, int SRC>
void launch_grad_k1(const KgradArgs &g, int it, dim3 grid, hipStream_t s)
{
    constexpr int N = KC_ITERS;
    if (!g.k1) {
        hipLaunchKernelGGL((k_kernel_grad<R, ALPHA, SRC, false, N>), grid, dim3(KC_THREADS), 0, s, g);
        return;
    }
    grid.z = (unsigned)((g.k.ps.d + g.dims_per_block - 1) / g.dims_per_block);
    if constexpr (SRC < 3 && sizeof(R) == 4) {
        if (it == 2 * N) {
            hipLaunchKernelGGL((k_kernel_grad<R, ALPHA, SRC, true, 2 * N>), grid, dim3(KC_THREADS), 0, s, g);
            return;
        }
    }
    hipLaunchKernelGGL((k_kernel_grad<R, ALPHA, SRC, true, N>), grid, dim3(KC_THREADS), 0, s, g);
}

template <typename R, int ALPHA>
void launch_grad_src(int src, const KgradArgs &g, int it, dim3 grid, hipStream_t s)
{
    switch (src) {
    case 0: launch_grad_k1<R, ALPHA, 0>(g, it, grid, s); break;
    case 1: launch_grad_k1<R, ALPHA, 1>(g, it, grid, s); break;
    default: launch_grad_k1<R, ALPHA, 2>(g, it, grid, s); break;
    }
}

template <typename R>
void launch_grad(int src, int uniform, const KgradArgs &g, int it, dim3 grid, hipStream_t s)
{
    if (src >= 3) {  // points given: generic orders
        if (src == 3) launch_grad_k1<R, 0, 3>(g, it, grid, s);
        else launch_grad_k1<R, 0, 4>(g, it, grid, s);
        return;
    }
    switch (uniform) {
    case 1: launch_grad_src<R, 1>(src, g, it, grid, s); break;
    case 2: launch_grad_src<R, 2>(src, g, it, grid, s); break;
    case 3: launch_grad_src<R, 3>(src, g, it, grid, s); break;
    case 4:
        if (src == 2) {
            launch_grad_k1<R, 4, 2>(g, it, grid, s);
            break;
        }
        [[fallthrough]];
    default: launch_grad_src<R, 0>(src, g, it, grid, s);
    }
}

// Tiles of KC_THREADS it points covering [n_min, n_max): aligned to absolute
// multiples of their size when regenerating, from n_min when points are given.
void grad_tiles(bool given, int it, int64_t n_min, int64_t n_max, int64_t *base, int64_t *tiles)
{
    const int64_t tile = (int64_t)KC_THREADS * it;
    *base = given ? n_min : (n_min / tile) * tile;
    *tiles = (n_max - *base + tile - 1) / tile;
}

}  // namespace

}  // namespace ldk

using namespace ldk;

extern "C" size_t ldk_kernel_grad_workspace_bytes(int R, int d, int64_t n_min, int64_t n_max,
                                                  int points_given)
{
    if (R < 1 || d < 1 || d > LDK_MAX_D || n_min < 0 || n_max < n_min) return 0;
    int64_t base, tiles;
    // the smallest tile gives the most partial sums
    grad_tiles(points_given != 0, KC_ITERS, n_min, n_max, &base, &tiles);
    return (size_t)R * (size_t)tiles * (size_t)(d + 1) * sizeof(double);
}

extern "C" int ldk_kernel_grad(const ldk_kernel *k, const ldk_pointset *ps, const uint64_t *pts,
                               const uint64_t *x0, int64_t n_min, int64_t n_max, int dtype,
                               const void *k1, const double *a, double *grad, void *ws,
                               ldk_stream stream)
{
    KgradArgs g{};
    int uniform = 0;
    const int st = prepare_kernel_args(k, ps, pts, x0, n_min, n_max, dtype, &g.k, &uniform);
    if (st) return st;
    const PointsetArgs &p = g.k.ps;
    if (!grad) return LDK_EINVAL;
    hipStream_t s = as_stream(stream);
    if (n_max == n_min) {
        // empty window: every sum is zero
        return launch_grad_final(nullptr, 0, p.R, p.d, grad, s);
    }
    if (!a || !ws) return LDK_EINVAL;
    const bool given = pts != nullptr;
    int it = KC_ITERS;
    g.dims_per_block = p.d;
    if (k1 && !given) {
        const GradSplit sp = grad_split(p.kind == LDK_LATTICE, dtype == LDK_F32, p.R, p.d, n_min, n_max);
        it = sp.it;
        g.dims_per_block = sp.dims;
    }
    grad_tiles(given, it, n_min, n_max, &g.tile_base, &g.tiles);
    if (g.tiles > 0x7fffffff) return LDK_ENOTSUP;
    g.a = a;
    g.k1 = k1;
    g.part = static_cast<double *>(ws);
    const int src = given ? (p.kind == LDK_DNET_B2 ? 4 : 3)
                          : (p.kind == LDK_DNET_B2 ? 2 : (p.order == LDK_LINEAR ? 1 : 0));
    const dim3 grid((unsigned)g.tiles, (unsigned)p.R);
    if (dtype == LDK_F64) launch_grad<double>(src, uniform, g, it, grid, s);
    else launch_grad<float>(src, uniform, g, it, grid, s);
    LDK_LAUNCH_CHECK();
    return launch_grad_final(g.part, g.tiles, p.R, p.d, grad, s);
}
