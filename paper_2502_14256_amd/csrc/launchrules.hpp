// Launch shapes of the kernels that regenerate points, as functions of the
// problem's sizes alone (plain host C++).
//
// A block takes KC_THREADS consecutive indices per point of a thread, in tiles
// aligned to absolute multiples of the tile; indices outside the window are
// formed and dropped.
#pragma once

#include <cstdint>

namespace ldk {

constexpr int KC_THREADS = 256;
constexpr int KC_LOG_THREADS = 8;
constexpr int KC_ITERS = 8;  // points per thread (spaced KC_THREADS apart) of the gradient
constexpr int NT_DIMS = 16;  // dimensions whose net tables sit in LDS at once

// Tiles of KC_THREADS it indices that cover [n_min, n_max).
inline int64_t window_tiles(int64_t n_min, int64_t n_max, int it)
{
    const int64_t tile = (int64_t)KC_THREADS * it;
    return (n_max - (n_min / tile) * tile + tile - 1) / tile;
}

// The points per thread, of `its` (descending, the first is the most that the
// size of the whole problem suggests), whose tiles of one replication cost
// least.  A tile costs its points and `setup` points' worth of per-dimension
// constants and tables, so a replication that does not fill a large tile takes
// a smaller one (column, lattice FP64, d = 16, us for 16 points per thread / by
// this rule: R = 2048, n = 2^11 38.5 / 22.9; R = 16384, n = 2^8 243 / 34.2).
template <int N>
inline int least_work(const int (&its)[N], int most, int setup, int64_t n_min, int64_t n_max)
{
    int best = most;
    int64_t cost = window_tiles(n_min, n_max, most) * (setup + most);
    for (int it : its) {
        const int64_t c = window_tiles(n_min, n_max, it) * (setup + it);
        if (it < most && c < cost) {
            cost = c;
            best = it;
        }
    }
    return best;
}

// Kernel column: by the number of points R cnt, more points per thread (tables
// and per-dimension constants serve more of them) where that leaves one (nets,
// 4 points) to four (16 points) blocks per compute unit, one point where the
// launch would otherwise leave compute units idle or hang on one block's chain
// of dimensions.  Measured (us
// for 1 / 4 / 8 / 16 points per thread, order 2, FP64): net 2^16 x d = 16: 8.7 /
// 10.3 / 13.3 / 20.3; 2^18 x 32: 21.6 / 19.5 / 24.8 / 38.5; 2^20 x 32: 64 /
// 28.8 / 26.9 / 40; 2^22 x 64: 401 / 168 / 140 / 139 (FP32 206 / 81 / 62 / 59);
// lattice 2^16 x 16: 3.9 / 4.8 / 5.7 / 7.6; 2^18 x 32: 7.5 / 7.5 / 9.1 / 12.4;
// 2^20 x 32: 18.6 / 13.4 / 12.7 / 13.5; 2^22 x 64: 107 / 70 / 64 / 62.  From
// the 2^22 rows a tile's setup is worth 3.5 points (nets; FP32 4.3) and 0.85
// (lattices).
inline int column_iters(bool lattice, int R, int64_t n_min, int64_t n_max)
{
    constexpr int its[] = {16, 8, 4, 1};
    const int64_t pts = (int64_t)R * (n_max - n_min), one = (int64_t)1 << (lattice ? 19 : 18);
    const int most = pts < one ? 1 : pts < (1 << 20) ? 4 : pts < (1 << 22) ? 8 : 16;
    return least_work(its, most, lattice ? 1 : 4, n_min, n_max);
}

// The column beside the point words in one launch: column blocks share the
// chip with the stores, so one point per thread only while the launch is short.
// Measured (us for 1 / 4 / 8 / 16 points per thread, FP64): lattice 2^16 x d =
// 16: 5.6 / 5.6 / 7.2 / 9.2; 2^17 x 2: 4.6 / 4.4 / 4.4 / 4.4, x 32: 9.7 / 11.3 /
// 13.1 / 16.5; 160000 x 16: 7.5 / 8.4 / 8.2 / 10.4, x 64: 20.6 / 17.9 / 21.2 /
// 27.8; 2^18 x 6: 7.1 / 6.3 / 6.4 / 6.6, x 64: 30.4 / 22.8 / 22.7 / 27.8; 2^19 x
// 16: 14.2 / 17.3 / 13.7 / 13.5; 2^22 x 6: 37.6 / 39.1 / 47.2 / 38.2, x 16: 106 /
// 111 / 105 / 107.  Net 2^16 x 64: 32.2 / 33.9 / 47.1 / 74.5; 2^17 x 4: 15.1 /
// 14.1 / 14.2 / 14.3, x 32: 30.0 / 26.3 / 26.2 / 40.8; 2^18 x 16: 29.4 / 22.0 / 21.1
// / 21.6; 2^19 x 6: 25.0 / 18.6 / 18.3 / 17.7, x 32: 60.5 / 38.8 / 44.7 / 49.1.
inline int points_column_iters(bool lattice, int R, int d, int64_t n_min, int64_t n_max)
{
    constexpr int its[] = {16, 8, 4, 1};
    const int64_t pts = (int64_t)R * (n_max - n_min);
    const int64_t eight = (int64_t)1 << (lattice || d <= NT_DIMS ? 18 : 20);
    const int most = pts < (1 << 17) ? 1 : pts < eight ? 4 : pts < (1 << 22) ? 8 : 16;
    return least_work(its, most, lattice ? 1 : 4, n_min, n_max);
}

// Gradient given the forward column, points regenerated.  The dimensions are
// independent then, so a grid short of two to three blocks per compute unit is
// split over them, sooner the more dimensions a block keeps (FP64 net, whole /
// split, us: d = 3, 384 tiles 11.3 / 10.4, 640 13.4 / 14.4, 758 13.5 / 18.7; d =
// 6, 512 15.9 / 14.6, 758 19.2 / 23.3; d = 16, 640 36.0 / 31.6, 758 37.3 / 38.6).
// A large grid takes twice the points per thread in FP32 (the dimension's setup
// and reduction serve more factors; in FP64, where it would change the order of
// the sums, nets lose their occupancy to it and lattices gain 5 %).  Measured
// (us, D = 16 / 8 / 4 / 2 dimensions per block): FP64 net 2^16 points x d = 16:
// 21.0 / 13.8 / 10.2 / 8.8; 2^18 x 32: 22.0 / 18.2 / 17.0 / 20.5; 2^20 x 32: 42.4 /
// 43.8 / 48.3 / 63.6; 16 instead of 8 points per thread at 2^22 x 64: lattice FP32
// 133 -> 127, net FP32 132 -> 130, net FP64 268 -> 272: a tile's setup is worth
// less than a point.  A lattice of a few dimensions is bound by its column and
// weights, and in a grid of more than one round of blocks fewer of its reads are
// in flight then (895 x 2^13, 8 / 16 points: d = 2 25.0 / 28.2, d = 8 42.3 / 42.1,
// d = 12 55.2 / 53.3; but 64 x 2^16, d = 2: 20.0 / 18.6), unless a replication has
// so many tiles that their sum is the longer part (2^22, d = 2: 77 / 46).
struct GradSplit {
    int it, dims;
};
inline GradSplit grad_split(bool lattice, bool f32, int R, int d, int64_t n_min, int64_t n_max)
{
    constexpr int its[] = {2 * KC_ITERS, KC_ITERS};
    auto blocks = [&](int it, int dims) {
        return window_tiles(n_min, n_max, it) * R * ((d + dims - 1) / dims);
    };
    GradSplit s{KC_ITERS, NT_DIMS};
    const int64_t b2 = blocks(2 * KC_ITERS, NT_DIMS);
    const bool twice = !lattice || d >= 12 || b2 <= 1280 || window_tiles(n_min, n_max, KC_ITERS) >= 256;
    if (f32 && twice && b2 >= 1024) s.it = least_work(its, 2 * KC_ITERS, 1, n_min, n_max);
    while (s.dims > 2 && blocks(s.it, s.dims) < (s.dims > 8 ? 704 : s.dims > 4 ? 640 : 512)) s.dims /= 2;
    return s;
}

// RQMC sums: 8 points per thread, 2 where the grid would then hold fewer than
// two blocks per compute unit; 16 for nets that still fill four a unit (the
// blocks' tables and a dimension's constants serve twice the points).  Corner
// peak (us a call, 8 / 16 points): R = 16, n = 2^18, d = 50: 67.2 / 64.4; 2^20:
// 213 / 204; R = 21, n = 2^20, d = 25: 159 / 150; R = 1, n = 2^22, d = 8: 31.2 /
// 25.8: a tile's setup is worth about a point.
inline int rqmc_iters(bool net, int R, int64_t n)
{
    constexpr int its[] = {16, 8, 2};
    const int most = net && window_tiles(0, n, 16) * R >= 1024 ? 16 : window_tiles(0, n, 8) * R < 512 ? 2 : 8;
    return least_work(its, most, 1, 0, n);
}

// Lattice solves by precomputed coefficients, FP64: whether a workgroup runs the
// same tile of two right-hand sides in turn (the coefficients then come from the
// L2 lines that the first one brought in; the same bits).  It needs two
// workgroups a CU after the halving.  Measured (solve, us, paired / not, blocks
// after the halving): n = 2^13 19.4 / 16.2 (2), 28.1 / 25.2 (128); 2^16 33.6 / 32.3
// (256), 50.0 / 51.0 (512); 2^19 51.9 / 53.1 (512), 173 / 182 (2048); 2^20 42.2 /
// 40.4 (256), 56.3 / 58.0 (512).  FP32: 0.97 to 1.02 of each other from 512 on,
// and 104 against 116 unpaired at 2^20: never paired.
inline bool pair_rows(int nrhs, int64_t blocks) { return nrhs % 2 == 0 && blocks >= 1024; }

// The n -> 2n update of a lattice on its real new half: packed rows of n / 2
// complex entries, or rows of n.  Packed halves the transform and lengthens each
// workgroup's chain (untangling, two twiddles), so it loses where many short rows
// are a workgroup of one or a few lanes each, and for a few rows of FP32 in two
// passes.  Measured (us, rows of n / packed): FP64 m = 3, 1 row 4.2 / 3.5; m = 5,
// 256 rows 5.9 / 6.1, 2048 rows 9.9 / 14.5; m = 7, 2048 rows 9.5 / 16.3; m = 8
// 10.3 / 11.4; m = 9 14.7 / 13.9; FP32 m = 9, 256 rows 6.3 / 6.7, m = 10 7.2 / 6.2;
// m = 15, 1 row 12.9 / 14.3, 16 rows 14.3 / 15.5; m = 17, 1 row 14.3 / 15.0, 16
// rows 25.4 / 20.5; m = 19, 1 row 17.0 / 16.7.
inline bool packed_update(bool f32, int64_t rows, int m)
{
    if (m < 2 || (m >= 4 && m <= (f32 ? 9 : 8))) return false;
    return !(f32 && m >= 14 && rows << (m - 13) <= 64);
}

}  // namespace ldk
