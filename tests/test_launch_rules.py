"""CPU tests of the launch shapes (csrc/launchrules.hpp, plain C++): no more
points are formed for small replications than they hold, and full tiles keep
the most points per thread."""
import ctypes as C
import os
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))),
                    "paper_2502_14256_amd", "csrc")
SRC = '''
#include "launchrules.hpp"
extern "C" {
long long tiles(long long lo, long long hi, int it) { return ldk::window_tiles(lo, hi, it); }
int column(int lattice, int R, long long lo, long long hi) { return ldk::column_iters(lattice, R, lo, hi); }
int points(int lattice, int R, int d, long long lo, long long hi) { return ldk::points_column_iters(lattice, R, d, lo, hi); }
int grad(int lattice, int f32, int R, int d, long long lo, long long hi) { return ldk::grad_split(lattice, f32, R, d, lo, hi).it; }
int grad_dims(int f32, int R, int d, long long lo, long long hi) { return ldk::grad_split(false, f32, R, d, lo, hi).dims; }
int packed(int f32, long long rows, int m) { return ldk::packed_update(f32, rows, m); }
int pair(int nrhs, long long blocks) { return ldk::pair_rows(nrhs, blocks); }
int rqmc(int net, int R, long long n) { return ldk::rqmc_iters(net, R, n); }
}
'''


@pytest.fixture(scope="module")
def rules(tmp_path_factory):
    d = tmp_path_factory.mktemp("rules")
    (d / "r.cpp").write_text(SRC)
    subprocess.run(["g++", "-std=c++17", "-Wall", "-Werror", "-shared", "-fPIC", "-I", CSRC,
                    str(d / "r.cpp"), "-o", str(d / "r.so")], check=True)
    L = C.CDLL(str(d / "r.so"))
    i, q = C.c_int, C.c_longlong
    L.tiles.argtypes, L.tiles.restype = [q, q, i], q
    L.column.argtypes = [i, i, q, q]
    L.points.argtypes = L.grad_dims.argtypes = [i, i, i, q, q]
    L.grad.argtypes = [i, i, i, i, q, q]
    L.rqmc.argtypes = [i, i, q]
    L.packed.argtypes = [i, q, i]
    L.pair.argtypes = [i, q]
    return L


WINDOWS = [(0, 1), (0, 255), (0, 256), (0, 1000), (0, 1024), (0, 2048), (0, 2049), (0, 4096),
           (0, 4097), (5, 4101), (1024, 2048), (2048, 4096), (0, 10000), (77, 2**15), (0, 2**18)]


@pytest.mark.parametrize("R", [1, 3, 64, 300, 1024, 2048, 4096, 16384, 65535])
@pytest.mark.parametrize("lo,hi", WINDOWS)
def test_points_formed(rules, R, lo, hi):
    """Against tiles of 8 points per thread: nets form at most a quarter more
    points (a tile's tables are worth four), lattices and the sums a tenth."""
    eight = 8 * rules.tiles(lo, hi, 8)
    for lattice in (0, 1):
        it = rules.column(lattice, R, lo, hi)
        assert it * rules.tiles(lo, hi, it) <= (1.1 if lattice else 1.25) * eight
        for d in (4, 40):
            it = rules.points(lattice, R, d, lo, hi)
            assert it * rules.tiles(lo, hi, it) <= (1.1 if lattice else 1.25) * eight
    for d in (1, 16, 33, 100):
        for lattice in (0, 1):
            assert rules.grad(lattice, 0, R, d, lo, hi) == 8
            it = rules.grad(lattice, 1, R, d, lo, hi)
            assert it * rules.tiles(lo, hi, it) <= 1.1 * eight
    for net in (0, 1):
        it = rules.rqmc(net, R, hi)
        assert it * rules.tiles(0, hi, it) <= 1.1 * 8 * rules.tiles(0, hi, 8)


def test_small_replications_and_full_tiles(rules):
    assert [rules.column(k, 2048, 0, 2**11) for k in (0, 1)] == [8, 8]
    assert [rules.column(k, 4096, 0, 2**10) for k in (0, 1)] == [4, 4]
    assert [rules.column(k, 16384, 0, 2**8) for k in (0, 1)] == [1, 1]
    assert [rules.column(k, 1024, 0, 2**12) for k in (0, 1)] == [16, 16]
    assert [rules.column(0, 1, 0, 2**m) for m in (17, 18, 20, 22)] == [1, 4, 8, 16]
    assert [rules.column(1, 1, 0, 2**m) for m in (18, 19, 20, 22)] == [1, 4, 8, 16]
    assert rules.grad(0, 1, 1024, 16, 0, 2**11) == 8 and rules.grad(0, 1, 64, 64, 0, 2**16) == 16
    # a lattice of few dimensions takes 8 in more than one round of blocks, but
    # for a long sum over its tiles
    assert [rules.grad(1, 1, 895, d, 0, 2**13) for d in (2, 11, 12)] == [8, 8, 16]
    assert rules.grad(1, 1, 64, 2, 0, 2**16) == 16 and rules.grad(1, 1, 4, 2, 0, 2**22) == 16
    assert rules.grad(1, 1, 1, 2, 0, 2**22) == 16 and rules.grad(0, 1, 895, 2, 0, 2**13) == 16
    assert rules.rqmc(1, 1024, 2**11) == 8 and rules.rqmc(1, 16, 2**18) == 16
    assert rules.rqmc(0, 16, 2**18) == 8 and rules.rqmc(1, 2048, 512) == 2
    assert rules.grad_dims(0, 1, 16, 0, 2**10) == 2
    # a grid of nearly three blocks a compute unit stays whole
    blocks = lambda tiles, d: -(-d // rules.grad_dims(0, tiles, d, 0, 2**11))
    assert [blocks(758, d) for d in (2, 3, 6, 16)] == [1, 1, 1, 1]
    assert [blocks(640, d) for d in (3, 6, 16)] == [1, 1, 2] and [blocks(500, d) for d in (3, 6)] == [2, 2]


def test_column_beside_the_point_words(rules):
    """One point per thread only while the launch is short; lattices and nets of
    one chunk of dimensions take 8 from 2^18 points on, where fewer measured
    slower."""
    pts = lambda lattice, d: [rules.points(lattice, 1, d, 0, 2**m) for m in (16, 17, 18, 19, 20, 22)]
    assert pts(1, 4) == pts(1, 40) == pts(0, 16) == [1, 4, 8, 8, 8, 16]
    assert pts(0, 17) == [1, 4, 4, 4, 8, 16]
    assert rules.points(1, 10, 4, 0, 2**15) == 8 and rules.points(1, 4096, 4, 0, 2**10) == 4


def test_packed_update(rules):
    """Short rows, and a few rows of FP32 in two passes, transform rows of n."""
    for f32, short in ((0, {4, 5, 6, 7, 8}), (1, {4, 5, 6, 7, 8, 9})):
        assert {m for m in range(2, 26) if not rules.packed(f32, 2048, m)} == short
    assert not rules.packed(0, 1, 1) and rules.packed(0, 1, 14)
    assert [m for m in range(10, 26) if not rules.packed(1, 1, m)] == [14, 15, 16, 17, 18, 19]
    assert [rules.packed(1, R, 15) for R in (16, 17)] == [0, 1]


def test_right_hand_sides_paired_in_a_full_grid_only(rules):
    assert [rules.pair(q, b) for q, b in ((2, 4), (2, 1022), (2, 1024), (8, 4096), (3, 3000), (1, 4096))] == \
        [0, 0, 1, 1, 0, 0]
