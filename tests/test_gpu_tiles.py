"""GPU tests of the tile shapes of the regenerating kernels: the first column
with 1, 4, 8 and 16 points per thread (chosen by the number of points) and the
gradient split over dimensions, and of the nested scrambling's blocks.  Every column shape forms a factor with the same
roundings, so a window's column equals, bit for bit, the columns of its
pieces; the gradient given the forward column is held to the gradient formed
without it (both gated elsewhere against the oracle)."""
import numpy as np
import pytest
import torch

import paper_2502_14256_amd as ldk
import workloads as W
from ldk_dev import dev_u64, kernel, kernel_scale, pointset

pytestmark = pytest.mark.gpu


def _inst(kind, m, d, R, alpha):
    w = W.small_lattice(31, m, d, R) if kind == "lattice" else W.small_net(32, m, d, R)
    al = np.array([1 + j % 3 for j in range(d)]) if alpha == 0 else np.full(d, alpha)
    w.update(alpha=al.astype(np.int32), gamma=0.8 ** np.arange(1, d + 1), zeta=1.1, sigma2=1e-3)
    return w


# points R (hi - lo): one below, at and above each step of the rule, windows
# that start and end inside a tile; d across the 16-dimension table chunk
WINDOWS = [(18, 1, 0, 2**18 - 1), (18, 1, 1, 2**18), (19, 1, 0, 2**19), (19, 3, 77, 2**19 - 5),
           (20, 1, 5, 2**20), (20, 1, 0, 2**20), (18, 17, 300, 2**18 - 300)]


@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
@pytest.mark.parametrize("kind,order,alpha", [("dnet", "natural", 2), ("dnet", "gray", 4),
                                              ("dnet", "gray", 0), ("dnet", "natural", 1),
                                              ("dnet", "natural", 3), ("lattice", "natural", 2),
                                              ("lattice", "linear", 0)])
@pytest.mark.parametrize("m,R,lo,hi", WINDOWS)
def test_column_equals_its_pieces(kind, order, alpha, dtype, m, R, lo, hi):
    d = 17 if R == 1 else 3
    w = _inst(kind, m, d, R, alpha)
    k, ps = kernel(w), pointset(w, order)
    full = ldk.kernel_column(k, ps, lo, hi, dtype=dtype)
    step = 50000 // R  # pieces of one point per thread
    for a in list(range(lo, hi, step))[:: max(1, (hi - lo) // step // 5)]:
        b = min(a + step, hi)
        part = ldk.kernel_column(k, ps, a, b, dtype=dtype)
        assert torch.equal(full[:, a - lo:b - lo], part), (a, b)


@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
@pytest.mark.parametrize("kind,order,alpha", [("dnet", "natural", 2), ("dnet", "gray", 0),
                                              ("dnet", "gray", 4), ("lattice", "natural", 2),
                                              ("lattice", "linear", 3)])
@pytest.mark.parametrize("m,d,R,lo", [(4, 1, 1, 0), (11, 5, 1, 0), (12, 33, 2, 9), (16, 17, 3, 0),
                                      (17, 70, 5, 1000), (16, 100, 20, 0)])
def test_gradient_given_the_column(kind, order, alpha, dtype, m, d, R, lo):
    w = _inst(kind, m, d, R, alpha)
    w["gamma"] = w["gamma"] * 0.3
    k, ps, n = kernel(w), pointset(w, order), 2**m
    k1 = ldk.kernel_column(k, ps, lo, n, dtype=dtype)
    g = torch.Generator("cuda").manual_seed(m)
    a = torch.randn((R, n - lo), dtype=torch.float64, device="cuda", generator=g)
    one = ldk.kernel_grad(k, ps, lo, n, a, dtype=dtype, k1=k1)
    two = ldk.kernel_grad(k, ps, lo, n, a, dtype=dtype)
    # each side within tol |a|_1 scale of the exact sums
    tol = 1e-14 if dtype == torch.float64 else 2e-6
    bound = 2 * tol * a.abs().sum(1, keepdim=True) * kernel_scale(w)
    assert (one.isfinite() & ((one - two).abs() <= bound)).all()


def test_gradient_with_a_zero_factor():
    """A tile holding a zero k1_i (a factor exactly zero) forms the products
    itself, also where the dimensions are split over blocks."""
    d, m = 9, 12
    w = _inst("dnet", m, d, 1, 1)
    w["gamma"] = np.full(d, 0.3)
    w["gamma"][4] = 2.0  # 1 + 2 K = 0 where K = 1 - 3/2 (beta = 1)
    k, ps, n = kernel(w), pointset(w), 2**m
    k1 = ldk.kernel_column(k, ps, 0, n)
    assert (k1 == 0).any()
    a = torch.randn((1, n), dtype=torch.float64, device="cuda")
    one = ldk.kernel_grad(k, ps, 0, n, a, k1=k1)
    two = ldk.kernel_grad(k, ps, 0, n, a)
    assert (one - two).abs().max() <= 2e-14 * a.abs().sum() * kernel_scale(w)


@pytest.mark.parametrize("R,d,m,lo,hi", [(1, 1, 7, 3, 128), (3, 5, 17, 37, 2**17 - 11),
                                         (16, 9, 16, 1, 2**16), (32, 61, 14, 0, 2**14),
                                         (2, 52, 20, 2**19 + 5, 2**20)])
def test_nus_block_shapes(orc, R, d, m, lo, hi):
    """Short and long blocks, flip tables of 0 to 12 digits, windows that
    start inside a tile of 64, dimensions that do not fill a block: bit-exact
    at both ends and in the middle."""
    t = W.small_net(m, m, d)
    seed = W.nus_seeds(m, R, d)
    ps = ldk.BPointSet("nus", R, d, gen=dev_u64(t["gen"]), seed=dev_u64(seed), m=m)
    x = ldk.gen_bpoints(ps, lo, hi).cpu().numpy()
    mid = (lo + hi) // 2
    for a, b in ((lo, min(lo + 70, hi)), (mid, min(mid + 70, hi)), (max(lo, hi - 70), hi)):
        ref = orc.unit_points(orc.nus_points(t["gen"], seed, m, a, b))
        assert np.array_equal(x[:, a - lo:b - lo], ref), (a, b)


@pytest.mark.parametrize("m", [0, 1, 5, 9, 12])
@pytest.mark.parametrize("R,nrhs", [(1, 2), (2, 8), (3, 100), (129, 2), (300, 3)])
def test_one_launch_net_fit_split_over_right_hand_sides(m, R, nrhs):
    """The right-hand sides of a one-pass net shared out over workgroups: the
    eigenvalues and solutions of the separate calls bit for bit, also with the
    eigenvalues written over the column (one workgroup a row then)."""
    n, s2 = 2**m, 1e-2
    g = torch.Generator("cuda").manual_seed(m)
    k1 = torch.rand((R, n), dtype=torch.float64, device="cuda", generator=g)
    k1[:, 0] += n
    y = torch.randn((R, nrhs, n), dtype=torch.float64, device="cuda", generator=g)
    lam_ref = ldk.eig("dnet", k1)
    c_ref, ld_ref = ldk.solve("dnet", lam_ref, s2, y), ldk.logdet(lam_ref, s2)
    over = k1.clone()
    for col, out in ((k1, None), (over, over)):
        lam, c, ld = ldk.fit("dnet", col, s2, y, lam=out)
        assert torch.equal(lam, lam_ref) and torch.equal(c, c_ref)
        assert torch.allclose(ld, ld_ref, rtol=1e-13, atol=1e-13 * n)


@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
@pytest.mark.parametrize("m", range(13, 21))
@pytest.mark.parametrize("nrhs", [2, 3])
def test_lattice_solve_by_coefficients_equals_single_solves(m, nrhs, dtype):
    """Every default top pass of a solve with its filter formed once (4 to 8
    axis bits, geometry fixed at compile time) against the solves of the single
    rows: both within the solve's first-order rounding bound; the fused fit
    runs the same kernel."""
    n, s2 = 2**m, 1e-2
    g = torch.Generator("cuda").manual_seed(m)
    k1 = torch.rand((1, n), dtype=torch.float64, device="cuda", generator=g)
    k1 = k1 + k1.roll(-1, 1).flip(1)
    k1[:, 0] += 2 * n
    k1 = k1.to(dtype)
    y = torch.randn((1, nrhs, n), dtype=torch.float64, device="cuda", generator=g).to(dtype)
    lam, c, _ = ldk.fit("lattice", k1, s2, y)
    many = ldk.solve("lattice", lam, s2, y)
    assert torch.equal(c, many)
    eps = float(torch.finfo(dtype).eps)
    inv = 1 / (lam + s2).abs().min()
    for q in range(nrhs):
        one = ldk.solve("lattice", lam, s2, y[:, q:q + 1].contiguous())
        tol = 2 * 4 * (2 * m + 2) * eps * inv * y[0, q].double().norm()
        assert (one[0, 0] - many[0, q]).double().norm() <= tol


@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
@pytest.mark.parametrize("m,R,nrhs", [(13, 1, 1), (13, 300, 3), (13, 3, 17), (14, 2, 8), (15, 5, 2),
                                      (16, 5, 3), (16, 40, 2), (17, 1, 1), (17, 33, 1), (18, 1, 9),
                                      (19, 2, 2), (20, 1, 1), (20, 3, 2), (21, 1, 1)])
def test_two_pass_net_fit_equals_separate_calls(m, R, nrhs, dtype):
    """A two-pass net's fit in three launches, a column tile's right-hand sides
    in one workgroup or shared out over several: the separate calls bit for
    bit, with the eigenvalues written over the column (FP64) and the solutions
    written over it too."""
    n, s2 = 2**m, 1e-2
    g = torch.Generator("cuda").manual_seed(m)
    k1 = torch.rand((R, n), dtype=torch.float64, device="cuda", generator=g)
    k1[:, 0] += n
    k1 = k1.to(dtype)
    y = torch.randn((R, nrhs, n), dtype=torch.float64, device="cuda", generator=g).to(dtype)
    lam_ref = ldk.eig("dnet", k1)
    c_ref, ld_ref = ldk.solve("dnet", lam_ref, s2, y), ldk.logdet(lam_ref, s2)
    runs = [(k1, None, None), (k1, None, y.clone())]
    if dtype == torch.float64:
        over = k1.clone()
        runs.append((over, over, None))
    if nrhs == 1:
        over = k1.clone()
        runs.append((over, None, over[:, None]))
    for col, lam_out, c_out in runs:
        rhs = c_out if c_out is not None and c_out.data_ptr() != col.data_ptr() else y
        lam, c, ld = ldk.fit("dnet", col, s2, rhs, lam=lam_out, c=c_out)
        assert torch.equal(lam, lam_ref) and torch.equal(c, c_ref)
        assert torch.allclose(ld, ld_ref, rtol=1e-13, atol=1e-13 * n)
    lam, c, ld = ldk.fit("dnet", k1, s2, y, logdet=False)
    assert ld is None and torch.equal(lam, lam_ref) and torch.equal(c, c_ref)


@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
@pytest.mark.parametrize("m,R", [(12, 3), (13, 5), (14, 1), (15, 2), (16, 9), (17, 1), (18, 2),
                                 (19, 1), (20, 1), (21, 1)])
def test_net_likelihood_terms(m, R, dtype):
    """The terms formed in the response's top pass (2^13 .. 2^20 points) and in
    the pass of their own, against the same formulas on the transform's output
    (orthonormal: a rounding of the working type more a side)."""
    n, s2 = 2**m, 1e-2
    g = torch.Generator("cuda").manual_seed(m)
    lam = torch.rand((R, n), dtype=torch.float64, device="cuda", generator=g) * 3
    y = torch.randn((R, n), dtype=torch.float64, device="cuda", generator=g).to(dtype)
    L, gr, ds = ldk.mll("dnet", lam, s2, y)
    q = ldk.transform("dnet", y).double().square() / (lam + s2)
    ref = 0.5 * (q - 1) / (lam + s2)
    eps, u = float(torch.finfo(dtype).eps), 2.0**-52
    # the transforms' values agree but for the scale's rounding; then a few FP64 ones
    bound = (2 * eps * q + 8 * u * (q + 1)) / (lam + s2)
    assert ((gr - ref).abs() <= bound).all()
    Lref = -0.5 * q.sum(1) - 0.5 * (lam + s2).log().sum(1) - 0.5 * n * np.log(2 * np.pi)
    assert ((L - Lref).abs() <= (2 * eps + m * u) * q.sum(1) + m * u * n * 8).all()
    assert ((ds - s2 * gr.sum(1)).abs() <= 2 * m * u * s2 * gr.abs().sum(1)).all()


@pytest.mark.parametrize("flags", [0, 1, 2, 4, 3, 5, 7])
@pytest.mark.parametrize("kind,base,R,d,lo,n", [("halton", 0, 16, 52, 5, 4133), ("halton", 0, 512, 1, 0, 129),
                                                ("halton", 0, 33, 54, 2**24 - 77, 2049),
                                                ("faure", 7, 32, 5, 3, 4111), ("faure", 2, 64, 2, 1, 2051),
                                                ("faure", 53, 8, 53, 0, 16385), ("faure", 67, 8, 60, 9, 16385)])
def test_digit_sets_two_points_a_lane_equal_their_pieces(kind, base, R, d, lo, n, flags):
    """Halton and Faure sets large enough for two points a lane (and one whose
    tile is too large for it) against windows small enough for one: the same
    arithmetic, bit for bit."""
    rng = np.random.default_rng(d)
    T = 53
    primes = [p for p in range(2, 252) if all(p % q for q in range(2, p))]
    lms = np.zeros((R, d, T, T), np.uint8)
    perm = np.zeros((R, d, T, 256), np.uint8)
    shift = np.zeros((R, d, T), np.uint8)
    for j in range(d):
        b = primes[j] if kind == "halton" else base
        lms[:, j] = np.tril(rng.integers(0, b, (R, T, T)), -1)
        lms[:, j, range(T), range(T)] = rng.integers(1, b, (R, T))
        perm[:, j, :, :b] = np.argsort(rng.random((R, T, b)), -1)
        shift[:, j] = rng.integers(0, b, (R, T))
    dev = lambda a: torch.from_numpy(a).cuda()
    ps = ldk.BPointSet(kind, R, d, base=base, flags=flags, lms=dev(lms), perm=dev(perm), shift=dev(shift))
    x = ldk.gen_bpoints(ps, lo, lo + n)
    step = max(1, min(1000 // R, n)) * 63
    for a in list(range(0, n, max(step, n // 4)))[:5] + [max(0, n - 65)]:
        b = min(n, a + min(step, 63 * 15))
        assert (b - a + 63) // 64 * R < 1024
        assert torch.equal(ldk.gen_bpoints(ps, lo + a, lo + b), x[:, a:b]), (a, b)


@pytest.mark.parametrize("m,R,d,n", [(17, 16, 3, 2**17 - 3), (18, 16, 17, 2**18 - 4095), (18, 16, 9, 2**18),
                                     (13, 512, 16, 2**12 + 1), (13, 1024, 5, 4096), (20, 4, 33, 2**20 - 1)])
def test_rqmc_net_points_per_thread(m, R, d, n):
    """Net tiles with 8 and 16 points per thread, d across the 16-dimension
    table chunk, ragged n: the replication means against the points written
    out (corner peak: relative error (d + 1) d u of a term for the sum in
    another order, the power's (d + 10) u, then sums of depth log2 n)."""
    w = _inst("dnet", m, d, R, 1)
    ps = pointset(w)
    coef = torch.full((d,), 1.0 / d, dtype=torch.float64, device="cuda")
    mu, _ = ldk.rqmc(ps, n, "corner_peak", coef)
    x = ldk.gen_points(ps, 0, n)
    f = torch.empty((R, n), dtype=torch.float64, device="cuda")
    for r in range(R):
        u = ((x[r] >> 32) & 0xffffffff).double() * 2.0**-32 + (x[r] & 0xffffffff).double() * 2.0**-64
        f[r] = (1 + u @ coef) ** -(d + 1.0)
    ref = f.mean(1)
    tol = 4 * (2 * d * (d + 1) + (d + 10) + 2 * m + 20) * 2.0**-52
    assert ((mu - ref).abs() <= tol * ref).all()
