"""GPU tests of calls at the edges of the fast paths: parameters of other types
and devices, operands that are infinite or overlap, and the launch rules' shapes."""
import numpy as np
import pytest
import torch

import paper_2502_14256_amd as ldk
import test_gpu_cubature as cub
import workloads as W
from ldk_dev import dev_u64, kernel, pointset
from paper_2502_14256_amd.autograd import MarginalLogLikelihood

pytestmark = pytest.mark.gpu

F64, F32 = torch.float64, torch.float32


@pytest.mark.parametrize("dg,dz,ds,dev", [(F64, F64, F64, "cuda"), (F32, F32, F32, "cuda"),
                                          (F32, F64, F64, "cuda"), (F64, F32, F64, "cuda"),
                                          (F64, F64, F64, "cpu"), (F32, F32, F64, "cpu")])
def test_likelihood_parameters_of_any_float_type(dg, dz, ds, dev):
    """Each parameter's exp is taken in its own type and on its own device, in
    both passes: the likelihood of exactly those numbers, bit for bit, and the
    same gradient with and without recomputation."""
    w = W.small_net(3, 9, 3, 2)
    ps, n = pointset(w), 2**9
    y = torch.from_numpy(np.ascontiguousarray(w["y"][:, 0])).cuda()
    lg = torch.tensor([-0.1, -0.7, 0.3], dtype=dg, device="cuda", requires_grad=True)
    lz = torch.tensor(0.13, dtype=dz, device=dev, requires_grad=True)
    ls = torch.tensor(-2.0, dtype=ds, device=dev, requires_grad=True)
    k = ldk.Kernel("dnet", [2, 2, 2], torch.exp(lg.detach()).double(), torch.exp(lz.detach()).item())
    lam = ldk.eig("dnet", ldk.kernel_column(k, ps, 0, n))
    ref = ldk.mll("dnet", lam, torch.exp(ls.detach()).item(), y)[0]
    grads = []
    for recompute in (True, False):
        L = MarginalLogLikelihood.apply(lg, lz, ls, ps, "dnet", [2, 2, 2], y, F64, recompute)
        assert torch.equal(L, ref)
        grads.append(torch.autograd.grad(L.sum(), (lg, lz, ls)))
    for a, b, t in zip(*grads, (lg, lz, ls)):
        assert a.dtype == t.dtype and a.device == t.device and torch.equal(a, b)
        assert a.isfinite().all()


@pytest.mark.parametrize("kind", ["dnet", "lattice"])
@pytest.mark.parametrize("given", ["column", "nothing"])
def test_gradient_of_infinite_and_overflowing_products(kind, given):
    """P / f with P infinite, or past the largest number: the quotient that IEEE
    division gives (infinite), not NaN; a large f keeps its finite quotient."""
    m, n = 10, 1024
    gam = [0.5, 0.3, 0.2, 0.25] if given == "column" else [0.9, 0.8, 0.5, 0.4]
    w = W.small_net(3, m, 4, 1) if kind == "dnet" else W.small_lattice(3, m, 4, 1)
    w.update(alpha=[2, 1, 2, 1], gamma=gam, zeta=1.0)
    ps, i = pointset(w), 517
    a = torch.zeros((1, n), dtype=F64, device="cuda")
    a[0, i] = 1.0
    one = lambda j, g: ldk.kernel_column(
        ldk.Kernel(kind, w["alpha"], torch.tensor([g if q == j else 0.0 for q in range(4)],
                                                  dtype=F64, device="cuda"), 1.0), ps, 0, n)[0, i].item()
    f = [one(j, gam[j]) for j in range(4)]
    f = np.array(f)  # the four factors of point i
    if given == "column":
        k = kernel(w)
        k1 = ldk.kernel_column(k, ps, 0, n)
        for v in (np.inf, -np.inf, 1.7e308, np.nan):
            k1[0, i] = v
            with np.errstate(over="ignore", invalid="ignore"):
                want = np.append((f - 1) * (v / f), v)
            got = ldk.kernel_grad(k, ps, 0, n, a, k1=k1)[0].cpu().numpy()
            assert np.array_equal(np.isnan(got), np.isnan(want))
            assert np.array_equal(got[np.isinf(want)], want[np.isinf(want)])
            ok = np.isfinite(want)
            assert np.allclose(got[ok], want[ok], rtol=1e-13)
        return
    # products formed by the gradient: one factor of 2^1020 or more overflows
    # P, or leaves P finite at f >= 2^1022
    for big in (4e307, 1.1e308):
        gam = np.array([big, 0.8, 0.5, 0.4])
        k = ldk.Kernel(kind, w["alpha"], torch.from_numpy(gam).cuda(), 1.0)
        g = ldk.kernel_grad(k, ps, i, i + 1, a[:, i:i + 1].contiguous())[0].cpu().numpy()
        f0 = one(0, big)  # a lattice's polynomial overflows itself here (NaN)
        with np.errstate(over="ignore", invalid="ignore"):
            P = f0 * f[1] * f[2] * f[3]
            want = np.append(np.array([f0, *(f[1:] - 1)]) * (P / np.array([f0, *f[1:]])), P)
        assert np.array_equal(np.isnan(g), np.isnan(want)), (g, want)
        assert np.array_equal(g[np.isinf(want)], want[np.isinf(want)])
        ok = np.isfinite(want)
        assert np.allclose(g[ok], want[ok], rtol=1e-12)


@pytest.mark.parametrize("m", [3, 10, 12])
@pytest.mark.parametrize("R,nrhs", [(1, 1), (1, 3), (4, 1), (4, 3), (300, 2)])
@pytest.mark.parametrize("at", [0, 1])
def test_one_pass_net_fit_over_its_column(m, R, nrhs, at):
    """Solutions written over the column: every column row is read before any
    solution lies over it, wherever in c the column begins (row 0, or the last
    row it fits at)."""
    n, s2 = 2**m, 1e-2
    g = torch.Generator("cuda").manual_seed(m)
    k1 = torch.rand((R, n), dtype=F64, device="cuda", generator=g)
    k1[:, 0] += n
    y = torch.randn((R, nrhs, n), dtype=F64, device="cuda", generator=g)
    lam_ref = ldk.eig("dnet", k1)
    c_ref, ld_ref = ldk.solve("dnet", lam_ref, s2, y), ldk.logdet(lam_ref, s2)
    c = torch.empty((R, nrhs, n), dtype=F64, device="cuda")
    first = at * (R * nrhs - R) * n
    col = c.view(-1)[first:first + R * n].view(R, n)
    col.copy_(k1)
    lam, c, ld = ldk.fit("dnet", col, s2, y, c=c)
    assert torch.equal(lam, lam_ref) and torch.equal(c, c_ref)
    assert torch.allclose(ld, ld_ref, rtol=1e-13, atol=1e-13 * n)


@pytest.mark.parametrize("m", [3, 10, 12])
def test_one_pass_lattice_fit_over_another_row_of_its_column(m):
    """One right-hand side per replication, the solutions one row behind the
    column they lie over: every column row is read first."""
    n, s2, R = 2**m, 1e-2, 40
    g = torch.Generator("cuda").manual_seed(m)
    k1 = torch.rand((R, n), dtype=F64, device="cuda", generator=g)
    k1[:, 0] += 2 * n
    y = torch.randn((R, 1, n), dtype=F64, device="cuda", generator=g)
    lam_ref = ldk.eig("lattice", k1)
    c_ref, ld_ref = ldk.solve("lattice", lam_ref, s2, y), ldk.logdet(lam_ref, s2)
    buf = torch.empty(((R + 1) * n,), dtype=F64, device="cuda")
    col, c = buf[n:].view(R, n), buf[:R * n].view(R, 1, n)
    col.copy_(k1)
    lam, c, ld = ldk.fit("lattice", col, s2, y, c=c)
    # (the fused and the separate passes may contract a twiddle differently)
    assert torch.allclose(lam, lam_ref, rtol=0, atol=1e-13 * n * m)
    assert torch.allclose(c, c_ref, rtol=0, atol=1e-12 * y.abs().max().item())
    assert torch.allclose(ld, ld_ref, rtol=1e-12, atol=1e-12 * n)


@pytest.mark.parametrize("tiles", [1, 2, 3, 4, 5, 8, 15, 16, 17, 19, 64, 66])
@pytest.mark.parametrize("kind,d,R", [("lattice", 2, 300), ("dnet", 70, 2)])
@pytest.mark.parametrize("with_k1", [False, True])
def test_gradient_tile_sums(kind, d, R, tiles, with_k1):
    """The gradient is the sum over tiles of 2048 points in the stated order (four
    interleaved sums, the tiles past the last multiple of four in the first),
    bit for bit, by either of the two summing kernels."""
    n = 2048 * tiles
    w = W.small_lattice(7, 1, d, R, m_max=18) if kind == "lattice" else W.small_net(7, 1, d, R, m_max=18)
    w.update(alpha=[2] * d, gamma=0.3 * 0.8 ** np.arange(d), zeta=1.1)
    k, ps = kernel(w), pointset(w)
    g = torch.Generator("cuda").manual_seed(tiles)
    a = torch.randn((R, n), dtype=F64, device="cuda", generator=g)
    k1 = ldk.kernel_column(k, ps, 0, n) if with_k1 else None
    part = lambda t, q: None if t is None else t[:, 2048 * q:2048 * (q + 1)].contiguous()
    s = [torch.zeros((R, d + 1), dtype=F64, device="cuda") for _ in range(4)]
    for q in range(tiles):
        s[q % 4 if q < tiles // 4 * 4 else 0] += ldk.kernel_grad(k, ps, 2048 * q, 2048 * (q + 1), part(a, q),
                                                                  k1=part(k1, q))
    assert torch.equal(ldk.kernel_grad(k, ps, 0, n, a, k1=k1), (s[0] + s[1]) + (s[2] + s[3]))


@pytest.mark.parametrize("R,d,m,lo,hi", [(1, 1, 16, 0, 2**16), (16, 1, 15, 3, 2**15), (2, 2, 13, 65, 8000),
                                         (7, 3, 12, 0, 4096), (5, 6, 14, 1, 2**14 - 1), (3, 7, 10, 0, 1000),
                                         (4, 9, 13, 100, 101), (1, 13, 12, 0, 64)])
def test_nus_dimensions_that_do_not_fill_a_block(orc, R, d, m, lo, hi):
    """One to four dimensions a block, uneven groups: bit-exact at both ends."""
    t = W.small_net(m, m, d)
    seed = W.nus_seeds(m, R, d)
    ps = ldk.BPointSet("nus", R, d, gen=dev_u64(t["gen"]), seed=dev_u64(seed), m=m)
    x = ldk.gen_bpoints(ps, lo, hi).cpu().numpy()
    for a, b in ((lo, min(lo + 130, hi)), (max(lo, hi - 130), hi)):
        ref = orc.unit_points(orc.nus_points(t["gen"], seed, m, a, b))
        assert np.array_equal(x[:, a - lo:b - lo], ref), (a, b)


def test_nus_work_goes_with_the_dimensions():
    """One dimension costs well below four (a third measured, the same when the
    block's other waves repeat it)."""
    us = {}
    for d in (1, 4):
        t = W.small_net(5, 16, d)
        ps = ldk.BPointSet("nus", 16, d, gen=dev_u64(t["gen"]), seed=dev_u64(W.nus_seeds(5, 16, d)), m=16)
        out = torch.empty((16, 2**16, d), dtype=F64, device="cuda")
        times = []
        for _ in range(8):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            for _ in range(10):
                ldk.gen_bpoints(ps, 0, 2**16, out=out)
            b.record()
            b.synchronize()
            times.append(a.elapsed_time(b))
        us[d] = min(times)
    assert us[1] < 0.7 * us[4], us


@pytest.mark.parametrize("dtype", [F64, F32])
@pytest.mark.parametrize("B,m", [(1, 2), (5, 3), (3, 4), (1000, 5), (2, 9), (3, 10), (1, 14), (65, 14), (2, 16), (2, 17),
                                 (1, 18), (3, 18), (1, 19), (1, 20), (2, 20), (1, 21), (1, 22)])
def test_lattice_update_plans(B, m, dtype):
    """Every plan of the n -> 2n update (rows of n and packed rows; one, two and
    three passes; every top pass of a fixed geometry; several rows), against the
    transform and the eigenvalues of the whole, also in place (the old half's
    values at the start of the output)."""
    n = 2**m
    g = torch.Generator("cuda").manual_seed(m)
    cdt = torch.complex128 if dtype == F64 else torch.complex64
    y = torch.randn((B, 2 * n), dtype=F64, device="cuda", generator=g).to(dtype)
    old, new = y[:, :n].contiguous(), y[:, n:].contiguous()
    whole = ldk.transform("lattice", y.to(torch.complex128))
    yt = ldk.transform("lattice", old.to(torch.complex128)).to(cdt)
    got = ldk.update_double("lattice", yt, new)
    rel = lambda a, b: ((a - b).norm() / b.norm()).item()
    assert rel(got.to(torch.complex128), whole) < (1e-14 * (m + 10) if dtype == F64 else 3e-7 * (m + 10))
    lam_old, lam = ldk.eig("lattice", old.double()), ldk.eig("lattice", y.double())
    lam_got = ldk.eig_update_double("lattice", lam_old, new)
    assert rel(lam_got, lam) < 1e-14 * (m + 10)
    if B == 1:
        buf = torch.empty((1, 2 * n), dtype=cdt, device="cuda")
        buf[:, :n] = yt
        assert torch.equal(ldk.update_double("lattice", buf[:, :n], new, out=buf), got)
        buf = torch.empty((1, 2 * n), dtype=F64, device="cuda")
        buf[:, :n] = lam_old
        assert torch.equal(ldk.eig_update_double("lattice", buf[:, :n], new, out=buf), lam_got)


@pytest.mark.parametrize("m", [15, 17, 18, 19])
@pytest.mark.parametrize("dtype", [F64, F32])
def test_cubature_top_passes(orc, m, dtype):
    """The sizes whose top passes (5 to 8 axis bits) the cubature's own tests leave
    out, with their oracle and bounds."""
    cub.test_wce(orc, "lattice", m, dtype)
    cub.test_bayes_cubature(orc, "lattice", m, dtype)


@pytest.mark.parametrize("dtype", [F64, F32])
@pytest.mark.parametrize("m,nrhs", [(13, 1), (13, 20), (16, 3), (18, 2)])
def test_two_pass_net_fit_of_bad_rows(m, nrhs, dtype):
    """A row with some lambda + s2 <= 0 (log-det NaN), columns with an infinity and
    a NaN, and responses with an infinity, beside a good row: eigenvalues and
    solutions as the separate calls give them, bit for bit."""
    n, R, s2 = 2**m, 5, 1e-2
    g = torch.Generator("cuda").manual_seed(m)
    k1 = torch.rand((R, n), dtype=F64, device="cuda", generator=g)
    k1[:, 0] += n
    k1[1, 0] -= 1.2 * n  # lambda of about -0.2 n, the sum row apart
    k1[2, 5], k1[3, n - 1] = float("inf"), float("nan")
    k1 = k1.to(dtype)
    y = torch.randn((R, nrhs, n), dtype=F64, device="cuda", generator=g).to(dtype)
    y[4, 0, 7] = float("-inf")
    lam_ref = ldk.eig("dnet", k1)
    c_ref, ld_ref = ldk.solve("dnet", lam_ref, s2, y), ldk.logdet(lam_ref, s2)
    assert ld_ref[[0, 4]].isfinite().all() and ld_ref[1:4].isnan().all()
    same = lambda a, b: torch.equal(a.isnan(), b.isnan()) and torch.equal(a[~a.isnan()], b[~b.isnan()])
    for logdet in (True, False):
        lam, c, ld = ldk.fit("dnet", k1, s2, y, logdet=logdet)
        assert same(lam, lam_ref) and same(c, c_ref)
        if logdet:
            assert ld[1:4].isnan().all()
            assert torch.allclose(ld[[0, 4]], ld_ref[[0, 4]], rtol=1e-13, atol=1e-13 * n)
