"""GPU tests of calls at the edges of the fast paths: parameters of other types
and devices, operands that are infinite or overlap, and the launch rules' shapes."""
import numpy as np
import pytest
import torch

import paper_2502_14256_amd as ldk
import workloads as W
from ldk_dev import kernel, pointset
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
