"""The slot-fastest vectors of a 2D apply: batches around the 16-slot chunks
and the move kernels' power-of-two tiles, a batch of more right-hand sides than
one pass takes, single-problem solves of such batches, and the fixed-size work
buffers at sizes where the problems run in parts.  Each right-hand side's
result is bitwise that of the same vector in another batch; one of them is
checked against the CPU FP64 oracle (bounds of the other parity tests on rough
fields: FP64 1e-11, FP32 4e-5)."""
import math

import numpy as np
import pytest
import torch

import workloads
from oracle.operator import Problem
from oracle.sweep import Preconditioner

pytestmark = pytest.mark.gpu
asp = pytest.importorskip("paper_1504_04058_amd.asp")

if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)


def setup(n, gamma, b, big):
    c = workloads.velocity_random(n, 2, seed=3, width=4.0)
    P = Problem(2, n, 2 * math.pi * (n + 1) / 8, gamma, 25.0, b, c)
    g = torch.Generator(device="cuda")
    g.manual_seed(n)
    return c, P, torch.randn(big, P.N, dtype=torch.complex128, device="cuda", generator=g)


@pytest.mark.parametrize("prec,tol", [(asp.ASP_PREC_FP64, 1e-11), (asp.ASP_PREC_FP32, 4e-5)])
@pytest.mark.parametrize("n,gamma,b,big,parts", [(67, 5, 8, 35, (1, 2, 3, 5, 8, 9, 15, 16, 31, 33)),
                                                 (16, 4, 5, 4113, (1, 4095, 4096, 4097))])
def test_batches(n, gamma, b, big, parts, prec, tol):
    print(f"apply layout n={n} batch={big} prec={prec}", flush=True)
    c, P, r = setup(n, gamma, b, big)
    with asp.Plan(2, c, P.omega, n, b, gamma, C=P.C, prec=prec) as plan:
        plan.factor()
        wide = plan.apply(r)
        for k in parts:
            assert torch.equal(plan.apply(r[:k].contiguous()), wide[:k]), k
        xs, xe = plan.layers()[0][1]
        pts = n * (xe - xs + 1)
        for kind, size in ((0, pts), (1, n)):
            w = r[:, :size].contiguous()
            one = plan.subsolve(kind, 2, w[big - 1:].contiguous(), pts)
            assert torch.equal(plan.subsolve(kind, 2, w, pts).view(big, pts)[big - 1], one), kind
    ref = Preconditioner(P).apply(r[big - 1].cpu().numpy())
    e = float(np.linalg.norm(wide[big - 1].cpu().numpy() - ref) / np.linalg.norm(ref))
    print(f"apply layout n={n} batch={big} prec={prec}: rel err {e:.2e}", flush=True)
    assert e < tol


# work buffers of the whole batch past the fixed scratch: solved in parts
@pytest.mark.parametrize("n,gamma,b,big", [(105, 5, 8, 119), (133, 9, 20, 93)])
def test_noalloc_in_parts(n, gamma, b, big):
    print(f"noalloc in parts n={n} batch={big}", flush=True)
    c, P, r = setup(n, gamma, b, big)
    with asp.Plan(2, c, P.omega, n, b, gamma, C=P.C, prec=asp.ASP_PREC_FP64) as plan:
        plan.factor()
        z = torch.empty_like(r)
        plan.apply_noalloc(r, z)
        torch.cuda.synchronize()
        assert torch.equal(z, plan.apply(r))
