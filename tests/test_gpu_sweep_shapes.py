"""The sweep-step kernel's shapes (one or two tiles of right-hand sides per
block, four or eight wavefronts): a right-hand side's result is bitwise the
same in a batch that takes one tile and in one that takes two, at sizes on both
sides of the wavefront rule and with column counts that end inside a batch, and
agrees with the CPU FP64 oracle (FP64 1e-11; FP32 4e-5, the bound of the other
parity tests on rough fields; bf16 split 1e-4)."""
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


@pytest.mark.parametrize("prec,tol", [(asp.ASP_PREC_FP64, 1e-11), (asp.ASP_PREC_FP32, 4e-5),
                                      (asp.ASP_PREC_BF16X3, 1e-4)])
@pytest.mark.parametrize("n,big", [(65, 420), (129, 260), (192, 180), (193, 180), (209, 170)])
def test_sweep_shapes(n, big, prec, tol):
    print(f"sweep shapes n={n} batch={big} prec={prec}", flush=True)
    c = workloads.velocity_random(n, 2, seed=7, width=4.0)
    P = Problem(2, n, 2 * math.pi * (n + 1) / 8, 9, 25.0, 8, c)
    g = torch.Generator(device="cuda")
    g.manual_seed(n)
    r = torch.randn(big, P.N, dtype=torch.complex128, device="cuda", generator=g)
    with asp.Plan(2, c, P.omega, n, 8, 9, C=P.C, prec=prec) as plan:
        plan.factor()
        wide = plan.apply(r)                 # two tiles per block
        for k in (1, 17, 33):                # one
            assert torch.equal(plan.apply(r[:k].contiguous()), wide[:k]), k
    M = Preconditioner(P)
    for k in (0, big - 1):
        ref = M.apply(r[k].cpu().numpy())
        e = float(np.linalg.norm(wide[k].cpu().numpy() - ref) / np.linalg.norm(ref))
        print(f"sweep shapes n={n} prec={prec} rhs {k}: rel err {e:.2e}", flush=True)
        assert e < tol
