"""2D applies with enough problems to fill the chip give bitwise the same result
every time (a block step's vectors pass between wavefronts through LDS: every
write has to be complete at the barrier)."""
import math

import pytest
import torch

import workloads
from oracle.operator import Problem

pytestmark = pytest.mark.gpu
asp = pytest.importorskip("paper_1504_04058_amd.asp")

if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)


@pytest.mark.parametrize("prec", [asp.ASP_PREC_FP64, asp.ASP_PREC_FP32, asp.ASP_PREC_BF16X3])
@pytest.mark.parametrize("n,gamma", [(200, 4), (262, 4), (145, 9), (161, 17)])
def test_repeat(n, gamma, prec):
    print(f"repeat n={n} gamma={gamma} prec={prec}", flush=True)
    c = workloads.velocity_random(n, 2, seed=8, width=4.0)
    P = Problem(2, n, 2 * math.pi * (n + 1) / 8, gamma, 25.0, 1, c)
    g = torch.Generator(device="cuda")
    g.manual_seed(n)
    r = torch.randn(17, P.N, dtype=torch.complex128, device="cuda", generator=g)
    with asp.Plan(2, c, P.omega, n, 1, gamma, C=P.C, prec=prec) as plan:
        plan.factor()
        z = plan.apply(r)
        for i in range(12):
            assert torch.equal(plan.apply(r), z), i
