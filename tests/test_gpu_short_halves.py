"""2D layer solves whose halves are shorter than, as long as and longer than the
loads kept in flight (two or three block steps): n = 3 .. 9, FP64 and FP32.  Apply against the CPU FP64 oracle (the
bounds of the other parity tests on rough fields: FP64 1e-11, FP32 4e-5), and
each vector bitwise as in a batch."""
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


@pytest.mark.parametrize("prec,tol", [(asp.ASP_PREC_FP64, 1e-11), (asp.ASP_PREC_FP32, 4e-5)])
@pytest.mark.parametrize("n,gamma,b", [(3, 2, 1), (4, 2, 1), (5, 2, 2), (6, 3, 2), (7, 3, 2), (8, 3, 2), (9, 4, 3)])
def test_short_halves(n, gamma, b, prec, tol):
    print(f"short halves n={n} gamma={gamma} b={b} prec={prec}", flush=True)
    c = workloads.velocity_random(n, 2, seed=5, width=2.0)
    P = Problem(2, n, 2 * math.pi * (n + 1) / 8, gamma, 25.0, b, c)
    rng = np.random.default_rng(n)
    r = rng.standard_normal((3, P.N)) + 1j * rng.standard_normal((3, P.N))
    with asp.Plan(2, c, P.omega, n, b, gamma, C=P.C, prec=prec) as plan:
        plan.factor()
        z = plan.apply(torch.from_numpy(r).cuda()).cpu().numpy()
        one = plan.apply(torch.from_numpy(r[2:].copy()).cuda()).cpu().numpy()
    assert np.array_equal(one[0], z[2])
    ref = Preconditioner(P).apply(r[2])
    e = float(np.linalg.norm(z[2] - ref) / np.linalg.norm(ref))
    print(f"short halves n={n} gamma={gamma} b={b} prec={prec}: rel err {e:.2e}", flush=True)
    assert e < tol
