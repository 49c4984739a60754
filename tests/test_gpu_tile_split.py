"""2D layer solves on both sides of the rule that gives a 16-row tile one or more
wavefronts (FP32: several up to 256, 128 and 64 layers for problems of 16, 32 and
64 rows), with problems at the ends of the sweep that leave whole four-column
steps of a tile unused.  Apply in FP32 against the CPU FP64 oracle (4e-5, the
bound of the other parity tests on rough fields), one vector bitwise as in a
batch."""
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


# (n, gamma): layers of one line, rows 2 gamma - 1 (M) and gamma (R/L)
@pytest.mark.parametrize("n,gamma", [(96, 17), (97, 17), (144, 9), (145, 9), (161, 17), (262, 4), (263, 4)])
def test_tile_split(n, gamma):
    print(f"tile split n={n} gamma={gamma}", flush=True)
    c = workloads.velocity_random(n, 2, seed=8, width=4.0)
    P = Problem(2, n, 2 * math.pi * (n + 1) / 8, gamma, 25.0, 1, c)
    rng = np.random.default_rng(n)
    r = rng.standard_normal((17, P.N)) + 1j * rng.standard_normal((17, P.N))
    with asp.Plan(2, c, P.omega, n, 1, gamma, C=P.C, prec=asp.ASP_PREC_FP32) as plan:
        plan.factor()
        z = plan.apply(torch.from_numpy(r).cuda()).cpu().numpy()
        one = plan.apply(torch.from_numpy(r[16:].copy()).cuda()).cpu().numpy()
    assert np.array_equal(one[0], z[16])
    ref = Preconditioner(P).apply(r[16])
    e = float(np.linalg.norm(z[16] - ref) / np.linalg.norm(ref))
    print(f"tile split n={n} gamma={gamma}: rel err {e:.2e}", flush=True)
    assert e < 4e-5
