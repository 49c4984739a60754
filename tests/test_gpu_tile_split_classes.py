"""FP32 2D applies on both sides of the line where the R and L launches, counted
by their own problems, change the wavefronts per 16-row tile (128 and 130 layers
of one line), and sequential sweeps of more layers than that line.  Apply
against the CPU FP64 oracle (4e-5, the bound of the other parity tests on rough
fields), one vector bitwise as in a batch."""
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


@pytest.mark.parametrize("n,gamma,seq", [(134, 4, 0), (136, 4, 0), (134, 4, 1), (264, 4, 1), (262, 10, 1)])
def test_tile_split_classes(n, gamma, seq):
    print(f"tile split classes n={n} gamma={gamma} seq={seq}", flush=True)
    c = workloads.velocity_random(n, 2, seed=8, width=4.0)
    P = Problem(2, n, 2 * math.pi * (n + 1) / 8, gamma, 25.0, 1, c)
    rng = np.random.default_rng(n)
    r = rng.standard_normal((17, P.N)) + 1j * rng.standard_normal((17, P.N))
    with asp.Plan(2, c, P.omega, n, 1, gamma, C=P.C, prec=asp.ASP_PREC_FP32,
                  sweep2d=asp.ASP_SWEEP2D_SEQUENTIAL if seq else asp.ASP_SWEEP2D_MAPS) as plan:
        plan.factor()
        z = plan.apply(torch.from_numpy(r).cuda()).cpu().numpy()
        one = plan.apply(torch.from_numpy(r[16:].copy()).cuda()).cpu().numpy()
    assert np.array_equal(one[0], z[16])
    ref = Preconditioner(P).apply(r[16])
    e = float(np.linalg.norm(z[16] - ref) / np.linalg.norm(ref))
    print(f"tile split classes n={n} gamma={gamma} seq={seq}: rel err {e:.2e}", flush=True)
    assert e < 4e-5


# (n, b, gamma): sizes around the lines of the map chains' rule (products of 16 x 16
# tiles: 3584, 5680, 8736; 32 rows 8192 and 8448; 64 rows), FP64 1e-11
@pytest.mark.parametrize("prec,tol", [(asp.ASP_PREC_FP64, 1e-11), (asp.ASP_PREC_FP32, 4e-5)])
@pytest.mark.parametrize("n,b,gamma", [(120, 1, 4), (150, 1, 4), (190, 1, 4), (100, 1, 18), (102, 1, 18), (99, 24, 13)])
def test_map_split(n, b, gamma, prec, tol):
    print(f"map split n={n} b={b} gamma={gamma} prec={prec}", flush=True)
    c = workloads.velocity_random(n, 2, seed=9, width=4.0)
    P = Problem(2, n, 2 * math.pi * (n + 1) / 8, gamma, 25.0, b, c)
    rng = np.random.default_rng(n)
    r = rng.standard_normal((1, P.N)) + 1j * rng.standard_normal((1, P.N))
    with asp.Plan(2, c, P.omega, n, b, gamma, C=P.C, prec=prec) as plan:
        plan.factor()
        z = plan.apply(torch.from_numpy(r).cuda()).cpu().numpy()[0]
    ref = Preconditioner(P).apply(r[0])
    e = float(np.linalg.norm(z - ref) / np.linalg.norm(ref))
    print(f"map split n={n} b={b} gamma={gamma} prec={prec}: rel err {e:.2e}", flush=True)
    assert e < tol
