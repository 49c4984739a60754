"""GPU parity of the twisted 2D layer factorization and its solves at the
sizes where the two halves, the 16-row tiles, the pivot pairs and the 16-wide
right-hand-side chunks end: even and odd n (halves of equal and unequal
length, one map-free plan), problems of odd and even line counts just below,
at and above a multiple of 16, mixed row counts of the M and R/L problems, and
batches of 1, 16 and 17.  Apply against the CPU FP64 oracle; the bounds are
those of the other parity tests for the same operators on rough fields (FP64
1e-11; FP32 4e-5; bf16 split 1e-4)."""
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

# (n, gamma, b): lines of an interior M problem b + 2 (gamma - 1), R/L b + gamma - 1
CASES = [(17, 2, 1),      # L = 3 and 2, one tile everywhere
         (16, 4, 9),      # m = 2, no maps; L = 15 / 12
         (31, 5, 8),      # L = 16 (a full tile) / 12, odd n
         (32, 5, 9),      # L = 17 (one line past a tile) / 13, even n
         (48, 9, 8),      # L = 24 / 16
         (65, 12, 8),     # L = 30 / 19 (two tiles both)
         (64, 12, 10),    # L = 32 (full) / 21
         (75, 12, 13),    # L = 35 / 24: 64-row and 32-row problems together
         (75, 17, 3)]     # L = 35 / 19
PRECS = [(asp.ASP_PREC_FP64, 1e-11), (asp.ASP_PREC_FP32, 4e-5), (asp.ASP_PREC_BF16X3, 1e-4)]


@pytest.mark.parametrize("prec,tol", PRECS)
@pytest.mark.parametrize("n,gamma,b", CASES)
def test_twisted_apply(n, gamma, b, prec, tol):
    print(f"twisted apply n={n} gamma={gamma} b={b} prec={prec}", flush=True)
    c = workloads.velocity_random(n, 2, seed=4, width=4.0)
    P = Problem(2, n, 2 * math.pi * (n + 1) / 8, gamma, 25.0, b, c)
    M = Preconditioner(P)
    rng = np.random.default_rng(6)
    r = rng.standard_normal((17, P.N)) + 1j * rng.standard_normal((17, P.N))
    with asp.Plan(2, c, P.omega, n, b, gamma, C=P.C, prec=prec) as plan:
        plan.factor()
        zs = {k: plan.apply(torch.from_numpy(r[:k].copy()).cuda()).cpu().numpy() for k in (1, 16, 17)}
    for k, z in zs.items():
        assert np.array_equal(z, zs[17][:k]), f"batch of {k} differs from the same vectors in 17"
    for k in (0, 15, 16):
        ref = M.apply(r[k])
        e = float(np.linalg.norm(zs[17][k] - ref) / np.linalg.norm(ref))
        print(f"twisted apply n={n} gamma={gamma} b={b} prec={prec} rhs {k}: rel err {e:.2e}", flush=True)
        assert e < tol
