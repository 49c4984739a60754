"""GPU parity of the symmetric block Gauss-Jordan elimination (tiles on and
above the diagonal only, the rest mirrored by the last panel) where its panels
and tiles end: one panel, two (one look-ahead pair), three (a pair and a single
one), fronts whose separator fills or just passes a 64-row panel, fronts with
and without a boundary part, for nested dissection and the dense blocks.  The
apply against the CPU FP64 oracle; the bounds are those of the other 3D parity
tests (FP64 1e-11; FP32 3e-5 by nested dissection, 2e-4 by blocks; bf16 split
1e-4, by blocks 2e-4)."""
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

# (n, gamma, b): columns of L = b + 2 (gamma - 1) unknowns in M problems
CASES = [(4, 2, 1),     # one leaf (48 rows), no boundary
         (9, 2, 2),     # L = 4: separators of one panel; blocks of 36 rows
         (13, 3, 3),    # L = 7: root separator 91 rows, two panels
         (12, 4, 5),    # L = 11: root separator 132 rows, three panels
         (16, 4, 2)]    # L = 8: root separator of exactly two panels
TOL = {("nd", asp.ASP_PREC_FP64): 1e-11, ("blocks", asp.ASP_PREC_FP64): 1e-11,
       ("nd", asp.ASP_PREC_FP32): 3e-5, ("blocks", asp.ASP_PREC_FP32): 2e-4,
       ("nd", asp.ASP_PREC_BF16X3): 1e-4, ("blocks", asp.ASP_PREC_BF16X3): 2e-4}


@pytest.mark.parametrize("prec", [asp.ASP_PREC_FP64, asp.ASP_PREC_FP32, asp.ASP_PREC_BF16X3])
@pytest.mark.parametrize("fact", ["nd", "blocks"])
@pytest.mark.parametrize("n,gamma,b", CASES)
def test_symmetric_elimination(n, gamma, b, fact, prec):
    print(f"symmetric elimination n={n} gamma={gamma} b={b} {fact} prec={prec}", flush=True)
    c = workloads.velocity_random(n, 3, seed=5, width=2.0)
    P = Problem(3, n, 2 * math.pi * (n + 1) / 8, gamma, 25.0, b, c)
    M = Preconditioner(P)
    rng = np.random.default_rng(8)
    r = rng.standard_normal((2, P.N)) + 1j * rng.standard_normal((2, P.N))
    with asp.Plan(3, c, P.omega, n, b, gamma, C=P.C, prec=prec, nd3d=fact == "nd") as plan:
        plan.factor()
        z = plan.apply(torch.from_numpy(r).cuda()).cpu().numpy()
    for k in range(2):
        ref = M.apply(r[k])
        e = float(np.linalg.norm(z[k] - ref) / np.linalg.norm(ref))
        print(f"symmetric elimination n={n} {fact} prec={prec} rhs {k}: rel err {e:.2e}", flush=True)
        assert e < TOL[fact, prec]
