"""FP64 2D GMRES over whole cycles (the last basis vector of a cycle lies in the
apply's third vector): restart lengths 1 to 3 and one that is not reached, after
an apply of more right-hand sides, against the CPU FP64 oracle (iterations within
one, true residuals at the tolerance) and bitwise against a fresh plan; the plan's
workspaces are those of the estimate."""
import math

import numpy as np
import pytest
import torch

import workloads
from oracle.gmres import gmres as oracle_gmres
from oracle.operator import Problem
from oracle.sweep import Preconditioner

pytestmark = pytest.mark.gpu
asp = pytest.importorskip("paper_1504_04058_amd.asp")

if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)


@pytest.mark.parametrize("n,gamma,b,seq", [(31, 5, 4, 0), (40, 4, 5, 1), (20, 3, 16, 0)])
@pytest.mark.parametrize("restart", [1, 2, 3, 30])
def test_cycles(n, gamma, b, seq, restart):
    print(f"gmres cycles n={n} gamma={gamma} b={b} seq={seq} restart={restart}", flush=True)
    c = workloads.velocity_random(n, 2, seed=6, width=3.0)
    P = Problem(2, n, 2 * math.pi * (n + 1) / 8, gamma, 25.0, b, c)
    rng = np.random.default_rng(n)
    f = rng.standard_normal((3, P.N)) + 1j * rng.standard_normal((3, P.N))
    F = torch.from_numpy(f).cuda()
    big = torch.randn(20, P.N, dtype=torch.complex128, device="cuda")
    kw = dict(C=P.C, prec=asp.ASP_PREC_FP64,
              sweep2d=asp.ASP_SWEEP2D_SEQUENTIAL if seq else asp.ASP_SWEEP2D_MAPS)
    tol = 1e-9
    with asp.Plan(2, c, P.omega, n, b, gamma, **kw) as plan:
        u, it, rr, st = plan.gmres(F, tol=tol, restart=restart, maxit=400)
        assert plan.info()["workspace_bytes"] <= asp.asp_workspace_estimate(plan.handle, 3, restart)
    with asp.Plan(2, c, P.omega, n, b, gamma, **kw) as plan:
        plan.factor()
        z = plan.apply(big)
        u2, it2, rr2, _ = plan.gmres(F, tol=tol, restart=restart, maxit=400)
        assert torch.equal(plan.apply(big), z)
    assert torch.equal(u, u2) and np.array_equal(it, it2)
    assert st == asp.ASP_OK and np.all(rr <= tol)
    A, M, s = P.A(), Preconditioner(P), P.scale()
    for k in range(3):
        rhs = f[k] / s
        _, its, _, _ = oracle_gmres(lambda v: A @ v, M.apply, rhs, tol, restart, 400)
        assert abs(int(it[k]) - its) <= 1
        x = u[k].cpu().numpy()
        res = float(np.linalg.norm(rhs - A @ x) / np.linalg.norm(rhs))
        print(f"gmres cycles n={n} restart={restart} rhs {k}: {it[k]} iterations (oracle {its}), relres {res:.2e}", flush=True)
        assert res <= tol * (1 + 1e-6)
