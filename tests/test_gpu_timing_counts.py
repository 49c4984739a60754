"""The bytes and launches that asp_timing_read reports for a 2D apply are those of
its kernels: vectors with the right-hand sides fastest in the factor precision
between the caller's complex128 ones, boundary rows in complex128, every factor
and map entry once.  Written out here from the layers; m = 1, 2 and more, both
sweeps, FP64 and FP32."""
import math

import pytest
import torch

import workloads

pytestmark = pytest.mark.gpu
asp = pytest.importorskip("paper_1504_04058_amd.asp")

if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

SOLVE_M, SOLVE_RL, SWEEP, COMBINE = 2, 3, 4, 5


def expected(n, nrhs, e, layers, subs, seq):
    """{class: (launches, bytes)}; e: bytes of a factor entry, subs (kind, lines of X, lines)."""
    m, z, N = len(layers), 16, n * n
    fac = lambda k: sum(n * L * L * e for kind, _, L in subs if kind in k)
    lines = lambda k: sum(x for kind, x, _ in subs if kind in k)
    out = {SOLVE_M: (3, fac("M") + nrhs * N * (z + e + 2 * e)),
           COMBINE: (1, nrhs * (n * lines("MRL") * e + N * z))}
    if m > 1:
        slots = -(-nrhs // 32) * 32
        rl = fac("RL") + nrhs * (n * (2 * m - 2) * z + n * lines("RL") * e)
        seed = 2 * nrhs * n * (e + z) + 2 * slots * n * e
        step = 2 * (N * e + nrhs * n * (3 * e + z))
        hand = 2 * nrhs * n * (2 * e + z)
        if seq:
            out[SWEEP] = (1 + 2 * (m - 1) + m - 2, seed + rl + (m - 2) * hand)
        else:
            out[SWEEP] = (m - 1, seed + (m - 2) * step)
            out[SOLVE_RL] = (2, rl)
    return out


@pytest.mark.parametrize("prec,e", [(asp.ASP_PREC_FP64, 16), (asp.ASP_PREC_FP32, 8)])
@pytest.mark.parametrize("n,gamma,b,nrhs,seq", [(31, 5, 4, 3, 0), (31, 5, 4, 3, 1), (40, 4, 5, 35, 0),
                                                (16, 4, 5, 2, 0), (20, 3, 16, 2, 0)])
def test_counts(n, gamma, b, nrhs, seq, prec, e):
    print(f"timing counts n={n} gamma={gamma} b={b} nrhs={nrhs} seq={seq} prec={prec}", flush=True)
    c = workloads.velocity_random(n, 2, seed=3, width=2.0)
    r = torch.randn(nrhs, n * n, dtype=torch.complex128, device="cuda")
    with asp.Plan(2, c, 2 * math.pi * (n + 1) / 8, n, b, gamma, prec=prec,
                  sweep2d=asp.ASP_SWEEP2D_SEQUENTIAL if seq else asp.ASP_SWEEP2D_MAPS) as plan:
        plan.factor()
        layers, subs = plan.layers()[:2]
        asp.asp_timing_enable(plan.handle, 1)
        plan.apply(r)
        got = {k: asp.asp_timing_read(plan.handle, k) for k in (SOLVE_M, SOLVE_RL, SWEEP, COMBINE)}
        asp.asp_timing_enable(plan.handle, 0)
    width = {p + 1: int(xe - xs + 1) for p, (xs, xe) in enumerate(layers)}
    subs = [("MRL"[s[0]], width[s[1]], int(s[3] - s[2] + 1)) for s in subs]
    want = expected(n, nrhs, e, layers, subs, seq)
    assert {k: (v[0], v[2]) for k, v in got.items() if v[0]} == want
