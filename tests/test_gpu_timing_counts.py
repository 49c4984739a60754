"""What asp_timing_read reports.  3D factorizations: the work of an elimination
that keeps the symmetry.  2D applies: the bytes and launches of their kernels,
vectors with the right-hand sides fastest in the factor precision between the
caller's complex128 ones, boundary rows in complex128, every factor and map
entry once.  Written out here from the layers; m = 1, 2 and more, both sweeps,
FP64 and FP32."""
import math

import pytest
import torch

import workloads

pytestmark = pytest.mark.gpu
asp = pytest.importorskip("paper_1504_04058_amd.asp")

if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

FACTOR, SOLVE_M, SOLVE_RL, SWEEP, COMBINE = 0, 2, 3, 4, 5


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


def fronts(n, x0, x1, y0, y1):
    """(separator, boundary) columns of every node of the dissection of n x n columns
    (regions of at most 4 x 4 are leaves, others are cut at the middle of the longer side)."""
    w, h = x1 - x0 + 1, y1 - y0 + 1
    t = h * ((x0 > 0) + (x1 < n - 1)) + w * ((y0 > 0) + (y1 < n - 1))
    if w <= 4 and h <= 4:
        return [(w * h, t)]
    if w >= h:
        c = x0 + (w - 1) // 2
        parts, s = [(x0, c - 1, y0, y1), (c + 1, x1, y0, y1)], h
    else:
        c = y0 + (h - 1) // 2
        parts, s = [(x0, x1, y0, c - 1), (x0, x1, c + 1, y1)], w
    return [(s, t)] + [f for p in parts if p[0] <= p[1] and p[2] <= p[3] for f in fronts(n, *p)]


@pytest.mark.parametrize("n,gamma,b", [(9, 2, 2), (16, 4, 2)])
@pytest.mark.parametrize("nd", [True, False])
def test_factor_work_3d(n, gamma, b, nd):
    print(f"factor work n={n} gamma={gamma} b={b} nd={nd}", flush=True)
    c = workloads.velocity_random(n, 3, seed=3, width=2.0)
    with asp.Plan(3, c, 2 * math.pi * (n + 1) / 8, n, b, gamma, prec=asp.ASP_PREC_FP32, nd3d=nd) as plan:
        lines = [int(s[3] - s[2] + 1) for s in plan.layers()[1]]
        asp.asp_timing_enable(plan.handle, 1)
        plan.factor()
        flops = asp.asp_timing_read(plan.handle, FACTOR)[3]
        asp.asp_timing_enable(plan.handle, 0)
    if nd:
        want = sum(4 * ((s * L) ** 3 / 3 + (s * L) ** 2 * t * L + s * L * (t * L) ** 2)
                   for L in lines for s, t in fronts(n, 0, n - 1, 0, n - 1))
    else:
        want = sum(4 * n * (n * L) ** 3 for L in lines)
    assert abs(flops - want) <= 1e-9 * want
