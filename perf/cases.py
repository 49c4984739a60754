"""The work a user has this library do, as timed cases.

Every case goes through paper_1504_04058_amd.asp.Plan, the way a program calls
it: a plan for one velocity field, then one of

* "factor_solve": a problem not seen before (a new frequency or velocity):
  factor the layers and solve a batch of right-hand sides with GMRES;
* "solve": the factors stay resident (a served problem) and a new batch of
  right-hand sides arrives;
* "apply": the preconditioner alone, for a program with a Krylov loop of its own;
* "matvec": the PML stencil alone, for such a program or a residual check.

Grids, PML widths, layers, batch sizes and restarts are those of the named
workloads, the paper's experiments and the served streams of this repository,
with odd and ragged sizes between them.  Full-precision solves stop at the
tolerances of those workloads (1e-6, and the paper's 1e-3); solves with FP32
factors or bf16-split products run to 1e-10, the tolerance at which the tests
hold mixed-precision solutions against full-precision ones.  A solve returns
the solutions; the iteration counts say how they were reached, not what they are.
"""
import math

import numpy as np
import torch

from paper_1504_04058_amd import asp

PREC = {"fp64": asp.ASP_PREC_FP64, "fp32": asp.ASP_PREC_FP32, "bf16x3": asp.ASP_PREC_BF16X3}
STRENGTH = 25.0     # PML constant C of every workload


def _case(name, call, dim, n, nrhs, prec, field, gamma=None, aux=0, b=4, tol=None, restart=20, sweep="maps"):
    """Defaults: 12 PML lines in 2D and 8 in 3D, layers of 4 lines, GMRES(20)."""
    gamma = gamma or (12 if dim == 2 else 8)
    tol = tol or (1e-6 if prec == "fp64" else 1e-10)
    c = dict(call=call, dim=dim, n=n, nrhs=nrhs, prec=prec, field=field, gamma=gamma, aux=aux, b=b,
             tol=tol, restart=restart, sweep=sweep)
    return dict(c, name=name) if name else c


def listed():
    return [
        # the smallest solve: one source on a small grid, factors resident
        _case("2d_n63_one_source", "solve", 2, 63, 1, "fp64", "constant"),
        # a few residuals of a caller's own Krylov loop, a size no tile divides
        _case("2d_n150_apply", "apply", 2, 150, 3, "fp64", "lens"),
        # the paper's 2D experiment (Section 3.2): two forces, thin layers of 8 lines, 1e-3
        _case("2d_n255_paper", "factor_solve", 2, 255, 2, "fp64", "waveguide", gamma=9, b=8, tol=1e-3, restart=40),
        # a new lens problem of ordinary size with mixed precision
        _case("2d_n511_lens", "factor_solve", 2, 511, 8, "fp32", "lens"),
        # the largest batch: random medium, 64 sources
        _case("2d_n1023_random", "factor_solve", 2, 1023, 64, "fp32", "random"),
        # a served problem in full precision, ragged last layer
        _case("2d_n700_served", "solve", 2, 700, 24, "fp64", "random"),
        # a served problem on the split bf16 products, ragged batch
        _case("2d_n383_split", "solve", 2, 383, 40, "bf16x3", "lens"),
        # Algorithm 2 as stated, for plans whose boundary maps would not fit or not pay
        _case("2d_n150_sequential", "factor_solve", 2, 150, 1, "fp32", "random", sweep="sequential"),
        # the 3D lens workload
        _case("3d_n63_lens", "factor_solve", 3, 63, 16, "fp32", "lens"),
        # the paper's 3D experiment (Section 4.2): thin auxiliary PML, two forces, 1e-3
        _case("3d_n39_paper", "factor_solve", 3, 39, 2, "fp64", "waveguide", gamma=9, aux=5, tol=1e-3, restart=40),
        # a served 3D problem with a small batch
        _case("3d_n31_served", "solve", 3, 31, 5, "fp32", "random"),
        # the stencil on a batch of large grid vectors
        _case("2d_n1023_matvec", "matvec", 2, 1023, 16, "fp64", "random"),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case of the same ranges, no larger than the largest listed one."""
    prec = rng.choice(["fp64", "fp32", "fp32", "bf16x3"])
    if rng.random() < 0.6:
        n = _log_int(rng, 48, 760)
        nrhs = min(_log_int(rng, 1, 64), max(1, 12_000_000 // (n * n)))
        field = rng.choice(["constant", "lens", "waveguide", "random"])
        call = rng.choice(["solve", "factor_solve", "factor_solve", "apply", "matvec"])
        if call in ("apply", "matvec"):
            return _case(None, call, 2, n, nrhs, "fp64", field)
        if rng.random() < 0.15 and n < 180:
            return _case(None, call, 2, n, min(nrhs, 8), prec, field, sweep="sequential")
        if rng.random() < 0.3:
            return _case(None, call, 2, n, nrhs, prec, field, gamma=9, b=8, restart=40,
                         tol=1e-3 if prec == "fp64" else None)
        return _case(None, call, 2, n, nrhs, prec, field)
    n = rng.randint(19, 47)
    nrhs = rng.randint(1, 16)
    field = rng.choice(["constant", "lens", "waveguide", "random"])
    call = rng.choice(["solve", "factor_solve", "factor_solve", "matvec"])
    if call == "matvec":
        return _case(None, call, 3, n, nrhs, "fp64", field)
    if rng.random() < 0.4:
        return _case(None, call, 3, n, nrhs, prec, field, gamma=9, aux=5, restart=40,
                     tol=1e-3 if prec == "fp64" else None)
    return _case(None, call, 3, n, nrhs, prec, field)


# -- inputs ----------------------------------------------------------------------

def _grid(case):
    t = np.arange(1, case["n"] + 1) / (case["n"] + 1)
    return np.meshgrid(*([t] * case["dim"]), indexing="ij")


def _omega(case):
    return 2 * math.pi * (case["n"] + 1) / 8      # eight points per wavelength


def _velocity(case, rng):
    """(n,)*dim velocities: the converging lens, the waveguide along the sweep
    axis, or Gaussian-smoothed noise mapped to [0.8, 1.2]."""
    n, dim, field = case["n"], case["dim"], case["field"]
    if field == "constant":
        return np.ones((n,) * dim)
    if field == "random":
        width = 8.0 if dim == 2 else (n + 1) / 16
        z = rng.standard_normal((n,) * dim)
        k2 = sum(np.meshgrid(*([np.fft.fftfreq(n) ** 2] * dim), indexing="ij"))
        z = np.fft.ifftn(np.fft.fftn(z) * np.exp(-2 * (math.pi * width) ** 2 * k2)).real
        return 0.8 + 0.4 * (z - z.min()) / (z.max() - z.min())
    x = _grid(case)
    cross = x if field == "lens" else x[:-1]
    r2 = sum((a - 0.5) ** 2 for a in cross)
    if field == "lens" and dim == 3:
        return 1.0 + 0.3 * np.exp(-32 * r2)
    return (4.0 / 3.0) * (1.0 - 0.5 * np.exp(-32 * r2))


def _forces(case, rng):
    """nrhs right-hand sides, column-major rows: Gaussian point sources at seeded
    points; the paper's settings take a wave packet as every second one."""
    n, dim, w = case["n"], case["dim"], _omega(case)
    t = np.arange(1, n + 1) / (n + 1)
    rows = []
    for k in range(case["nrhs"]):
        x0 = rng.uniform(0.2, 0.8, dim)
        packet = case["tol"] == 1e-3 and k % 2 == 1
        a = w / (2 * math.pi * math.sqrt(2)) if packet else 4 * w / math.pi
        d = rng.standard_normal(dim)
        d = w * d / np.linalg.norm(d) if packet else 0 * d
        f = np.ones(1)
        for j in range(dim):        # x1 fastest
            f = np.multiply.outer(np.exp(-(a * (t - x0[j])) ** 2 + 1j * d[j] * (t - x0[j])), f).reshape(-1)
        rows.append(f)
    return np.stack(rows)


def _inputs(case, seed):
    rng = np.random.default_rng(seed)
    c = _velocity(case, rng)
    if case["call"] in ("apply", "matvec"):
        shape = (case["nrhs"], case["n"] ** case["dim"])
        x = rng.standard_normal(shape) + 1j * rng.standard_normal(shape)
    else:
        x = _forces(case, rng)
    return c, x


def prepare(case, seed):
    c, x = _inputs(case, seed)
    plan = asp.Plan(case["dim"], c, _omega(case), case["n"], case["b"], case["gamma"], C=STRENGTH,
                    prec=PREC[case["prec"]], pml_aux=case["aux"],
                    sweep2d=asp.ASP_SWEEP2D_SEQUENTIAL if case["sweep"] == "sequential" else asp.ASP_SWEEP2D_MAPS)
    if case["call"] in ("solve", "apply"):
        plan.factor()
    return dict(plan=plan, x=torch.from_numpy(x).cuda(), call=case["call"], tol=case["tol"], restart=case["restart"])


def run(state):
    plan, x, call = state["plan"], state["x"], state["call"]
    if call == "apply":
        return plan.apply(x)
    if call == "matvec":
        return plan.matvec(x)
    if call == "factor_solve":
        plan.factor()
    u, _, _, _ = plan.gmres(x, tol=state["tol"], restart=state["restart"])
    return u


# -- what a pass cannot do without --------------------------------------------------

def _layers(case):
    """(first, last) sweep line of every layer."""
    n, g, b = case["n"], case["gamma"] - 1, case["b"]
    m = -(-(n - 2 * g) // b)
    starts = [1] + [g + 1 + b * p for p in range(1, m)]
    return [(s, e - 1) for s, e in zip(starts, starts[1:] + [n + 1])]


def _problems(case):
    """(kind, layer, first line, last line, zero region of the sweep-axis PML,
    PML widths below and above it) of every auxiliary problem."""
    n, gam = case["n"], case["gamma"]
    aux = case["aux"] or gam
    X = _layers(case)
    m = len(X)
    out = []
    for p, (s, e) in enumerate(X):
        phi, psi = max(s, gam), min(e, n + 1 - gam)
        lo, hi = (gam if p == 0 else aux), (gam if p == m - 1 else aux)
        out.append(("M", p, phi - (lo - 1), psi + hi - 1, phi, psi, lo, hi))
        if p > 0:
            out.append(("R", p, s, psi + hi - 1, s - 1, psi, hi, hi))
        if p < m - 1:
            out.append(("L", p, phi - (lo - 1), e, phi, e + 1, lo, lo))
    return out


def work(case):
    """Each input read once, the solutions written once, resident factors read
    once; the products of the layer solves, of the stencil, and the eliminations,
    with the iterations such solves take."""
    n, dim, nrhs = case["n"], case["dim"], case["nrhs"]
    N = n ** dim
    esz = 16 if case["prec"] == "fp64" else 8
    io = 2.0 * 16 * N * nrhs + 8.0 * N
    if case["call"] == "matvec":
        return {"bytes": io, "flops": (40.0 if dim == 2 else 56.0) * N * nrhs}
    lines = [q[3] - q[2] + 1 for q in _problems(case)]
    if dim == 2:      # n blocks of L x L per problem
        entries = sum(n * L * L for L in lines)
        factor = sum(8.0 * n * L ** 3 for L in lines)
    else:             # nested dissection of n x n columns of L unknowns
        entries = sum(8.0 * n * n * L * L * math.log2(n) for L in lines)
        factor = sum(30.0 * (n * L) ** 3 for L in lines)
    its = {1e-3: 4, 1e-6: 7, 1e-10: 12}[case["tol"]] if dim == 2 else {1e-3: 3, 1e-6: 3, 1e-10: 6}[case["tol"]]
    solve = 2 * 8.0 * entries * nrhs
    if case["call"] == "apply":
        return {"bytes": io + entries * esz, "flops": solve}
    flops = its * (solve + 60.0 * N * nrhs) + (factor if case["call"] == "factor_solve" else 0.0)
    return {"bytes": io + entries * esz, "flops": flops}


# -- the same in 64 bits, by other means ----------------------------------------------

def _pml(case, lo, hi, phi, psi, g_lo, g_hi):
    """s on lines lo..hi and on the half lines around them."""
    n, w = case["n"], _omega(case)

    def s(t):
        t = np.asarray(t, dtype=np.float64)
        below, above = np.maximum(phi - t, 0.0) / g_lo, np.maximum(t - psi, 0.0) / g_hi
        sig = STRENGTH * (n + 1) * (below ** 2 / g_lo + above ** 2 / g_hi)
        return 1.0 / (1.0 + 1j * sig / w)

    return s(np.arange(lo, hi + 1)), s(np.arange(lo, hi + 2) - 0.5)


def _axis(case):
    n, g = case["n"], case["gamma"]
    return _pml(case, 1, n, g, n + 1 - g, g, g)


def _second(half, h):
    return (np.diag(-(half[:-1] + half[1:])) + np.diag(half[1:-1], 1) + np.diag(half[1:-1], -1)) / h ** 2


def _solve_blocks(D, E, rhs):
    """Block tridiagonal solve: D[k] dense, E[k] the diagonal coupling of k and k+1."""
    n = len(D)
    inv, y = [None] * n, [None] * n
    for k in range(n):
        S = D[k] if k == 0 else D[k] - (E[k - 1][:, None] * inv[k - 1]) * E[k - 1]
        inv[k] = np.linalg.inv(S)
        y[k] = inv[k] @ (rhs[k] if k == 0 else rhs[k] - E[k - 1][:, None] * y[k - 1])
    for k in range(n - 2, -1, -1):
        y[k] = y[k] - inv[k] @ (E[k][:, None] * y[k + 1])
    return y


def _exact_solution(case, c, f):
    """A u = f / prod s with the slowest axis as the block index."""
    n, dim = case["n"], case["dim"]
    h, S = 1.0 / (n + 1), n ** (dim - 1)
    si, sh = _axis(case)
    ksq = (_omega(case) ** 2 / c ** 2).reshape(S, n, order="F").T     # [line][rest]
    T = _second(sh, h)
    if dim == 2:
        cross, cs = T, si
    else:
        one = np.diag(1.0 / si)
        cross, cs = np.kron(one, T) + np.kron(T, one), np.kron(si, si)
    D = [cross / si[k] + np.diag(ksq[k] / (cs * si[k]) + T[k, k] / cs) for k in range(n)]
    E = [sh[k + 1] / h ** 2 / cs for k in range(n - 1)]
    b = f.reshape(len(f), n, S) / (si[:, None] * cs)
    u = _solve_blocks(D, E, [b[:, k].T for k in range(n)])
    return np.stack(u).transpose(2, 0, 1).reshape(len(f), -1)


def _exact_stencil(case, c, x):
    n, dim = case["n"], case["dim"]
    h = 1.0 / (n + 1)
    si, sh = _axis(case)
    x = x.reshape((len(x),) + (n,) * dim)                # slowest axis first
    prod = 1.0
    for a in range(dim):
        prod = np.multiply.outer(prod, si)
    y = (_omega(case) ** 2 / c ** 2).T / prod * x
    for a in range(dim):
        v = np.moveaxis(x, 1 + a, -1)
        d = np.diff(v, axis=-1, prepend=0, append=0) * sh / h ** 2
        y = y + np.moveaxis(np.diff(d, axis=-1) * si, -1, 1 + a) / prod
    return y.reshape(len(x), -1)


def _exact_apply(case, c, r):
    """Algorithm 2 with every auxiliary problem solved in blocks of its sweep lines."""
    n, nr = case["n"], len(r)
    h = 1.0 / (n + 1)
    si, sh = _axis(case)
    ksq = _omega(case) ** 2 / c ** 2
    X = _layers(case)
    probs = {(q[0], q[1]): q for q in _problems(case)}
    r = r.reshape(nr, n, n)

    def green(kind, p, data):
        """data: [nrhs, lines of the layer, n], or one boundary line [nrhs, n]."""
        _, _, lo, hi, phi, psi, g_lo, g_hi = probs[kind, p]
        zi, zh = _pml(case, lo, hi, phi, psi, g_lo, g_hi)
        L = hi - lo + 1
        T = _second(zh, h)
        D = [T / si[k] + np.diag(-(sh[k] + sh[k + 1]) / (h ** 2 * zi) + ksq[k, lo - 1:hi] / (si[k] * zi))
             for k in range(n)]
        E = [sh[k + 1] / (h ** 2 * zi) for k in range(n - 1)]
        g = np.zeros((n, L, nr), dtype=np.complex128)
        s, e = X[p]
        if kind == "M":
            g[:, s - lo:e - lo + 1] = data.transpose(2, 1, 0)
        else:
            edge = zh[0] if kind == "R" else zh[-1]
            g[:, 0 if kind == "R" else L - 1] = -(edge / h ** 2 / si)[:, None] * data.T
        v = np.stack(_solve_blocks(D, E, g))
        return v[:, s - lo:e - lo + 1].transpose(2, 1, 0)

    m = len(X)
    u = [green("M", p, r[:, s - 1:e]) for p, (s, e) in enumerate(X)]
    z = [a.copy() for a in u]
    line = u[0][:, -1]
    for p in range(1, m):
        a = green("R", p, line)
        z[p] += a
        line = a[:, -1] + u[p][:, -1]
    line = u[-1][:, 0]
    for p in range(m - 2, -1, -1):
        a = green("L", p, line)
        z[p] += a
        line = a[:, 0] + u[p][:, 0]
    return np.concatenate(z, axis=1).reshape(nr, -1)


def exact(case, seed):
    n, dim = case["n"], case["dim"]
    if case["call"] == "matvec":
        return _exact_stencil(case, *_inputs(case, seed))
    if case["call"] == "apply":
        return _exact_apply(case, *_inputs(case, seed)) if n <= 200 else None
    if 11.0 * n * n ** (3 * (dim - 1)) > 4e11:      # the elimination would take too long
        return None
    return _exact_solution(case, *_inputs(case, seed))
