"""2D workspaces do not pass what two complex128 grid vectors, 2 restart + 2
Krylov vectors, the boundary rows, the transposed sweep lines and forward results
in groups of 1024 / LR right-hand sides take (the admission of a serving loop
counts with it), in any precision (CPU, host-only plans)."""
import ctypes
import math

import numpy as np
import pytest

from paper_1504_04058_amd import asp


def rows(L):
    return 16 if L <= 16 else 32 if L <= 32 else 64


def bound(n, nrhs, restart, esz, layers, subs):
    m, z, N = len(layers), 16, n * n
    ext = [max([s[3] - s[2] + 1 for s in subs if (s[0] == 0) == is_m], default=1) for is_m in (True, False)]
    LM, LRL = rows(ext[0]), rows(ext[1])
    groups = max(m * -(-nrhs // (1024 // LM)), max(2 * m - 2, 1) * -(-nrhs // (1024 // LRL)))
    small = asp.lib()._Z18krylov_small_bytesxi    # partial sums and small arrays of GMRES
    small.restype, small.argtypes = ctypes.c_double, [ctypes.c_longlong, ctypes.c_int]
    return (nrhs * N * z * (2 + 2 * restart + 2) + max(2 * m - 2, 1) * nrhs * n * z
            + 4 * n * -(-nrhs // 32) * 32 * esz + groups * n * 1024 * esz + small(N, nrhs))


@pytest.mark.parametrize("prec,esz", [(asp.ASP_PREC_FP64, 16), (asp.ASP_PREC_FP32, 8), (asp.ASP_PREC_BF16X3, 8)])
@pytest.mark.parametrize("n,gamma,b", [(16, 4, 5), (20, 3, 16), (63, 12, 4), (150, 2, 30), (255, 9, 8), (1023, 12, 4)])
def test_estimate(n, gamma, b, prec, esz):
    with asp.Plan(2, np.ones((n, n)), 2 * math.pi * (n + 1) / 8, n, b, gamma, prec=prec, host_only=True) as plan:
        layers, subs = plan.layers()
        for nrhs in (1, 15, 16, 17, 31, 32, 48, 64, 100, 128, 1000):
            for restart in (1, 20, 64):
                est = asp.asp_workspace_estimate(plan.handle, nrhs, restart)
                assert est <= bound(n, nrhs, restart, esz, layers.tolist(), subs.tolist()), (nrhs, restart)
