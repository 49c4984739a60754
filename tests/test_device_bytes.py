"""What a memory budget counts is the device memory of whole blocks, not the sizes
of the buffers in them (CPU: host-only plans, and a fake backend whose blocks are
larger than its sizes)."""
import ctypes
import math
import threading
import time

import numpy as np
import pytest

from paper_1504_04058_amd import asp
from paper_1504_04058_amd.serve import Backend, Request, Server

MIB = 1 << 20


def block(b):
    q = 512 if b < MIB else 2 * MIB
    return -(-max(b, 16) // q) * q


@pytest.mark.parametrize("prec,esz", [(asp.ASP_PREC_FP64, 16), (asp.ASP_PREC_FP32, 8)])
@pytest.mark.parametrize("n,gamma,b,nrhs,restart", [(16, 4, 5, 1, 1), (24, 10, 16, 2, 20), (63, 12, 4, 5, 20),
                                                    (255, 9, 8, 17, 40)])
def test_2d_blocks(n, gamma, b, nrhs, restart, prec, esz):
    with asp.Plan(2, np.ones((n, n)), 2 * math.pi * n / 8, n, b, gamma, prec=prec, host_only=True) as plan:
        layers, subs = plan.layers()
        fac, work, ws = asp.asp_device_bytes(plan.handle, nrhs, restart)
        est = asp.asp_workspace_estimate(plan.handle, nrhs, restart)
        info = plan.info()
    m, N, z = len(layers), n * n, 16
    rows = [16 if L <= 16 else 32 if L <= 32 else 64
            for L in (max([s[3] - s[2] + 1 for s in subs if (s[0] == 0) == is_m], default=1) for is_m in (True, False))]
    red = asp.lib()._Z16krylov_red_bytesxi
    red.restype, red.argtypes = ctypes.c_size_t, [ctypes.c_longlong, ctypes.c_int]
    small = asp.lib()._Z18krylov_small_bytesxi
    small.restype, small.argtypes = ctypes.c_double, [ctypes.c_longlong, ctypes.c_int]
    last = 0 if esz == 16 else 1           # FP64: the last basis vector lies in the apply's third
    sizes = [3 * nrhs * N * esz, max(2 * m - 2, 1) * nrhs * n * z, 4 * n * -(-nrhs // 32) * 32 * esz,
             max(m * rows[0], (2 * m - 2) * rows[1]) * -(-nrhs // 16) * 16 * n * esz,
             nrhs * N * z * (restart + last), nrhs * N * z * restart, nrhs * N * z,
             red(N, nrhs), int(small(N, nrhs)) - red(N, nrhs)]
    assert est == sum(sizes)
    assert ws == sum(block(s) for s in sizes) + block(4 * nrhs)
    assert work == 0 and info["factor_bytes"] <= fac < info["factor_bytes"] + 4 * MIB


def test_3d_and_arguments():
    for opt in (asp.ASP_FACT3D_ND, asp.ASP_FACT3D_BLOCKS, asp.ASP_FACT3D_RECURSIVE):
        with asp.Plan(3, np.ones((19,) * 3), 10.0, 19, 3, 5, prec=asp.ASP_PREC_FP32, fact3d=opt, host_only=True) as p:
            got = asp.asp_device_bytes(p.handle, 17, 20)
            info = p.info()
            size = (info["factor_bytes"], info["factor_work_bytes"], asp.asp_workspace_estimate(p.handle, 17, 20))
            for a, b, k in zip(got, size, (1, 4, 14)):     # at most k buffers
                assert b <= a <= b + 2 * k * MIB
            L = asp.lib()
            assert L.asp_device_bytes(p.handle, 1, 1, None, None, None) == 0
            assert L.asp_device_bytes(p.handle, 0, 1, None, None, None) != 0
            assert L.asp_device_bytes(p.handle, 1, 0, None, None, None) != 0
            assert L.asp_device_bytes(None, 1, 1, None, None, None) != 0


class Blocks(Backend):
    """Factors of 900 bytes in a block of 1000, workspaces of 100 per right-hand
    side in blocks of `step`."""

    def __init__(self, step):
        self.step, self.used, self.peak, self.lock = step, 0, 0, threading.Lock()

    def _take(self, b):
        with self.lock:
            self.used += b
            self.peak = max(self.peak, self.used)

    def factor_bytes(self, req):
        return 900

    def workspace_bytes(self, req, nrhs):
        return 100 * nrhs

    def device_bytes(self, req, nrhs):
        return 1000, 0, -(-100 * nrhs // self.step) * self.step

    def create(self, req):
        self._take(1000)
        return req

    def solve(self, req, f):
        b = self.device_bytes(req, f.shape[0])[2]
        self._take(b)
        time.sleep(0.003)
        self._take(-b)
        k = f.shape[0]
        return 2 * f, np.full(k, 3, np.int32), np.full(k, 1e-7), "ASP_OK"

    def destroy(self, req):
        self._take(-1000)


def serve(budget, step, keys, count, nrhs=1):
    be = Blocks(step)
    reqs = [Request(i, (2, 4, i % keys), 0.0, 2, 4, 1.0, nrhs, np.ones((4, 4)), np.ones((nrhs, 16), complex))
            for i in range(count)]
    srv, out = Server(be, budget_bytes=budget, max_rhs=4, workers=3, realtime=False), []
    th = threading.Thread(target=lambda: out.append(srv.run(reqs)), daemon=True)
    th.start()
    th.join(20)
    assert out, "the server made no progress"
    assert out[0][1]["peak_bytes"] <= budget
    return be, out[0][1]


# three plans of 900 and their workspaces by size (3000) would fit, by blocks not
def test_blocks_within_budget():
    be, summ = serve(3000, 400, 3, 12)
    assert summ["completed"] == 12 and be.peak <= 3000 and summ["evictions"] > 0


# a lone key whose sizes fit the budget exactly is still served, and one that
# passes it is still refused
@pytest.mark.parametrize("budget,ok", [(1000, True), (1100, True), (999, False)])
def test_sizes_decide_what_is_refused(budget, ok):
    _, summ = serve(budget, 400, 1, 3)
    assert summ["completed"] == (3 if ok else 0)
