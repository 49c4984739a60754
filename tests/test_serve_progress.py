"""Serving under budgets that cannot hold every key's plan with its workspace: plans
whose requests wait for workspace memory never block each other for good (a fake
backend; a run that does not end within its time fails)."""
import threading
import time

import numpy as np
import pytest

from paper_1504_04058_amd.serve import Backend, Request, Server


class FakeBackend(Backend):
    """Plans of 1000 bytes, workspaces of `per` bytes per right-hand side."""

    def __init__(self, per, work=0):
        self.per, self.work = per, work
        self.lock, self.used, self.peak = threading.Lock(), 0, 0

    def _take(self, nbytes):
        with self.lock:
            self.used += nbytes
            self.peak = max(self.peak, self.used)

    def factor_bytes(self, req):
        return 1000

    def factor_work_bytes(self, req):
        return self.work

    def workspace_bytes(self, req, nrhs):
        return self.per * nrhs

    def create(self, req):
        self._take(1000 + self.work)
        time.sleep(0.02)
        self._take(-self.work)
        return req.key

    def solve(self, handle, f):
        k = f.shape[0]
        self._take(self.per * k)
        time.sleep(0.003)
        self._take(-self.per * k)
        return 2 * f, np.full(k, 3, np.int32), np.full(k, 1e-7), "ASP_OK"

    def destroy(self, handle):
        self._take(-1000)


def req(rid, arrival, tag, nrhs=1):
    return Request(rid, (2, 4, tag), arrival, 2, 4, 1.0, nrhs, np.ones((4, 4)), np.ones((nrhs, 16), complex))


def run(reqs, budget, per, workers, work=0, realtime=True):
    be = FakeBackend(per, work)
    srv = Server(be, budget_bytes=budget, max_rhs=8, workers=workers, realtime=realtime)
    out = []
    th = threading.Thread(target=lambda: out.append(srv.run(reqs)), daemon=True)
    th.start()
    th.join(20)
    assert out, "the server made no progress"
    res, summ = out[0]
    assert summ["completed"] == len(reqs) and summ["peak_bytes"] <= budget
    assert be.peak <= budget and be.used == 0
    return summ


# two plans alone nearly fill the budget: neither could run next to the other
@pytest.mark.parametrize("workers", [2, 3])
def test_created_together(workers):
    run([req(0, 0.0, 0), req(1, 0.001, 1)], 2500, 600, workers)


# later requests need more than the first ones did, while both keys have some queued
def test_later_requests_larger():
    reqs = [req(i, 0.0, i % 2, 1 if i < 2 else 6) for i in range(12)]
    run(reqs, 2700, 250, 3, realtime=False)


# a factorization's work buffers count while it runs, the first workspace after it
def test_factorization_work():
    run([req(i, 0.001 * i, i % 3) for i in range(12)], 2400, 300, 3, work=900)


def test_many_keys():
    rng = np.random.default_rng(3)
    reqs = [req(i, 0.001 * i, int(rng.integers(6)), int(rng.integers(1, 5))) for i in range(80)]
    run(reqs, 3300, 300, 4)
