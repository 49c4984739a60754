"""Serving: requests of one key that arrive within the join window share a
solve while another key occupies the device, and a request on an idle device is
not held back (a fake backend; the scheduler's decisions only)."""
import time

import numpy as np

from paper_1504_04058_amd import serve
from paper_1504_04058_amd.serve import Backend, Request, Server


class FakeBackend(Backend):
    """Key 1 solves for 60 ms, the others for 1 ms."""

    def factor_bytes(self, req):
        return 1000

    def workspace_bytes(self, req, nrhs):
        return 10 * nrhs

    def create(self, req):
        return req.key

    def solve(self, handle, f):
        time.sleep(0.06 if handle[2] == 1 else 0.001)
        k = f.shape[0]
        return 2 * f, np.full(k, 3, np.int32), np.full(k, 1e-7), "ASP_OK"

    def destroy(self, handle):
        pass


def req(rid, arrival, tag):
    return Request(rid, (2, 4, tag), arrival, 2, 4, 1.0, 1, np.ones((4, 4)), np.ones((1, 16), complex))


def test_join_while_device_busy(monkeypatch):
    monkeypatch.setattr(serve, "JOIN_S", 0.02)
    reqs = [req(0, 0.0, 0), req(1, 0.010, 1), req(2, 0.020, 0), req(3, 0.028, 0), req(4, 0.2, 2)]
    srv = Server(FakeBackend(), budget_bytes=10 ** 6, workers=3)
    res, summ = srv.run(reqs)
    assert summ["completed"] == 5
    assert [ids for _, ids in srv.batches if 2 in ids] == [[2, 3]]


def test_no_hold_on_idle_device(monkeypatch):
    monkeypatch.setattr(serve, "JOIN_S", 0.5)
    reqs = [req(0, 0.0, 0), req(1, 0.05, 0), req(2, 0.1, 0)]
    res, summ = Server(FakeBackend(), budget_bytes=10 ** 6, workers=2).run(reqs)
    assert all(r.done - r.arrival < 0.3 for r in res)
