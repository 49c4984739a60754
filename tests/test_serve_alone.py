"""Serving: after three waits in vain the requests of a key no longer wait for
company, until two of them arrive close together again; a server option sets the
wait or switches it off (a fake backend; the scheduler's decisions only)."""
import time

import numpy as np
import pytest

from paper_1504_04058_amd import serve
from paper_1504_04058_amd.serve import Backend, Request, Server


class FakeBackend(Backend):
    """Key 1 solves for 2.6 s, the others for 1 ms."""

    def factor_bytes(self, req):
        return 1000

    def workspace_bytes(self, req, nrhs):
        return 10 * nrhs

    def create(self, req):
        return req.key

    def solve(self, handle, f):
        time.sleep(2.6 if handle[2] == 1 else 0.001)
        k = f.shape[0]
        return 2 * f, np.full(k, 3, np.int32), np.full(k, 1e-7), "ASP_OK"

    def destroy(self, handle):
        pass


def req(rid, arrival, tag):
    return Request(rid, (2, 4, tag), arrival, 2, 4, 1.0, 1, np.ones((4, 4)), np.ones((1, 16), complex))


# key 0 is factored first; key 1 keeps the device busy from 0.1 s to 2.7 s; a last
# request keeps the stream open until after that
def stream(times):
    return [req(0, 0.0, 0), req(1, 0.1, 1)] + [req(2 + i, t, 0) for i, t in enumerate(times)] + \
        [req(2 + len(times), 2.9, 2)]


def waits(res):
    return [r.start - r.arrival for r in res]


def test_lone_requests_stop_waiting(monkeypatch):
    monkeypatch.setattr(serve, "JOIN_S", 0.15)
    res, summ = Server(FakeBackend(), budget_bytes=10 ** 6, workers=3).run(stream([0.3, 0.7, 1.1, 1.5, 1.9]))
    assert summ["completed"] == 8
    w = waits(res)[2:7]
    assert min(w[:3]) > 0.1 and max(w[3:]) < 0.08, w


def test_close_arrivals_wait_again(monkeypatch):
    monkeypatch.setattr(serve, "JOIN_VAIN", 1)
    srv = Server(FakeBackend(), budget_bytes=10 ** 6, workers=3, join_s=0.15)
    res, summ = srv.run(stream([0.3, 0.7, 0.75, 0.8, 1.3, 1.35]))
    assert summ["completed"] == 9
    # 2 waits in vain, 3 does not wait, 4 and 5 share, so do 6 and 7
    assert [ids for _, ids in srv.batches if set(ids) & {2, 3, 4, 5, 6, 7}] == [[2], [3], [4, 5], [6, 7]]


@pytest.mark.parametrize("join_s", [0.0, 0.15])
def test_option(join_s):
    srv = Server(FakeBackend(), budget_bytes=10 ** 6, workers=3, join_s=join_s)
    res, _ = srv.run(stream([0.4]))
    assert (waits(res)[2] > 0.1) == (join_s > 0)
