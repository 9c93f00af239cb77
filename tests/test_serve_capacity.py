"""Requests whose queries have more candidates than their call's memory holds:
the server submits them again with the room that the failure named, ends what
never fits as failed, and serves every other request (CPU stand-in backend)."""
import numpy as np
import pytest

import oracle.brute as ob
from paper_2311_02573_amd import serve, synth
from test_serve_scheduler import FakeBackend, FakeWorkspace


class NoRoom(RuntimeError):
    def __init__(self, needed):
        super().__init__(f"{needed} candidates")
        self.needed_pairs = needed


class SmallWorkspace(FakeWorkspace):
    def submit(self, q, rho, pool, offset, nbytes, pairs):
        super().submit(q, rho, pool, offset, nbytes, pairs)
        self.pairs = pairs

    def finish(self):
        nq = len(self.pending[0])
        res = super().finish().to_lists()
        assert len(res) == nq
        worst = max(len(i) for i, _ in res)
        if worst > self.pairs:
            raise NoRoom(worst)
        return type("R", (), {"to_lists": lambda s: res})()


class SmallBackend(FakeBackend):
    def slot(self, max_queries):
        return SmallWorkspace(self, max_queries)


def _server(feats, budget=1 << 20, streams=2):
    est = serve.Estimator(entries_per_tile=10.0, pairs_per_query=1.0)
    est.pairs = lambda nq: 4 * nq + 8  # (the stand-in's calls are small)
    b = SmallBackend(feats)
    return serve.Server(b, budget, streams=streams, max_queries=64, estimator=est), b


def _requests(w, sizes, rho):
    reqs, at = [], 0
    for i, k in enumerate(sizes):
        r = np.full(k, 0.99)
        if i in rho:
            r[:] = rho[i]
        reqs.append(serve.Request(i, w.queries[at:at + k], r, arrival=0.0))
        at += k
    return reqs


def test_requests_without_room_run_again():
    w = synth.workload_small(400, 32, 40)
    srv, b = _server(w.feats)
    reqs = _requests(w, [1, 5, 1, 20, 3], {0: 0.0, 3: -1.0})  # every row matches
    for r in reqs:
        srv.submit(r)
    srv.drain(30.0)
    assert all(r.status == "done" for r in reqs)
    assert srv.summary()["retried_calls"] >= 1 and srv.arena.used == 0
    for r in reqs:
        for (gi, _), (oi, _) in zip(r.results, ob.range_search(w.feats, r.queries, r.rho)):
            np.testing.assert_array_equal(gi, oi)


def test_a_request_that_never_fits_ends_alone():
    w = synth.workload_small(400, 32, 12)
    # room for ordinary calls, not for the 400 candidates of one query
    srv, b = _server(w.feats, budget=4096 + 64 * 10 + 36 * 60 + 24 * 100 + 2048)
    reqs = _requests(w, [2, 1, 2, 3], {1: 0.0})
    for r in reqs:
        srv.submit(r)
    srv.drain(30.0)
    assert [r.status for r in reqs] == ["done", "failed", "done", "done"]
    assert "candidates" in reqs[1].error and reqs[1].results is None
    s = serve.latency_summary(reqs)
    assert s["requests"] == 3 and s["failed"] == 1
    assert srv.idle and srv.arena.used == 0 and len(srv.free) == 2


def test_cancelled_and_timed_requests_on_the_way():
    w = synth.workload_small(400, 32, 12)
    srv, b = _server(w.feats, streams=1)
    t = [0.0]
    srv.clock, srv.t0 = (lambda: t[0]), 0.0
    reqs = _requests(w, [1, 2], {0: 0.0})
    reqs[1].timeout_s = 1.0
    for r in reqs:
        srv.submit(r)
    srv.step()
    assert [r.status for r in reqs] == ["running", "running"]
    srv.cancel(reqs[0])
    t[0] = 5.0  # past the timeout, but it was admitted before
    for _ in range(20):
        srv.step()
    assert [r.status for r in reqs] == ["cancelled", "done"]


def test_other_errors_still_end_the_run():
    w = synth.workload_small(50, 16, 2)
    srv, b = _server(w.feats)

    def broken():
        raise RuntimeError("device")

    for ws in srv.free:
        ws.finish = broken
    srv.submit(_requests(w, [2], {})[0])
    with pytest.raises(RuntimeError, match="device"):
        srv.drain(5.0)
