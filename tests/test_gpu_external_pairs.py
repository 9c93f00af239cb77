"""A query whose candidates alone outgrow an external workspace's memory: the
call ends with their number, and gets through with that room (and the server
does so by itself)."""
import numpy as np
import pytest
import torch

import oracle.brute as ob
from paper_2311_02573_amd import serve, synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def gt():
    if not torch.cuda.is_available():
        pytest.fail("no GPU visible")
    from paper_2311_02573_amd import gt as g

    return g


def _index(gt, n, nq):
    w = synth.workload_small(n, 64, nq, seed_offset=5)
    return w, gt.GTIndex(torch.from_numpy(w.feats).cuda(), pools=("bf16", "f32")), \
        torch.from_numpy(w.queries).cuda()


@pytest.mark.parametrize("pool", ["bf16", "f32"])
def test_needed_pairs(gt, pool):
    w, idx, q = _index(gt, 30000, 3)
    rho = np.array([0.9, -1.0, 0.9])  # the second query keeps every row
    want = ob.range_search(w.feats, w.queries, rho)
    ws = gt.ExternalWorkspace(idx, 3)

    def call(pairs):
        _, least = gt.call_bytes(idx, 3, pool, 0, pairs)
        mem = torch.empty(least + 256, dtype=torch.uint8, device="cuda")
        ws.submit(q, rho, pool, mem.data_ptr() + -mem.data_ptr() % 256, least, pairs)
        return ws.finish().to_lists(), mem

    with pytest.raises(gt.GTError) as e:
        call(0)
    assert e.value.status == gt.GT_ERR_CAPACITY and e.value.needed_pairs == 30000
    got, _ = call(e.value.needed_pairs)
    for (gi, _), (oi, _) in zip(got, want):
        np.testing.assert_array_equal(gi, oi)
    ws.close()
    idx.close()


def test_server_submits_again(gt):
    w, idx, q = _index(gt, 30000, 60)
    est = serve.Estimator(entries_per_tile=512, pairs_per_query=1)
    # (float32 pools: a call gets hardly more than the least memory it accepts)
    srv = serve.Server(serve.GpuBackend(idx, pool="f32"), 64 << 20, streams=2, max_queries=32, pool="f32",
                       estimator=est)
    reqs = [serve.Request(i, q[i:i + 1 + i % 3], np.full(1 + i % 3, -1.0 if i % 7 == 3 else 0.9), 0.0)
            for i in range(50)]
    for r in reqs:
        srv.submit(r)
    srv.drain(60.0)
    assert all(r.status == "done" for r in reqs)
    assert srv.summary()["retried_calls"] >= 1
    for r in reqs:
        for (gi, _), (oi, _) in zip(r.results, ob.range_search(w.feats, r.queries.cpu().numpy(), r.rho)):
            np.testing.assert_array_equal(gi, oi)
    idx.close()
