"""Query preparation at its edges: the masks of live queries of a workgroup's
eight, of tiles of 32 and 64, calls on both sides of 256 thresholds, rows that
end inside a wave's columns, and queries that are refused."""
import numpy as np
import pytest
import torch

import oracle.brute as ob
from paper_2311_02573_amd import synth

pytestmark = pytest.mark.gpu
TOL = 1e-6  # the leaf similarity's bound


@pytest.fixture(scope="module")
def gt():
    if not torch.cuda.is_available():
        pytest.fail("no GPU visible")
    from paper_2311_02573_amd import gt as g

    return g


@pytest.mark.parametrize("d", [1, 63, 65, 258, 1000, 4096])
@pytest.mark.parametrize("nq", [1, 8, 9, 33, 64, 129, 256, 257])
def test_dead_queries_and_thresholds(gt, d, nq):
    w = synth.workload_small(300, d, nq, seed_offset=d % 7)
    q = w.queries.copy()
    q[3::8] = 0.0  # no direction: no result, whatever the threshold
    q[30:70:3] = 0.0
    rho = np.linspace(0.2, 0.95, nq)
    rho[::5] = -1.0
    want = ob.range_search(w.feats, q, rho)
    idx = gt.GTIndex(torch.from_numpy(w.feats).cuda(), pools=("f32", "bf16", "fp8"))
    for pool in ("f32", "bf16", "fp8"):
        got = idx.query(torch.from_numpy(q).cuda(), rho, pool=pool).to_lists()
        for (gi, gs), (oi, os_) in zip(got, want):
            assert np.array_equal(gi, oi)
            assert len(gs) == 0 or np.max(np.abs(gs - os_)) <= TOL


@pytest.mark.parametrize("at", [0, 7, 8, 63, 64, 299])
def test_refused_queries(gt, at):
    w = synth.workload_small(300, 96, 300)
    idx = gt.GTIndex(torch.from_numpy(w.feats).cuda(), pools=("f32", "bf16"))
    good = torch.from_numpy(w.queries).cuda()
    want = ob.range_search(w.feats, w.queries, 0.9)
    for value in (-1.0, float("nan"), float("inf")):
        bad = good.clone()
        bad[at, 95] = value
        for call in (lambda: idx.query(bad, 0.9, pool="bf16"), lambda: idx.query(bad, 0.9, pool="f32"),
                     lambda: idx.exhaustive(bad, 0.9)):
            with pytest.raises(gt.GTError):
                call()
        for (gi, gs), (oi, os_) in zip(idx.query(good, 0.9, pool="bf16").to_lists(), want):
            assert np.array_equal(gi, oi)
