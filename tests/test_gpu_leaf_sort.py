"""Leaf sweeps of 16 query tiles and more, whose entries are sorted by pool first,
against the oracle and against the same queries in calls of fewer tiles
(unsorted): few rows, part-filled trees, buckets of more pools than the sort
has bins, narrow and wide rows, float32 pools (32-query tiles), queries that
keep every row."""
import numpy as np
import pytest
import torch

import oracle.brute as ob
from paper_2311_02573_amd import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,d,cap,nq", [(50, 60, 64, 1030), (3000, 96, 4096, 1024),
                                        (20000, 600, 1 << 15, 1100), (5000, 40, 1 << 21, 1025),
                                        (2000, 1300, 2048, 2100)])
def test_sorted_sweep(n, d, cap, nq):
    from paper_2311_02573_amd import gt

    w = synth.workload_small(n, d, nq, seed_offset=n % 11)
    idx = gt.GTIndex(torch.from_numpy(w.feats).cuda(), capacity=cap, pools=("f32", "bf16", "fp8"))
    q = torch.from_numpy(w.queries).cuda()
    rho = np.full(nq, 0.9)
    rho[::300] = -1.0
    want = ob.range_search(w.feats, w.queries, rho)
    for pool in ("bf16", "fp8", "f32"):
        got = idx.query(q, rho, pool=pool).to_lists()
        few = idx.query(q[:500], rho[:500], pool=pool).to_lists()
        for k, ((gi, gs), (oi, os_)) in enumerate(zip(got, want)):
            assert np.array_equal(gi, oi), (pool, k)
            assert len(gs) == 0 or np.max(np.abs(gs - os_)) <= 1e-6
        for (gi, gs), (fi, fs) in zip(got, few):
            assert np.array_equal(gi, fi) and np.array_equal(gs, fs), pool
    idx.close()
