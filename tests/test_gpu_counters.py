"""Results and statistics where the shared counters are busiest: calls whose
queries accept every row (one, two, four, five and 65 queries: the shared
slots of few queries, and the single ones beyond the fourth query of a wave),
on the walk and the exhaustive path."""
import numpy as np
import pytest
import torch

from paper_2311_02573_amd import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nq", [1, 2, 4, 5, 65])
@pytest.mark.parametrize("n", [2, 63, 1000])
def test_every_row_accepted(nq, n):
    from paper_2311_02573_amd import gt

    w = synth.workload_small(n, 96, nq, seed_offset=7)
    idx = gt.GTIndex(torch.from_numpy(w.feats).cuda(), pools=("f32", "bf16"))
    q = torch.from_numpy(w.queries).cuda()
    for run in (lambda: idx.query(q, -1.0, pool="bf16"), lambda: idx.exhaustive(q, -1.0)):
        r = run()
        assert r.total == n * nq
        assert np.array_equal(r.offsets.cpu().numpy(), np.arange(nq + 1) * n)
        ids = r.ids[: r.total].cpu().numpy().reshape(nq, n)
        assert np.array_equal(ids, np.tile(np.arange(n), (nq, 1)))
        st = idx.stats()
        assert st["leaf_pairs"] == n * nq
        assert st["candidates"] == st["results"] == n * nq
        idx.query(q, 0.9, pool="bf16")  # counters start from zero on every call
    idx.close()
