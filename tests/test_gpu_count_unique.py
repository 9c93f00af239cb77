"""Counting distinct rows leaves the call as it is: the same levels, launches and
tests as without, and every row that its walk reads."""
import numpy as np
import pytest
import torch

from paper_2311_02573_amd import synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def gt():
    if not torch.cuda.is_available():
        pytest.fail("no GPU visible")
    from paper_2311_02573_amd import gt as g

    return g


@pytest.mark.parametrize("pool", ("f32", "bf16", "fp8", "max_f32", "max_bf16"))
@pytest.mark.parametrize("n,nq,grid", [(6000, 30, 0), (6000, 300, 0), (6000, 300, 256), (5000, 20, 256)])
def test_counted_call_is_the_call(gt, pool, n, nq, grid):
    w = synth.workload_small(n, 100, nq, seed_offset=5)
    idx = gt.GTIndex(torch.from_numpy(w.feats).cuda(), pools=(pool,))
    idx.set_option("grid", grid)
    q = torch.from_numpy(w.queries).cuda()
    plain_r = idx.query(q, 0.9, pool=pool).to_lists()
    plain = idx.stats()
    idx.set_option("count_unique", 1)
    got_r = idx.query(q, 0.9, pool=pool).to_lists()
    got = idx.stats()
    idx.close()
    for (a, sa), (b, sb) in zip(plain_r, got_r):
        np.testing.assert_array_equal(a, b)
        np.testing.assert_array_equal(sa, sb)
    for key in ("head_level", "dense_launches", "frontier_launches", "pairs", "entries", "leaf_pairs"):
        assert got[key] == plain[key], key
    D, h, uniq = got["depth"], got["head_level"], got["unique_rows"]
    if got["dense_launches"] == 0:
        # (the level kernels' first launch tests every pool of its level, also
        # the ones past the rows)
        pop = -(-n // (1 << (D - h - 1)))
        assert pop <= uniq[h + 1] <= (1 << (h + 1)) and (grid or uniq[h + 1] == pop)
    one_tile = nq <= 32
    for l in range(h + 1, D - 1):
        # both children of each pool that some tile kept
        most = 2 * got["entries"][l]
        if got["dense_launches"] == 0 and one_tile:
            assert most - 1 <= uniq[l + 1] <= most
        assert 0 < uniq[l + 1] <= min(most, 1 << (l + 1))
    assert 0 < uniq[D] <= min(n, 2 * got["entries"][D - 1])
    assert all(u == 0 for u in uniq[:h + 1])
