"""Float32 pools walked by levels in an external workspace's memory, from the
least that a call accepts (a frontier much smaller than the first level) up:
results equal those of a call with its own buffers."""
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


@pytest.mark.parametrize("n,d,nq", [(60000, 64, 2048), (60000, 64, 65), (9000, 1300, 300), (9000, 600, 300)])
@pytest.mark.parametrize("pool", ["f32", "max_f32"])
def test_levels_from_the_least_memory(gt, n, d, nq, pool):
    w = synth.workload_small(n, d, nq, seed_offset=11)
    idx = gt.GTIndex(torch.from_numpy(w.feats).cuda(), pools=(pool,))
    q = torch.from_numpy(w.queries).cuda()
    want = idx.query(q, 0.9, pool=pool).to_lists()
    idx.set_option("grid", 256)  # the level kernels
    need, least = gt.call_bytes(idx, nq, pool, 1 << 16, 4096)
    ws = gt.ExternalWorkspace(idx, nq)
    # twice: the second call's first level follows the first's frontier
    for nbytes in (least, least, need, need):
        print(f"[case] {pool} n={n} d={d} nq={nq} bytes={nbytes}", flush=True)
        mem = torch.empty(nbytes + 256, dtype=torch.uint8, device="cuda")
        off = -mem.data_ptr() % 256
        ws.submit(q, 0.9, pool, mem.data_ptr() + off, nbytes, 4096)
        got = ws.finish().to_lists()
        for (gi, gs), (oi, os_) in zip(got, want):
            np.testing.assert_array_equal(gi, oi)
            np.testing.assert_array_equal(gs, os_)
    ws.close()
    idx.close()
