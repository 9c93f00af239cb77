"""The sort of each query's results at its edges: segments on both sides of 512
(bins of the top 8 or 12 bits), of 4096 (held in registers or taken in windows)
and of 2^18 (windows or radix passes), ids spread and side by side, and one
query or many (whose segments share workgroups differently)."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def gt():
    if not torch.cuda.is_available():
        pytest.fail("no GPU visible")
    from paper_2311_02573_amd import gt as g

    return g


def _index(gt, n, d=8):
    """Rows along axis 0, and along axis 1 where a query's results shall not be."""
    g = torch.Generator(device="cuda").manual_seed(n)
    rows = torch.zeros(n, d, device="cuda")
    rows[:, 1] = 1.0
    return rows, g


CASES = [(n, count, nq) for n in (700, 5000, 70000, 600000) for nq in (1, 70)
         for count in (1, 511, 512, 513, 4095, 4096, 4097, 6200, 40000, 262144, 262145, 600000)
         if count <= (n if nq == 1 else min(n, 40000))]


@pytest.mark.parametrize("n,count,nq", CASES)
@pytest.mark.parametrize("spread", [True, False])
def test_segments(gt, n, count, nq, spread):
    rows, g = _index(gt, n)
    at = torch.randperm(n, device="cuda", generator=g)[:count] if spread else \
        (torch.arange(count, device="cuda") + (n - count) // 2)
    rows[at, 1] = 0.0
    rows[at, 0] = 1.0
    idx = gt.GTIndex(rows, pools=("f32",))
    q = torch.zeros(nq, 8, device="cuda")
    q[:, 1] = 1.0
    q[0] = 0.0
    q[0, 0] = 1.0
    if nq > 1:  # the others: the same query, or one without results
        q[1::2] = q[0]
        q[2::2] = torch.eye(8, device="cuda")[5]
    want = torch.sort(at).values
    r = idx.query(q, 0.9, pool="f32")
    o = r.offsets.cpu().numpy()
    assert o[1] == count and r.total == count * (1 + nq // 2)
    for i in range(nq):
        ids, sims = r.ids[o[i]:o[i + 1]], r.sims[o[i]:o[i + 1]]
        if i == 0 or i % 2 == 1:
            assert torch.equal(ids, want) and bool((sims == 1.0).all())
        else:
            assert ids.numel() == 0
    idx.close()
