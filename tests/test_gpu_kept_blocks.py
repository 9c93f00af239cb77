"""Device memory that the library keeps between indexes: what an index reports,
and what the device has back."""
import time

import pytest
import torch

pytestmark = pytest.mark.gpu

@pytest.fixture(scope="module")
def gt():
    if not torch.cuda.is_available():
        pytest.fail("no GPU visible")
    from paper_2311_02573_amd import gt as g

    return g


def _index(gt, n, d):
    x = torch.rand(n, d, device="cuda")
    idx = gt.GTIndex(x, pools=("f32", "bf16"))
    idx.query(x[:100].contiguous(), 0.9999, pool="bf16")
    return idx


def _used(gt):
    """Device bytes in use once the library's idle blocks have left (two seconds,
    and an allocation)."""
    time.sleep(2.5)
    _index(gt, 100, 8).close()
    torch.cuda.synchronize()
    torch.cuda.empty_cache()
    free, total = torch.cuda.mem_get_info()
    return total - free


def test_reported_bytes_are_what_is_held(gt):
    base = _used(gt)
    _index(gt, 1 << 17, 1100).close()  # blocks an eighth larger than the next index's
    idx = _index(gt, 1 << 17, 1000)
    held, reported = _used(gt) - base, idx.stats()["bytes_device"]
    # (small allocations share pages, large ones end in a partly used one)
    assert abs(held - reported) <= 48 << 20, (held, reported)
    idx.close()
    assert _used(gt) <= base + (16 << 20)
