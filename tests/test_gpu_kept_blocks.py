"""Device memory that the library keeps between indexes: what an index reports,
and what the device has back."""
import os
import subprocess
import sys
import time

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


def test_blocks_leave_by_themselves(gt):
    """A program that closes its index and goes on without the library."""
    base = _used(gt)
    _index(gt, 1 << 17, 1000).close()
    torch.cuda.empty_cache()
    free, total = torch.cuda.mem_get_info()
    assert total - free > base + (256 << 20)  # kept at first
    for _ in range(100):
        time.sleep(0.1)
        free, total = torch.cuda.mem_get_info()
        if total - free <= base + (16 << 20):
            break
    assert total - free <= base + (16 << 20)


def test_blocks_that_leave_during_a_stream_capture(gt):
    """Their frees disturb no capture of the program."""
    x = torch.arange(1 << 20, dtype=torch.float32, device="cuda")
    y = torch.zeros_like(x)
    s = torch.cuda.Stream()
    base = _used(gt)
    _index(gt, 1 << 17, 1000).close()
    s.wait_stream(torch.cuda.current_stream())
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=s):
        y.copy_(x)
        time.sleep(3.5)
        y.mul_(2.0).add_(1.0)
    torch.cuda.empty_cache()
    for k in range(3):
        x.fill_(float(k))
        graph.replay()
        torch.cuda.synchronize()
        np.testing.assert_array_equal(y.cpu().numpy(), np.full(1 << 20, 2.0 * k + 1.0, np.float32))
    free, total = torch.cuda.mem_get_info()
    assert total - free <= base + (64 << 20)  # (the graph and its memory)


def test_exit_with_idle_blocks():
    code = ("import torch\n"
            "from paper_2311_02573_amd import gt\n"
            "x = torch.rand(1 << 17, 256, device='cuda')\n"
            "i = gt.GTIndex(x)\n"
            "j = gt.GTIndex(x)\n"
            "i.close()\n"       # j is left to the interpreter's end
            "print('closed', flush=True)\n")
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    r = subprocess.run([sys.executable, "-c", code], cwd=root, capture_output=True, text=True, timeout=100)
    assert r.returncode == 0 and r.stdout == "closed\n", (r.returncode, r.stderr[-500:])
