"""Pools of every format bit for bit against a CPU construction, at the sizes
where the tree kernels change over: the single-workgroup path (at most 64
pools in a level), one and two launches of four levels, ragged last pools,
rows that are not four features aligned; for builds and for inserts whose
ranges start and end at odd rows, below and above those limits."""
import numpy as np
import pytest
import torch

from oracle import formats

pytestmark = pytest.mark.gpu

E4M3 = np.asarray(formats.e4m3_nonneg_values()[0], dtype=np.float64)


def _add_up(a, b):
    # s - (larger term) is exact in float64, so the comparison with the smaller
    # one is that of the real numbers
    s = (a + b).astype(np.float32)
    above = s.astype(np.float64) - np.maximum(a, b).astype(np.float64)
    return np.where(above < np.minimum(a, b), np.nextafter(s, np.float32(np.inf)), s)


def _bf16_up(x):
    u = x.view(np.uint32).copy()
    u[(u != 0) & (u < 0x00800000)] = 0x00800000
    return ((u >> 16) + ((u & 0xFFFF) != 0)).astype(np.uint16)


def _tree(rows, capacity, op):
    level = np.zeros((capacity, rows.shape[1]), np.float32)
    level[: len(rows)] = rows
    out = [level]
    while len(out[0]) > 1:
        out.insert(0, op(out[0][0::2], out[0][1::2]))
    return out


def _rows(n, d, seed):
    g = np.random.default_rng(seed)
    # magnitudes over many binades, exact zeros, and float32 subnormals
    x = g.random((n, d), dtype=np.float32) * np.exp2(g.integers(-30, 3, (n, d))).astype(np.float32)
    x[g.random((n, d)) < 0.1] = 0.0
    x[g.random((n, d)) < 0.01] = np.float32(1e-41)
    return x


def _check(idx, rows, capacity, d):
    st = idx.stats()
    sums = _tree(rows, capacity, _add_up)
    maxs = _tree(rows, capacity, np.maximum)
    for l in range(st["depth"]):
        for pool, want in (("f32", sums[l]), ("max_f32", maxs[l])):
            got = idx.read_pools(l, pool=pool)
            assert np.array_equal(got[:, :d].view(np.uint32), want.view(np.uint32)), (pool, l)
            assert not got[:, d:].any()
        assert np.array_equal(idx.read_pools(l, pool="bf16")[:, :d], _bf16_up(sums[l])), l
        assert np.array_equal(idx.read_pools(l, pool="max_bf16")[:, :d], _bf16_up(maxs[l])), l
        scaled = np.ldexp(sums[l].astype(np.float64), -st["fp8_exp"][l])
        codes = np.searchsorted(E4M3, scaled, side="left")
        assert np.array_equal(idx.read_pools(l, pool="fp8")[:, :d], codes.astype(np.uint8)), l
    norms = np.sqrt((rows.astype(np.float64) ** 2).sum(axis=1))
    live = norms[norms > 0]
    assert st["m_min"] == pytest.approx(live.min() if len(live) else np.inf, rel=1e-14)


ALL = ("f32", "bf16", "fp8", "max_f32", "max_bf16")


@pytest.mark.parametrize("n,d", [(1, 3), (2, 128), (127, 20), (128, 4), (129, 130), (1000, 33),
                                 (2049, 8), (9001, 6), (33000, 4)])
def test_build(n, d):
    from paper_2311_02573_amd import gt

    rows = _rows(n, d, n)
    idx = gt.GTIndex(torch.from_numpy(rows).cuda(), pools=ALL)
    _check(idx, rows, idx.stats()["capacity"], d)
    idx.close()


@pytest.mark.parametrize("n0,groups", [(0, (1, 2, 125)), (1, (126, 1, 129)), (1000, (100, 127, 128, 131)),
                                       (4095, (1, 4097)), (10, (9000, 3))])
def test_insert(n0, groups):
    from paper_2311_02573_amd import gt

    d, capacity = 10, 1 << 14
    rows = _rows(n0 + sum(groups), d, 5 + n0)
    dev = torch.from_numpy(rows).cuda()
    idx = gt.GTIndex(dev[:n0].reshape(n0, d), capacity=capacity, pools=ALL)
    at = n0
    for k in groups:
        assert idx.insert(dev[at:at + k]) == at
        at += k
    _check(idx, rows, capacity, d)
    idx.close()


def test_features_at_an_odd_address():
    """Rows of a multiple of four features that do not start on 16 bytes."""
    from paper_2311_02573_amd import gt

    rows = _rows(300, 64, 11)
    for dt in (torch.float32, torch.float16, torch.bfloat16):
        x = torch.from_numpy(np.minimum(rows, 4.0)).to(dt)
        flat = torch.empty(300 * 64 + 1, dtype=dt, device="cuda")
        flat[1:] = x.reshape(-1).cuda()
        idx = gt.GTIndex(flat[1:].view(300, 64), pools=("f32",))
        leaves = idx.read_pools(idx.stats()["depth"], count=300)
        assert np.array_equal(leaves[:, :64], x.float().numpy())
        idx.close()
