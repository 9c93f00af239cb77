"""Indexes built in memory that a destroyed index left behind: large blocks are
reused uncleared, so whatever an index relies on has to be written by its
build and its calls.  Two threads build and destroy at the same time."""
import threading

import numpy as np
import pytest
import torch

import oracle.brute as ob
from paper_2311_02573_amd import synth

pytestmark = pytest.mark.gpu

ALL = ("f32", "bf16", "fp8", "max_f32", "max_bf16")


def _dirty(n, d):
    """Fills blocks of an index's sizes with large values and frees them."""
    from paper_2311_02573_amd import gt

    full = torch.full((n, d), 0.7, device="cuda")
    idx = gt.GTIndex(full, pools=ALL)
    idx.query(full[:200].contiguous(), 0.99, pool="bf16", max_results=n * 200)
    idx.close()


def _use(seed, n, d, cap):
    from paper_2311_02573_amd import gt

    w = synth.workload_small(n, d, 70, seed_offset=seed)
    idx = gt.GTIndex(torch.from_numpy(w.feats[: n - 50]).cuda(), capacity=cap, pools=ALL)
    st = idx.stats()
    for l in range(st["depth"]):
        covered = ((n - 51) >> (st["depth"] - l)) + 1
        for pool in ALL:
            assert not idx.read_pools(l, covered, pool=pool).any()
    assert not idx.read_pools(st["depth"], n - 50).any()
    idx.insert(torch.from_numpy(w.feats[n - 50:]).cuda())
    want = ob.range_search(w.feats, w.queries, 0.9)
    for pool in ALL:
        got = idx.query(torch.from_numpy(w.queries).cuda(), 0.9, pool=pool).to_lists()
        assert all(np.array_equal(g[0], o[0]) for g, o in zip(got, want)), pool
    idx.close()


def test_build_in_reused_blocks():
    for k in range(3):
        _dirty(1 << 16, 128)
        _use(k, 40000, 128, 1 << 16)


def test_two_threads():
    errors = []

    def work(k):
        try:
            with torch.cuda.stream(torch.cuda.Stream()):
                for _ in range(3):
                    _dirty(1 << 16, 128)
                    _use(10 + k, 36000 + k, 128, 1 << 16)
        except Exception as e:  # reported by the main thread
            errors.append(e)

    ts = [threading.Thread(target=work, args=(k,)) for k in range(2)]
    for t in ts:
        t.start()
    for t in ts:
        t.join()
    assert not errors, errors
