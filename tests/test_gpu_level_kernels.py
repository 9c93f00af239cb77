"""Small calls with options that ask for steps of the level-by-level walk run
those steps: the launches that the options imply, and the oracle's results."""
import numpy as np
import pytest
import torch

import oracle.brute as ob
from paper_2311_02573_amd import synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def gt():
    if not torch.cuda.is_available():
        pytest.fail("no GPU visible")
    from paper_2311_02573_amd import gt as g

    return g


def _same(got, want):
    for (gi, gs), (oi, os_) in zip(got, want):
        np.testing.assert_array_equal(gi, oi)
        assert len(gs) == 0 or np.max(np.abs(gs - os_)) <= 1e-6


POOLS = ("f32", "bf16", "fp8", "max_f32", "max_bf16")


def _run(gt, d, options, pools, n=5000, nq=40):
    w = synth.workload_small(n, d, nq, temp=0.2, seed_offset=23)
    idx = gt.GTIndex(torch.from_numpy(w.feats).cuda(), pools=pools)
    q = torch.from_numpy(w.queries).cuda()
    want = ob.range_search(w.feats, w.queries, 0.9)
    for k, v in options.items():
        idx.set_option(k, v)
    out = {}
    for pool in pools:
        print(f"[case] d={d} {options} {pool}", flush=True)
        _same(idx.query(q, 0.9, pool=pool).to_lists(), want)
        out[pool] = idx.stats()
    idx.close()
    return out


@pytest.mark.parametrize("d", [300, 1300, 2400])
def test_dense_level(gt, d):
    """One dense launch at the given level, then one launch a level (rows of 1300
    bfloat16 and 2400 float8 columns: the kernels that pass windows)."""
    for pool, st in _run(gt, d, {"dense_last": 8}, POOLS).items():
        dense = "f32" not in pool
        assert st["dense_launches"] == dense
        first = 8 if dense else st["head_level"]
        assert st["frontier_launches"] == st["depth"] - 1 - first > 1


@pytest.mark.parametrize("d", [300, 1300])
def test_no_dense_level(gt, d):
    for st in _run(gt, d, {"dense_last": -1}, POOLS).values():
        assert st["dense_launches"] == 0
        assert st["frontier_launches"] == st["depth"] - 1 - st["head_level"] > 1


@pytest.mark.parametrize("ws", [0, 1, 2])
def test_subtraction_step(gt, ws):
    st = _run(gt, 300, {"walk_subtract": ws}, ("bf16",))["bf16"]
    assert st["dense_launches"] == 1 and st["frontier_launches"] > 1


def test_automatic_small_call_is_one_launch(gt):
    for st in _run(gt, 300, {}, POOLS).values():
        assert (st["dense_launches"], st["frontier_launches"]) == (0, 1)


@pytest.mark.parametrize("ws", [1, 2])
def test_subtraction_step_of_rows_inserted_behind_a_call(gt, ws):
    """Right children at or beyond a call's epoch, which an insert between its
    submit and its finish grows."""
    w = synth.workload_small(3000, 96, 70, seed_offset=3)
    F = torch.from_numpy(w.feats).cuda()
    q = torch.from_numpy(w.queries).cuda()
    idx = gt.GTIndex(F[:1111], capacity=4096, pools=("bf16",))
    idx.set_option("walk_subtract", ws)
    work = gt.Workspace(idx, 128)
    at = 1111
    for step in (1, 100, 1788):
        work.submit(q, 0.8)
        idx.insert(F[at:at + step])
        _same(work.finish().to_lists(), ob.range_search(w.feats[:at], w.queries, 0.8))
        at += step
    work.close()
    idx.close()
