"""The exhaustive path at tiny positive thresholds, where a match rests on
elements far below their row's largest: ids equal to the float64 oracle's and
to the walk's, similarities within 1e-6."""
import numpy as np
import pytest
import torch

import oracle.brute as ob

pytestmark = pytest.mark.gpu


def _check(rows, q, rho):
    from paper_2311_02573_amd import gt

    idx = gt.GTIndex(torch.from_numpy(rows).cuda(), pools=("f32",))
    qd = torch.from_numpy(q).cuda()
    want = ob.range_search(rows, q, rho)
    assert sum(len(i) for i, _ in want) > 0
    for got in (idx.exhaustive(qd, rho).to_lists(), idx.query(qd, rho, pool="f32").to_lists()):
        for (gi, gs), (oi, os_) in zip(got, want):
            np.testing.assert_array_equal(gi, oi)
            assert len(gs) == 0 or np.max(np.abs(gs - os_)) <= 1e-6
    idx.close()


def test_match_on_a_vanishing_element():
    """q = (1, 2^-45, 0, ...) and f = e_1: a cosine of 2^-45."""
    rows = np.zeros((3, 40), np.float32)
    rows[0, 0] = rows[1, 1] = rows[2, 2] = 1.0
    q = np.zeros((1, 40), np.float32)
    q[0, 0], q[0, 1] = 1.0, 2.0 ** -45
    _check(rows, q, 1e-14)


@pytest.mark.parametrize("n,d,nq", [(300, 50, 20), (129, 300, 130), (1000, 1025, 5)])
@pytest.mark.parametrize("rho", [1e-12, 1e-9, 1e-7, 1e-5, 2e-5, 1e-4])
def test_sparse_rows_of_wide_range(n, d, nq, rho):
    g = np.random.default_rng(n)

    def draw(m):
        x = np.abs(g.standard_normal((m, d))) * np.exp2(-g.uniform(0, 45, (m, d)))
        x *= g.random((m, d)) < 0.3
        x[np.arange(m), g.integers(0, d, m)] = 1.0
        return x.astype(np.float32)

    # every third query's threshold is an ordinary one
    _check(draw(n), draw(nq), np.where(np.arange(nq) % 3 == 2, 0.5, rho))
