"""Loss of the exhaustive path's split operands (x 2^e = hi + lo in float16, the
dropped lo.lo), against what the thresholds' slack leaves for it: for rows
>= 0 and scores of at least kSplitRho |q| |f|, half of the slack (K + 2) 2^-22
after the float32 accumulation's (K + 1) 2^-23."""
import os
import re

import numpy as np
import pytest

from paper_2311_02573_amd import build


def _split(x, e):
    y = np.ldexp(x.astype(np.float64), e)
    hi = y.astype(np.float16)
    lo = (y - hi.astype(np.float64)).astype(np.float16)
    return hi.astype(np.float64), lo.astype(np.float64)


def _split_score(q, f):
    """Sum of hi.hi + hi.lo + lo.hi in 64 bits, unscaled."""
    eq = 15 - np.frexp(q.max())[1]                              # q < 2^15 scaled
    norm = np.nextafter(np.float32(np.linalg.norm(f.astype(np.float64))), np.float32(0))
    ef = 14 - np.frexp(norm)[1]
    qh, ql = _split(q, eq)
    fh, fl = _split(f, ef)
    assert np.isfinite(qh).all() and np.isfinite(fh).all()
    return np.ldexp((qh * fh + qh * fl + ql * fh).sum(), -(eq + ef))


def _rho_line():
    src = open(os.path.join(build.CSRC, "gt_internal.h")).read()
    return float.fromhex(re.search(r"kSplitRho = (0x[0-9p.-]+);", src).group(1))


def _rows(rng, K, kind):
    x = np.abs(rng.standard_normal(K))
    if kind == "wide":       # elements over 2^60 of range
        x *= np.exp2(-rng.uniform(0, 60, K))
    elif kind == "spike":    # one large element, the score from tiny ones
        x *= np.exp2(-rng.uniform(15, 40, K))
        x[rng.integers(K)] = 1.0
    elif kind == "sparse":
        x *= rng.random(K) < 0.05
        x[rng.integers(K)] = 2.0 ** -rng.uniform(0, 30)
    return (x * np.exp2(rng.integers(-30, 30))).astype(np.float32)


@pytest.mark.parametrize("K", [128, 384, 1024, 4096])
def test_loss_is_covered_from_the_line_on(K):
    rng = np.random.default_rng(K)
    line, covered = _rho_line(), 0
    for i in range(400):
        kinds = ("plain", "wide", "spike", "sparse")
        q, f = _rows(rng, K, kinds[i % 4]), _rows(rng, K, kinds[i // 4 % 4])
        q64, f64 = q.astype(np.float64), f.astype(np.float64)
        exact = (q64 * f64).sum()
        scale = np.linalg.norm(q64) * np.linalg.norm(f64)
        loss = exact - _split_score(q, f)
        # the bound in the kernel's comment (the float64 sums here add 2^-40)
        assert abs(loss) <= 3 * 2.0 ** -22 * exact + np.sqrt(K) * 1.5 * 2.0 ** -38 * scale + 2.0 ** -40 * exact
        slack = (K + 2) * 2.0 ** -22 - (K + 1) * 2.0 ** -23
        if exact >= line * scale:
            covered += 1
            assert loss <= slack * exact
    assert covered > 20


def test_a_vanishing_element_is_lost_below_the_line():
    """Why there is a line: a score of 2^-45 that the split does not see."""
    q, f = np.zeros(128, np.float32), np.zeros(128, np.float32)
    q[0], q[1], f[1] = 1.0, 2.0 ** -45, 1.0
    assert _split_score(q, f) == 0.0


def test_the_line_follows_from_the_bound():
    for dp in range(128, 4097, 128):
        assert _rho_line() >= 3 * 2.0 ** -16 * np.sqrt(dp) / (dp - 6)
