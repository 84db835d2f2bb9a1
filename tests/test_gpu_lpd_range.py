"""The held-out density's short forms at the ends of their range: distances of
0, subnormal squares and infinity, pairs at the skip point of ln Phi, draws
whose densities lie hundreds of e-folds apart, more draws than a block holds
constants for.  Against the oracle, to the tolerance of the other density
tests (1e-12 of the sum)."""
import math

import numpy as np
import pytest

import oracle
from paper_1905_04582_amd import api

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d", [1, 2, 5])
@pytest.mark.parametrize("draws", [1, 2, 64, 65])
@pytest.mark.parametrize("diverged", [False, True])
def test_range(d, draws, diverged):
    n = 40
    rng = np.random.default_rng(10 * d + draws)
    x = rng.standard_normal((n, d))
    x[1] = x[0]                                  # delta = 0
    x[4] = 0.0
    x[5] = 0.0
    x[5, 0] = 1e-158                             # delta^2 subnormal
    x[6] = x[7]
    x[6, 0] += 9.0                               # t at the skip point where sigma = 1
    xs = np.stack([x] * draws)
    if diverged:
        xs[0, 8, 0] = np.inf                     # the first draw of a row's pairs: density 0
    sig = np.linspace(1.0, 0.02, draws)
    y = np.abs(rng.standard_normal((n, n)))
    y = np.tril(y, -1) + np.tril(y, -1).T
    held = np.ones((n, n), np.uint8)
    H = api.HeldOutPairs(y, held)
    H.add_draws(xs, sig)
    got = H.lpd().item()
    ref, m = oracle.lpd(xs, sig, y, held)
    assert H.m == m
    if math.isfinite(ref):
        assert abs(got - ref) <= 1e-12 * abs(ref)
    else:
        assert np.array_equal(got, ref, equal_nan=True)
