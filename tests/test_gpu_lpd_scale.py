"""The held-out density at the ends of the FP64 range: scaling X, Y and sigma by
a power of two shifts the density of every pair by a constant, down to squared
distances that are subnormal and up to those near overflow.  Coordinates are
small integers, so that subnormal squares are exact."""
import math

import numpy as np
import pytest

import oracle
from paper_1905_04582_amd import api

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("k", [-530, -518, -515, -512, -470, 400, 500, 505])
@pytest.mark.parametrize("draws", [1, 3])
def test_scaled_problem(k, draws):
    n = 48
    rng = np.random.default_rng(11)
    xs = rng.integers(0, 40, (draws, n, 1)).astype(np.float64)   # some coincide
    sig = np.array([4.0, 5.0, 3.5])[:draws]
    y = np.abs(xs[0][:, 0][:, None] - xs[0][:, 0][None, :]) + rng.integers(0, 8, (n, n)) * 0.5
    y = np.tril(y, -1) + np.tril(y, -1).T
    held = np.ones((n, n), np.uint8)
    ref, m = oracle.lpd(xs, sig, y, held)
    s = 2.0 ** k
    H = api.HeldOutPairs(y * s, held)
    H.add_draws(xs * s, sig * s)
    got = H.lpd().item()
    shift = m * k * math.log(2.0)
    print(f"k={k} draws={draws} lpd {got:.16g} expected {ref - shift:.16g}", flush=True)
    assert abs(got - (ref - shift)) <= 1e-12 * (abs(ref) + abs(shift))
