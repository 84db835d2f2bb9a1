"""The FP64 sweep's truncation terms at the edges of their range: the product
of 1/Phi over the longest walk, pairs on both sides of the skip point in one
wavefront, distances from 0 to beyond it, and near pairs beside missing ones.
Tolerances are those of the parity tests."""
import numpy as np
import pytest

import oracle
from paper_1905_04582_amd import api
from tests.test_gpu_parity import check64, gpu_eval

pytestmark = pytest.mark.gpu


def _line(kind, n, rng):
    """(x, sigma, mask): N x 1 locations on a line."""
    mask = None
    if kind == "close":        # every Phi = 1/2 to 1e-3: G = 2^(rows of the walk)
        x, sigma = 1e-3 * rng.random(n), 1.0
    elif kind == "skip_point":  # two clusters 9 sigma apart, to a few ulp and to 1e-9
        sigma = 0.7
        x = np.where(np.arange(n) % 2 == 0, 0.0, 9.0 * sigma)
        x = x + np.where(np.arange(n) % 3 == 0, 1e-9, 1e-15) * rng.standard_normal(n)
    elif kind == "ramp":       # t from 0 to 12 in every wavefront
        x, sigma = rng.permutation(np.linspace(0.0, 12.0, n)), 1.0
    else:                      # "missing": near pairs beside missing ones
        x, sigma = 3.0 * rng.random(n), 0.5
        low = np.tril(rng.random((n, n)) < 0.5, -1)
        mask = (low | low.T).astype(np.uint8)
    return x[:, None].copy(), sigma, mask


@pytest.mark.parametrize("kind", ["close", "skip_point", "ramp", "missing"])
@pytest.mark.parametrize("n,tile", [(2, (0, 0)), (65, (8, 1)), (520, (256, 1)),
                                    (777, (64, api.tile_waves(1, 4)))])
def test_near_terms(kind, n, tile):
    rng = np.random.default_rng(n)
    x, sigma, mask = _line(kind, n, rng)
    y = np.abs(x - x.T) + 0.3 * sigma * np.abs(rng.standard_normal((n, n)))
    y = np.tril(y, -1)
    y = y + y.T
    ref = oracle.evaluate(x, y, sigma, mask)
    got, _ = gpu_eval(y, x, sigma, mask, tile=tile)
    check64(got, ref, f"{kind} n={n} tile={tile}")
