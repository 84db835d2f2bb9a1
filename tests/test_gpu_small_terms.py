"""The FP64 log-likelihood where it consists of small truncation terms alone:
sigma = 1 (M ln sigma = 0) and every observed y equal to its distance, so that
L = -sum ln Phi(t) with each term far below one.  The sum keeps relative
precision: L within the parity tests' 1e-12 of |L|, beside the squares of the
residuals that two roundings of a distance leave (at most 2 units each); the
gradient, which consists of those residuals and m here, by the rows' rounding
scale."""
import numpy as np
import pytest

import oracle
from paper_1905_04582_amd import api
from tests.test_gpu_parity import TOL64, gpu_eval

pytestmark = pytest.mark.gpu

U = 2.0 ** -53
TILES = [(0, 0), (8, 1), (64, api.tile_waves(1, 4)), (256, 1)]


def _check(x, mask, tile, label):
    y = np.abs(x[:, 0][:, None] - x[:, 0][None, :])
    ref = oracle.evaluate(x, y, 1.0, mask)
    got, _ = gpu_eval(y, x, 1.0, mask, tile=tile)
    pairs = np.tril(mask == 0, -1) if mask is not None else np.tril(np.ones_like(y), -1) > 0
    bound = TOL64 * abs(ref.loglik) + 0.5 * ((4 * U * y[pairs]) ** 2).sum()
    print(f"{label}: L {got['loglik']:.17g} oracle {ref.loglik:.17g} bound {bound:.2g}", flush=True)
    assert got["m_obs"] == ref.m_obs
    assert abs(got["loglik"] - ref.loglik) <= bound
    assert abs(got["loglik_only"] - ref.loglik) <= bound
    assert abs(got["dsigma"] - ref.dsigma) <= TOL64 * ref.abs_dsigma
    rowerr = np.max(np.abs(got["grad"] - ref.grad), axis=1)
    assert np.all(rowerr <= TOL64 * ref.condrow + 1e-300)


@pytest.mark.parametrize("tile", TILES)
@pytest.mark.parametrize("t", [0.0, 0.7, 2.0, 4.0, 5.5, 7.0, 8.0, 8.99])
def test_one_pair(t, tile):
    _check(np.array([[0.0], [t]]), None, tile, f"t={t} tile={tile}")


@pytest.mark.parametrize("tile", TILES)
@pytest.mark.parametrize("n", [65, 520, 1281])
@pytest.mark.parametrize("lo", [1.0, 4.0, 6.0, 8.0])
def test_two_clusters(lo, n, tile):
    # the observed pairs, one location in each cluster, at t in [lo, lo + 0.9]
    rng = np.random.default_rng(n)
    side = np.arange(n) % 2
    x = (side * (lo + 0.45) + 0.45 * rng.random(n))[:, None].copy()
    mask = (side[:, None] == side[None, :]).astype(np.uint8)
    _check(x, mask, tile, f"n={n} t in [{lo}, {lo + 0.9}] tile={tile}")
