"""The FP64 evaluation under a scaling of X, Y and sigma by a power of two: the
gradient and dL/dsigma scale by its inverse, exactly, as long as the squared
distances, their reciprocals and the weights stay in range."""
import numpy as np
import pytest

from paper_1905_04582_amd import api
from tests.test_gpu_parity import _rand, gpu_eval

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("tile", [(0, 0), (8, 1), (64, api.tile_waves(1, 4))])
@pytest.mark.parametrize("k", [-300, 300, 400])
def test_scaled_problem(k, tile):
    x, y, mask, sigma = _rand(200, 2, seed=5)
    ref, _ = gpu_eval(y, x, sigma, mask, tile=tile)
    s = 2.0 ** k
    got, _ = gpu_eval(y * s, x * s, sigma * s, mask, tile=tile)
    assert np.array_equal(got["grad"] * s, ref["grad"])
    assert got["dsigma"] * s == ref["dsigma"]
