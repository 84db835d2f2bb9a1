"""Trajectories around the size where they leave the small-problem form: the
end point, gradient and L of the library's choice against those of a named
tiling, to the trajectory tests' tolerance."""
import numpy as np
import pytest
import torch

from paper_1905_04582_amd import api
from tests.test_gpu_parity import _rand

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,d", [(1025, 2), (1100, 1), (1100, 6), (1101, 2), (1025, 7), (1280, 8),
                                 (1281, 8)])
@pytest.mark.parametrize("steps", [1, 4])
def test_line(n, d, steps):
    x0, y, mask, sigma = _rand(n, d, seed=n)
    p0 = np.random.default_rng(n).standard_normal((n, d))
    out = []
    for tile in ((0, 0), api.mds_resolve_tiling(n, d, api.MDS_F64)):
        P = api.MDSProblem(y, d, mask, torch.float64, "cuda", *tile)
        x, p = (torch.as_tensor(v, device="cuda").clone() for v in (x0, p0))
        g = torch.empty_like(x)
        L = torch.empty((), dtype=torch.float64, device="cuda")
        P.leapfrog(x, p, sigma, 1e-3, steps, g, L)
        out.append((x, p, g, L))
    for a, b in zip(*out):
        assert float((a - b).abs().max()) <= 1e-11 * float(b.abs().max())
