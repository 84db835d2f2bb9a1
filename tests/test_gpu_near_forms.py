"""The special functions that the FP64 sweeps and the held-out density run for
pairs within nine sigma, one pair at a time against mpmath.  With delta = y = 1
exactly and sigma = 1/t the residual vanishes: the gradient is m(t)/sigma, and
the density's logarithm is -ln(sqrt(2 pi) sigma) - ln Phi(t)."""
import mpmath as mp
import numpy as np
import pytest
import torch

from paper_1905_04582_amd import api

pytestmark = pytest.mark.gpu

U = 2.0 ** -53
mp.mp.dps = 40
RANGES = [(1e-3, 0.1), (0.1, 3.0), (3.0, 6.0), (6.0, 8.999)]
X = [[0.0], [1.0]]
Y = [[0.0, 1.0], [1.0, 0.0]]


def _sigmas(lo, hi):
    return 1.0 / np.random.default_rng(1).uniform(lo, hi, 150)


def _f64(v):
    return torch.as_tensor(v, dtype=torch.float64, device="cuda")


@pytest.mark.parametrize("tile", [(0, 0), (8, 1)])
@pytest.mark.parametrize("lo,hi", RANGES)
def test_gradient_of_one_pair_is_m(lo, hi, tile):
    P = api.MDSProblem(_f64(Y), 1, None, torch.float64, "cuda", *tile)
    sig = _sigmas(lo, hi)
    s = _f64(sig)
    got = torch.stack([P.gradient(_f64(X), s[k])[0][:, 0] for k in range(sig.size)]).cpu().numpy()
    for v, g in zip(sig, got):
        t = 1 / mp.mpf(float(v))
        ref = mp.npdf(t) / mp.ncdf(t) * t
        # the rational 20 u, 2^f 2 u, the rest a rounding each; the factor
        # -log2(e)/(2 sigma^2) of the exponent 2.1 u of t^2/2
        bound = (40 + 1.1 * float(t) ** 2) * U
        assert abs((mp.mpf(float(g[0])) - ref) / ref) <= bound, float(t)
        assert g[1] == -g[0]


@pytest.mark.parametrize("lo,hi", RANGES)
def test_density_of_one_pair(lo, hi):
    sig = _sigmas(lo, hi)
    for v in sig:
        H = api.HeldOutPairs(_f64(Y), np.ones((2, 2), np.uint8))
        H.add_draw(_f64(X), float(v))
        s = mp.mpf(float(v))
        ref = -mp.log(mp.sqrt(2 * mp.pi) * s) - mp.log(mp.ncdf(1 / s))
        # two logarithms and their sums, each to a unit in the last place, of
        # numbers up to 10 (sigma in [0.11, 1000])
        assert abs(mp.mpf(H.acc[0].item()) - ref) <= 4 * 2 * U * (1 + abs(mp.log(s)))
