"""The exponential of the held-out density's running log-sum-exp against
mpmath: with the sum of a first draw set to zero, a second, less likely draw
leaves exp(l2 - l1) itself in the state."""
import mpmath as mp
import numpy as np
import pytest
import torch

from paper_1905_04582_amd import api

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("lo,hi", [(0.0, 1.0), (1.0, 40.0), (40.0, 690.0)])
def test_exp_of_a_less_likely_draw(lo, hi):
    # residuals r of the second draw: l2 - l1 = -r^2/2 (sigma = 1, and every
    # distance past the truncation terms)
    n = 64
    rng = np.random.default_rng(2)
    x1 = np.sort(rng.permutation(40 * n)[:n].astype(np.float64) * 64.0)[:, None]
    y = np.abs(x1 - x1.T)
    x2 = x1 + np.sqrt(rng.uniform(lo, hi, (n, 1)) / 2.0) * np.where(np.arange(n) % 2, 1, -1)[:, None]
    held = ((np.arange(n)[:, None] + np.arange(n)[None, :]) % 2).astype(np.uint8)
    one = api.HeldOutPairs(y, held)
    one.add_draw(x2, 1.0)
    both = api.HeldOutPairs(y, held)
    both.add_draw(x1, 1.0)
    state = both.acc.view(-1, 2)
    first = state[:both.m, 0].clone()
    state[:, 1] = 0.0
    both.add_draw(x2, 1.0)
    torch.cuda.synchronize()
    dl = (one.acc.view(-1, 2)[:one.m, 0] - first).cpu().numpy()
    got = state[:both.m, 1].cpu().numpy()
    less = dl < 0.0
    assert less.sum() > 500
    worst = max(abs(mp.mpf(g) / mp.exp(mp.mpf(v)) - 1) for g, v in zip(got[less], dl[less]))
    print(f"dl in [{dl.min():.3g}, {dl.max():.3g}], worst relative error {float(worst):.3g}", flush=True)
    # f's rounding (ln 2 / 4 of 2^-53), 2^f (2.2e-16, the polynomial's checked
    # error), all below two units in the last place
    assert worst < 2 * 2.0 ** -52
