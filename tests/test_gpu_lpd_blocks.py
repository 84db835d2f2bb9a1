"""One draw per pass around the lines of its launch shape (number of pairs,
dimension): the same bits as two draws per pass, whose shape does not change,
and the last pairs of the list as accurate as the first."""
import numpy as np
import pytest
import torch

from paper_1905_04582_amd import api

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d", [2, 4, 5, 8])
@pytest.mark.parametrize("m", [1, 127, 131071, 131072, 131073, 1048575, 1048576])
def test_one_draw_equals_two(m, d):
    rng = np.random.default_rng(m + d)
    n = 1500
    pi = rng.integers(1, n, m).astype(np.int32)
    pj = (pi * rng.random(m)).astype(np.int32)
    dev = dict(device="cuda")
    pi, pj = torch.as_tensor(pi, **dev), torch.as_tensor(pj, **dev)
    py = torch.as_tensor(4 * rng.random(m), **dev)
    xs = torch.as_tensor(rng.standard_normal((2, n, d)), **dev)
    sig = torch.tensor([0.5, 0.6], dtype=torch.float64, **dev)
    one = torch.full((2 * m + 2,), -7.0, dtype=torch.float64, **dev)
    two = one.clone()
    L, p = api.lib(), lambda t: t.data_ptr()
    for k in range(2):
        api._check(L.mds_lpd_accumulate(m, p(pi), p(pj), p(py), d, p(xs[k]), d, p(sig[k:]), p(one),
                                        1 if k == 0 else 0, api._stream()), "one")
    api._check(L.mds_lpd_accumulate_draws(m, p(pi), p(pj), p(py), d, p(xs), d, n * d, p(sig), 2,
                                          p(two), 1, api._stream()), "two")
    torch.cuda.synchronize()
    assert torch.equal(one, two)
    assert torch.all(one[2 * m:] == -7.0)
