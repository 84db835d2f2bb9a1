"""A gradient written beside X in one wider array, on either side of it, has
the bits of one written to an array of its own: only memory that the two share
changes the form of a small problem's evaluation."""
import pytest
import torch

from paper_1905_04582_amd import api
from tests.test_gpu_parity import _rand

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,d", [(2, 1), (300, 2), (1000, 5), (1100, 2)])
@pytest.mark.parametrize("x_at,g_at,width", [(0, 0, 0), (0, 1, 2), (1, 0, 2), (0, 2, 4)])
def test_same_bits(n, d, x_at, g_at, width):
    x0, y, mask, sigma = _rand(n, d, seed=n)
    P = api.MDSProblem(y, d, mask)
    want = P.gradient(torch.as_tensor(x0, device="cuda"), sigma)
    if width == 0:      # adjacent blocks of rows in one allocation
        buf = torch.full((2 * n, d), -5.0, dtype=torch.float64, device="cuda")
        x, g = buf[:n], buf[n:]
    else:
        buf = torch.full((n, width * d), -5.0, dtype=torch.float64, device="cuda")
        x, g = buf[:, x_at * d:(x_at + 1) * d], buf[:, g_at * d:(g_at + 1) * d]
    x.copy_(torch.as_tensor(x0))
    got = P.gradient(x, sigma, grad=g)
    for u, v in zip(got, want):
        assert torch.equal(u, v)
    assert torch.equal(x, torch.as_tensor(x0, device="cuda"))
