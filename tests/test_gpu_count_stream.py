"""Counts that a constructor or a check reads back on a caller's stream: the
read waits for the kernel that writes them, also while that stream is busy
with earlier work."""
import numpy as np
import pytest
import torch

from paper_1905_04582_amd import api

pytestmark = pytest.mark.gpu


def _busy(stream):
    a = torch.ones((4096, 4096), device="cuda")
    torch.cuda.synchronize()
    with torch.cuda.stream(stream):
        for _ in range(20):
            a = a @ a * 1e-4
    return a


def test_heldout_pairs_on_a_busy_stream():
    n = 700
    rng = np.random.default_rng(4)
    y = torch.as_tensor(np.abs(rng.standard_normal((n, n))), device="cuda")
    held = torch.as_tensor(rng.random((n, n)) < 0.2, device="cuda")
    ref = api.HeldOutPairs(y, held)
    side = torch.cuda.Stream()
    keep = _busy(side)
    got = api.HeldOutPairs(y, held, stream=side)
    side.synchronize()
    assert got.m == ref.m == int(torch.tril(held, -1).sum())
    for a in ("pi", "pj", "py"):
        assert torch.equal(getattr(got, a), getattr(ref, a))
    del keep


def test_symmetry_count_on_a_busy_stream():
    y = torch.zeros((500, 500), dtype=torch.float64, device="cuda")
    y[7, 3] = 1.0
    y[9, 450] = 2.0
    side = torch.cuda.Stream()
    keep = _busy(side)
    assert api.mds_check_symmetric(y, stream=side) == 2
    del keep
