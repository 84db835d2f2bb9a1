"""Default tile shapes by size, dimension and precision: the shape on both sides
of each line of the rule, every default valid with its workspace, and the
gradient with it against the oracle's rows."""
import numpy as np
import pytest
import torch

import oracle
from paper_1905_04582_amd import api, synth

F64, F32 = api.MDS_F64, api.MDS_F32
tw = api.tile_waves


@pytest.mark.parametrize("n,d,dtype,shape", [
    (1024, 4, F64, (8, 1)), (1025, 4, F64, (32, tw(1, 4))), (2048, 4, F32, (32, tw(1, 4))),
    (2048, 5, F64, (32, tw(1, 2))), (2049, 2, F32, (64, tw(1, 4))), (2049, 2, F64, (32, tw(1, 2))),
    (3072, 3, F64, (64, tw(1, 4))), (6144, 3, F64, (64, tw(1, 2))), (6145, 3, F64, (64, tw(2, 2))),
    (6145, 1, F32, (64, tw(1, 2))), (6145, 8, F64, (64, tw(1, 2))), (8192, 8, F32, (64, tw(2, 2))),
    (8193, 2, F64, (128, tw(2, 2))), (8193, 4, F64, (64, tw(2, 2))), (8193, 4, F32, (128, tw(2, 2))),
    (8193, 8, F32, (64, 4)), (8193, 8, F64, (64, tw(1, 2))), (8193, 1, F32, (64, tw(1, 2))),
    (12289, 7, F32, (128, tw(2, 2))), (12289, 4, F64, (128, 2)), (30000, 8, F32, (64, 4)),
])
def test_shape(n, d, dtype, shape):
    assert api.mds_resolve_tiling(n, d, dtype) == shape


def test_every_default_is_valid():
    for n in (1, 64, 1024, 1025, 1537, 2049, 3073, 6145, 8193, 12289, 100000):
        for d in range(1, 9):
            for dtype in (F64, F32):
                br, wv = api.mds_resolve_tiling(n, d, dtype)
                assert api.mds_resolve_tiling(n, d, dtype, br, wv) == (br, wv)
                assert api.mds_workspace_bytes(n, d, dtype, 0, 0) > 0


@pytest.mark.gpu
@pytest.mark.parametrize("n,d,dtype,tol", [
    (1601, 4, torch.float64, 1e-12), (2049, 3, torch.float64, 1e-12),
    (3071, 8, torch.float32, 2.0**-17), (6145, 2, torch.float32, 2.0**-17),
    (8193, 5, torch.float64, 1e-12), (8193, 8, torch.float32, 2.0**-17),
])
def test_gradient_rows(n, d, dtype, tol):
    # (the parity tests' bounds: a row's error over its condition bound)
    p = synth.make_problem(n, d, sigma=0.4, missing=0.1, seed=n)
    y = p.y.astype(np.float32) if dtype == torch.float32 else p.y
    P = api.MDSProblem(y, d, p.mask, dtype, "cuda")
    g, _, _ = P.gradient(torch.as_tensor(p.x, device="cuda"), p.sigma)
    rows = np.unique(np.r_[0, 63, 64, np.linspace(0, n - 1, 24).astype(int), n - 1])
    ref, _, b = oracle.grad_rows(p.x, y.astype(np.float64), p.sigma, rows, p.mask)
    err = np.max(np.abs(g.cpu().numpy()[rows] - ref), axis=1)
    assert np.all(err <= tol * b)
