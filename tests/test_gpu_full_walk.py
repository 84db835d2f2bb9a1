"""Walks of the tiled sweep: waves wholly below the diagonal with every column
inside the problem, waves on the diagonal, waves with columns past the end and
waves whose rows are no whole batch.  The gradient of a problem has all of
them at sizes around multiples of the tile; each size against the oracle."""
import numpy as np
import pytest
import torch

import oracle
from paper_1905_04582_amd import api, synth

pytestmark = pytest.mark.gpu
DEV = "cuda"


# (relative to |L|, to a row's condition bound and to dL/dsigma's absolute sum:
# the bounds of the parity tests in each precision)
@pytest.mark.parametrize("dtype,tol_l,tol_g,tol_s", [(torch.float64, 1e-12, 1e-12, 1e-12),
                                                     (torch.float32, 1e-5, 2.0**-17, 2.0**-19)])
@pytest.mark.parametrize("d", [1, 2, 3, 4, 6, 8])
@pytest.mark.parametrize("n", [64, 127, 128, 129, 192, 257, 321])
def test_walks_against_oracle(n, d, dtype, tol_l, tol_g, tol_s):
    p = synth.make_problem(n, d, sigma=0.4, missing=0.1, seed=77 + n + d)
    y = p.y.astype(np.float32) if dtype == torch.float32 else p.y
    P = api.MDSProblem(y, d, p.mask, dtype, DEV, 32)
    g, L, ds = P.gradient(torch.as_tensor(p.x, device=DEV), p.sigma)
    torch.cuda.synchronize()
    ref = oracle.evaluate(p.x, y.astype(np.float64), p.sigma, p.mask)
    assert abs(L.item() - ref.loglik) <= tol_l * abs(ref.loglik)
    assert abs(ds.item() - ref.dsigma) <= tol_s * ref.abs_dsigma
    err = np.max(np.abs(g.cpu().numpy() - ref.grad), axis=1)
    assert np.all(err <= tol_g * ref.condrow)
