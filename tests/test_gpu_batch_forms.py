"""The batched sweep's two forms and its grid: few tiles (one work-group per
CU), as many as the ordinary form holds, and more (the form with fewer
registers).  Every problem equals its single-problem call bit for bit, twice,
and the grid never exceeds the tiles rounded up to whole CUs."""
import numpy as np
import pytest
import torch

from paper_1905_04582_amd import api, synth

pytestmark = pytest.mark.gpu
DEV = "cuda"


@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
@pytest.mark.parametrize("dims", [(1, 2), (3, 4), (5, 6), (7, 8, 2)])
@pytest.mark.parametrize("sizes,many", [((2, 65, 130), False), ((900, 1501, 700), False),
                                        ((3001, 2050, 3500, 2700, 3300, 2900), True)])
def test_forms_equal_single_calls_bitwise(dtype, dims, sizes, many):
    probs = [synth.make_problem(n, dims[k % len(dims)], sigma=0.4, missing=0.1, seed=500 + k)
             for k, n in enumerate(sizes)]
    yv = [p.y.astype(np.float32) if dtype == torch.float32 else p.y for p in probs]
    B = api.MDSBatch([dict(y=y, d=p.d, mask=p.mask, tile_rows=32) for y, p in zip(yv, probs)],
                     dtype, DEV)
    for k, p in enumerate(probs):
        B.set_x(k, p.x)
        B.sigma[k] = p.sigma
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    tiles = B.plan.total_tiles
    assert B.plan.grid <= cus * max(1, -(-tiles // cus))
    assert bool(B.plan.flags & 2) == (dtype == torch.float64 or many)
    for _ in range(2):
        B.eval()
        torch.cuda.synchronize()
        for k, p in enumerate(probs):
            P = api.MDSProblem(yv[k], p.d, p.mask, dtype, DEV, *B.tiles[k])
            g, L, ds = P.gradient(B.x[k], p.sigma)
            torch.cuda.synchronize()
            assert torch.equal(g, B.grad[k]), k
            assert L.item() == B.loglik[k].item() and ds.item() == B.dsigma[k].item(), k
            B.grad[k].zero_()
