"""The set-up kernels at the edges of their forms: the order by ranks and by
the radix sort, the relabelling prepare through LDS and by the direct gather,
the held-out compaction with rows at any byte alignment.  All of it is whole
numbers or copies, so every comparison is exact."""
import ctypes

import numpy as np
import pytest
import torch

from paper_1905_04582_amd import api
from tests import order_ref

pytestmark = pytest.mark.gpu

DEV = "cuda"


@pytest.mark.parametrize("n", [63, 64, 65, 257, 16385, 131072, 131073])
def test_order_forms(n):
    rng = np.random.default_rng(n)
    x = rng.standard_normal((n, 2))
    x[rng.integers(0, n, n // 3)] = x[5]        # ties keep index order
    perm = api.mds_spatial_order(torch.as_tensor(x, device=DEV)).cpu().numpy()
    assert np.array_equal(perm, order_ref.spatial_order(x))


@pytest.mark.parametrize("n", [511, 512, 1025, 8192, 8193])
@pytest.mark.parametrize("sdt,odt", [(torch.float64, torch.float64), (torch.float64, torch.float32),
                                     (torch.float32, torch.float64)])
def test_relabelling_prepare(n, sdt, odt):
    gen = torch.Generator(device=DEV)
    gen.manual_seed(n)
    ld = n + 3
    y = torch.rand((n, ld), generator=gen, dtype=sdt, device=DEV)[:, :n]
    y[n // 2, :7] = float("nan")
    mask = (torch.rand((n, ld), generator=gen, device=DEV) < 0.2).to(torch.uint8)[:, :n]
    perm = torch.randperm(n, generator=gen, device=DEV)
    perm[3], perm[n - 1] = -1, n                # out of range: missing pairs
    got, m = api.mds_prepare_y(y, odt, mask, perm=perm)
    ok = (perm >= 0) & (perm < n)
    p = perm.clamp(0, n - 1)
    want = y[p][:, p].to(odt)
    want[mask[p][:, p] != 0] = float("nan")
    want[~ok] = float("nan")
    want[:, ~ok] = float("nan")
    assert torch.equal(torch.nan_to_num(got[:, :n], nan=-1.0), torch.nan_to_num(want, nan=-1.0))
    assert m.item() == int((~torch.isnan(want)).tril(-1).sum().item())


@pytest.mark.parametrize("n", [2, 5, 64, 1025, 1030])
@pytest.mark.parametrize("pad,off", [(0, 0), (4 - 1030 % 4, 0), (1, 0), (2, 1)])
@pytest.mark.parametrize("masked", [False, True])
def test_heldout_rows_of_any_alignment(n, pad, off, masked):
    rng = np.random.default_rng(n + 7 * pad)
    ld = n + pad
    # the last row ends with the buffer: nothing past its n columns
    def rows(rate):
        a = (rng.random(off + (n - 1) * ld + n) < rate).astype(np.uint8) * 3
        t = torch.as_tensor(a, device=DEV)
        return t, torch.as_strided(t, (n, n), (ld, 1), off).cpu().numpy()

    held, h = rows(0.3)
    miss, m = rows(0.2)
    yn = rng.random((n, n))
    yn[rng.random((n, n)) < 0.05] = np.nan
    y = torch.as_tensor(yn, device=DEV)
    L = api.lib()
    nb = ctypes.c_size_t()
    assert L.mds_heldout_workspace_bytes(n, ctypes.byref(nb)) == 0
    ws = api.alloc_workspace(nb.value, DEV)
    cnt = torch.zeros((), dtype=torch.int64, device=DEV)
    args = (ctypes.c_void_p(y.data_ptr()), api.MDS_F64, n,
            ctypes.c_void_p(miss.data_ptr() + off) if masked else None, ld if masked else 0,
            ctypes.c_void_p(held.data_ptr() + off), ld, n)
    s = ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)
    assert L.mds_heldout_count(*args, cnt.data_ptr(), ws.data_ptr(), ws.numel(), s) == 0
    keep = np.tril(h != 0, -1) & ~np.isnan(yn)
    if masked:
        keep &= m == 0
    i, j = np.nonzero(keep)
    assert cnt.item() == len(i)
    k = max(len(i), 1)
    pi = torch.full((k,), -1, dtype=torch.int32, device=DEV)
    pj = torch.full((k,), -1, dtype=torch.int32, device=DEV)
    py = torch.zeros(k, dtype=torch.float64, device=DEV)
    assert L.mds_heldout_fill(*args, ws.data_ptr(), ws.numel(), len(i), pi.data_ptr(),
                              pj.data_ptr(), py.data_ptr(), s) == 0
    torch.cuda.synchronize()
    assert np.array_equal(pi.cpu().numpy()[:len(i)], i)
    assert np.array_equal(pj.cpu().numpy()[:len(i)], j)
    assert np.array_equal(py.cpu().numpy()[:len(i)], yn[i, j])


@pytest.mark.parametrize("kind", ["uint8", "bool", "int32", "float64", "strided", "numpy"])
def test_masks_of_any_type(kind):
    # any type marks its non-zero entries; the caller's mask is left alone
    rng = np.random.default_rng(3)
    n = 70
    y = rng.random((n, n))
    m = np.tril(rng.random((n, n)) < 0.3, -1)
    m = m | m.T
    if kind == "numpy":
        mask = m
    elif kind == "strided":
        wide = torch.zeros((n, 2 * n), dtype=torch.bool, device=DEV)
        wide[:, ::2] = torch.as_tensor(m)
        mask = wide[:, ::2]
    else:
        mask = torch.as_tensor(m).to(getattr(torch, kind)).to(DEV) * (7 if kind == "uint8" else 1)
    before = mask.copy() if kind == "numpy" else mask.clone()
    P = api.MDSProblem(y, 2, mask)
    H = api.HeldOutPairs(y, mask)
    want = np.where(m, np.nan, y)
    assert np.array_equal(P.y[:, :n].cpu().numpy(), want, equal_nan=True)
    assert int(P.m_obs.item()) == int((~m).sum() - n) // 2
    assert H.m == int(np.tril(m, -1).sum())
    assert np.array_equal(np.asarray(before if kind == "numpy" else before.cpu()),
                          np.asarray(mask if kind == "numpy" else mask.cpu()))
