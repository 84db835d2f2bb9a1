"""Lines of the default tile rule that follow from both the gradient and the
log-likelihood alone, and from the size of the workspace."""
import pytest

from paper_1905_04582_amd import api

F64, F32 = api.MDS_F64, api.MDS_F32
tw = api.tile_waves


@pytest.mark.parametrize("n,d,dtype,shape", [
    (8193, 2, F32, (64, tw(2, 2))), (10240, 2, F32, (64, tw(2, 2))),
    (10241, 2, F32, (128, tw(2, 2))), (8384, 3, F32, (64, tw(2, 2))),
    (8385, 3, F32, (128, tw(2, 2))), (8320, 5, F32, (128, tw(2, 2))),
    (8321, 5, F32, (64, tw(2, 2))), (8193, 6, F32, (64, tw(2, 2))),
    (9216, 7, F32, (64, tw(2, 2))), (9217, 7, F32, (128, tw(2, 2))),
    (8193, 6, F64, (128, tw(2, 2))), (9216, 1, F32, (64, tw(1, 2))),
])
def test_shape_lines(n, d, dtype, shape):
    assert api.mds_resolve_tiling(n, d, dtype) == shape


@pytest.mark.parametrize("n,d,dtype", [(32769, 8, F32), (60000, 8, F32), (240000, 8, F32),
                                       (60000, 8, F64), (60000, 2, F32)])
def test_workspace_of_large_problems(n, d, dtype):
    # no more partial sums than tiles of 128 x 128 leave
    assert api.mds_workspace_bytes(n, d, dtype) <= api.mds_workspace_bytes(n, d, dtype, 128, 2)


def test_shape_before_the_workspace_weighs():
    assert api.mds_resolve_tiling(32768, 8, F32) == (64, 4)
    assert api.mds_resolve_tiling(32769, 8, F32) == (128, 2)


@pytest.mark.parametrize("d", range(1, 9))
def test_static_scratch_holds_what_wide_tiles_leave(d):
    # mds_gradient_noalloc takes any FP32 problem above 8192 locations whose
    # partial sums of 128 x 128 tiles fit its scratch
    scratch = api.lib().mds_noalloc_scratch_bytes()
    for n in range(8193, 12289, 32):
        if api.mds_workspace_bytes(n, d, F32, 128, tw(2, 2)) <= scratch:
            assert api.mds_workspace_bytes(n, d, F32) <= scratch, n
