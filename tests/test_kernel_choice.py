"""Which kernel a call gets, asked of the library's host side: no GPU needed."""
import pytest

import paper_2604_17720_amd.binding as fb

kernel = fb.ffps_describe_kernel


def test_the_kernels_of_the_sizes():
    assert kernel(1, 256, 100) == fb.FFPS_KERNEL_WAVE
    assert kernel(1, 256, 100, fb.FFPS_VARIANT_WG) == fb.FFPS_KERNEL_WAVE
    assert kernel(1, 257, 100) == fb.FFPS_KERNEL_BLOCK
    assert kernel(1, 257, 1) == fb.FFPS_KERNEL_WG
    assert kernel(1, 1024, 512, fb.FFPS_VARIANT_WG) == fb.FFPS_KERNEL_WG
    assert kernel(1, 1024, 512, fb.variant_with_picks(0, 7)) == fb.FFPS_KERNEL_WG
    assert kernel(1, 4608, 9) == fb.FFPS_KERNEL_BLOCK
    assert kernel(32, 8192, 9) == fb.FFPS_KERNEL_BLOCK
    assert kernel(31, 8192, 9) == fb.FFPS_KERNEL_GRID
    assert kernel(1, 200000, 50000) == fb.FFPS_KERNEL_LOCAL
    assert kernel(1, 200000, 50000, fb.FFPS_VARIANT_GRID) == fb.FFPS_KERNEL_GRID
    assert kernel(1, 5000011, 1024) == fb.FFPS_KERNEL_LOCAL
    assert kernel(1, 5242881, 1024) == fb.FFPS_KERNEL_STREAM
    for bad in ((0, 10, 5), (1, 10, 11), (1, 10, 5, 9), (1, 10, 5, 0, 0), (1 << 16, 1 << 16, 1)):
        with pytest.raises(fb.FlashFPSError) as e:
            kernel(*bad, ws_bytes=1 << 40)
        assert e.value.code == fb.FFPS_ERR_INVALID_ARG


def test_more_clouds_than_a_grid_dimension_holds():
    """The sorts around the local-maximum kernel have a grid row per cloud, at most 65535: exact
    sampling of more clouds than that (it has no limit on them) goes through the grid kernel."""
    assert kernel(65535, 8193, 4097) == fb.FFPS_KERNEL_LOCAL
    assert kernel(65536, 8193, 4097) == fb.FFPS_KERNEL_GRID
    assert kernel(65536, 30000, 30000) == fb.FFPS_KERNEL_GRID
