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
    assert kernel(80, 8192, 9) == fb.FFPS_KERNEL_BLOCK
    assert kernel(79, 8192, 9) == fb.FFPS_KERNEL_GRID
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
    assert kernel(65535, 30000, 20000) == fb.FFPS_KERNEL_LOCAL
    assert kernel(65536, 30000, 20000) == fb.FFPS_KERNEL_GRID
    assert kernel(65536, 8193, 8193) == fb.FFPS_KERNEL_GRID


def test_few_samples_and_many_clouds_stay_with_rounds_of_candidates():
    """Where picks by local maxima were measured to be slower than the kernel they replaced: few
    samples of many points, and many clouds, each of which has only few workgroups then."""
    local, grid = fb.FFPS_KERNEL_LOCAL, fb.FFPS_KERNEL_GRID
    assert [kernel(1, n, m) for n, m in ((65536, 512), (65537, 512), (100000, 336), (100000, 672), (200000, 335), (200000, 336))] == \
        [local, grid, grid, local, grid, local]
    assert kernel(1, 3145729, 80) == local and kernel(1, 3145729, 79) == fb.FFPS_KERNEL_STREAM
    assert [kernel(b, 30000, 7500) for b in (1, 8, 15, 16, 64)] == [local, local, local, grid, grid]
    assert [kernel(b, 16384, 4096) for b in (16, 17, 256)] == [local, grid, grid]
    assert [kernel(b, 30000, 15000) for b in (16, 128)] == [local, local]
    assert [kernel(b, 8192, 4096) for b in (1, 16, 17, 79)] == [local, local, grid, grid]
    # a device with fewer CUs
    assert kernel(8, 30000, 7500, num_cu=64) == grid and kernel(4, 16384, 4096, num_cu=64) == local


def test_a_workspace_sized_for_other_clouds():
    """What a workspace held before the local-maximum kernel had an area of its own still suffices:
    such a call runs the kernels without it."""
    other = fb.ffps_workspace_bytes(1, 6000000, 1024)  # of a larger cloud, which has no such area
    assert other < fb.ffps_workspace_bytes(1, 5000000, 1024)
    assert kernel(1, 5000000, 1024, ws_bytes=other) == fb.FFPS_KERNEL_STREAM
    assert kernel(1, 5000000, 1024) == fb.FFPS_KERNEL_LOCAL
    # bytes per call: status, exchange, coordinates, samples, bitmap, distances, candidates, starts
    up = lambda v: (v + 255) // 256 * 256
    least = 256 + 256 * 2 * 6 * 256 * 16 + up(12 * 200000) + up(4 * 50000) + up(4 * 6250) + 2 * up(4 * 200000) + up(4)
    assert kernel(1, 200000, 50000, ws_bytes=least) == fb.FFPS_KERNEL_GRID
    with pytest.raises(fb.FlashFPSError) as e:
        kernel(1, 200000, 50000, ws_bytes=least - 1)
    assert e.value.code == fb.FFPS_ERR_WORKSPACE_TOO_SMALL


@pytest.mark.parametrize("b,n,m", [(4096, 4700, 90), (1, 200000, 167), (1, 1000000, 33), (1, 5000000, 6), (70000, 9000, 4000)])
def test_no_area_for_calls_that_cannot_use_it(b, n, m):
    assert kernel(b, n, m) != fb.FFPS_KERNEL_LOCAL
    assert fb.ffps_workspace_bytes(b, n, m) == _least(b, n, m)


def _least(b, n, m):
    """What a workspace needs without the area of the local-maximum kernel."""
    up = lambda v: (v + 255) // 256 * 256
    return 256 + 256 * 2 * 6 * 256 * 16 + up(12 * b * n) + up(4 * b * m) + up(4 * b * ((n + 31) // 32)) + 2 * up(4 * b * n) + up(4 * b)


def test_small_clouds_go_to_local_maxima_early():
    """Up to four clouds of up to 8192 points from a fifth of the points as samples on, up to fifteen from a third,
    beyond that size with a line of its own as well."""
    local, grid = fb.FFPS_KERNEL_LOCAL, fb.FFPS_KERNEL_GRID
    assert [kernel(1, 5000, m) for m in (999, 1000, 2223, 2500, 5000)] == [grid, local, local, local, local]
    assert [kernel(b, 5000, 1000) for b in (4, 5)] == [local, grid]
    assert [kernel(b, 5000, 1667) for b in (5, 15, 16)] == [local, local, grid]
    assert kernel(5, 5000, 1666) == grid
    assert [kernel(1, n, n // 2) for n in (4610, 6500, 8000, 8191)] == [local] * 4
    assert [kernel(15, 8193, m) for m in (2730, 2731)] == [grid, local]
    assert [kernel(1, 9000, m) for m in (1500, 2097, 2098)] == [grid, grid, local]
    assert [kernel(1, 16000, m) for m in (1500, 2097, 2098)] == [grid, grid, local]
    assert [kernel(1, 65536, m) for m in (511, 512)] == [grid, local]


@pytest.mark.parametrize("b", [1, 4, 5, 15, 16, 17, 64])
def test_more_samples_never_lead_back(b):
    """Once a cloud has the samples for local maxima, more of them do not make it another kernel's."""
    for n in (4609, 5000, 6999, 8192, 8193, 11000, 30000, 65536, 65537, 200000):
        ks = [kernel(b, n, m) for m in sorted({min(n, int(80 * 1.03 ** i)) for i in range(400)})]
        assert ks == sorted(ks), (b, n)


def test_candidates_and_stages_have_the_area():
    """What a call samples on the way has no more points and no more samples than the call; where that is a case for
    local maxima, the workspace of the call holds its area."""
    sizes = (4609, 4700, 6000, 8192, 8193, 9500, 12953, 20000, 52500, 65536, 65537, 70000, 100000, 400000, 3000000)
    samples = (96, 300, 470, 512, 700, 921, 922, 1200, 1536, 1537, 1667, 2098, 3000, 6000, 40000)
    used = 0
    for b in (1, 4, 5, 15, 16, 17):
        for n in sizes:
            for m in [s for s in samples if s <= n]:
                area = fb.ffps_workspace_bytes(b, n, m) - _least(b, n, m)
                for n1 in [s for s in sizes if s <= n]:
                    for m1 in [s for s in samples if s <= min(m, n1)]:
                        if kernel(b, n1, m1) == fb.FFPS_KERNEL_LOCAL:
                            used += 1
                            assert kernel(b, n1, m1, ws_bytes=_least(b, n1, m1) + area) == fb.FFPS_KERNEL_LOCAL, (b, n, m, n1, m1)
    assert used > 1000
    assert fb.ffps_workspace_bytes(1, 12000, 300) == _least(1, 12000, 300)  # and none that nothing can use
