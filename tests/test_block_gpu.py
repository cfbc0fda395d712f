"""The local-maximum kernel of one workgroup behind FFPS_VARIANT_AUTO, at the edges of its
shapes and on clouds with ties, against the oracle bit for bit (indices and squared pick
distances are the same individually rounded numbers on both sides)."""
import numpy as np
import pytest

from paper_2604_17720_amd import inputs

pytestmark = pytest.mark.gpu


def _shape(b, n):
    return np.stack([inputs.shape_cloud(n, 61000 + 5 * n + i) for i in range(b)])


def _far_clusters(b, n):
    """Eight clusters far apart in each cloud: most units are out of one another's reach, all of a half at times."""
    r = np.random.default_rng(n)
    c = r.uniform(-1, 1, (b, 8, 3)) * 100
    return (np.take_along_axis(c, r.integers(0, 8, (b, n))[..., None], 1) + r.uniform(-.5, .5, (b, n, 3))).astype(np.float32)


CASES = {
    # name: (clouds, M, start); a row of 16 lanes holds 16 points per step, 32 rows make the cloud
    "smallest": (lambda: _shape(3, 257), 257, 256),
    "two samples": (lambda: _shape(2, 300), 2, 7),
    "one point per lane, exactly": (lambda: _shape(2, 512), 500, 1),
    "one point more": (lambda: _shape(2, 513), 513, 512),
    "two per lane": (lambda: _shape(4, 1024), 512, 0),
    "odd": (lambda: _shape(3, 1531), 777, 1530),
    "three per lane and one": (lambda: _shape(2, 1537), 1537, 3),
    "five per lane": (lambda: _shape(2, 2049), 1000, 3),
    "seven per lane": (lambda: _shape(2, 3073), 900, 3072),
    "eight per lane, exactly": (lambda: _shape(2, 4096), 4096, 5),
    "largest of a workgroup": (lambda: _shape(2, 4608), 4608, 4607),
    "many clouds, twelve per lane": (lambda: _shape(80, 4609), 300, 4608),
    "many clouds, sixteen per lane": (lambda: _shape(81, 8192), 400, 8191),
    "more clouds than CUs": (lambda: _shape(300, 700), 90, 2),
    "more clouds than CUs, three per lane": (lambda: _far_clusters(257, 1537), 300, 2),
    "more clouds than CUs, four per lane": (lambda: np.concatenate([_shape(30, 1800), _far_clusters(240, 1800)]), 200, 2),
    "more clouds than CUs, six per lane": (lambda: _far_clusters(257, 3072), 150, 2),
    "more clouds than CUs, eight per lane": (lambda: np.concatenate([_shape(30, 4096), _far_clusters(230, 4096)]), 100, 2),
    "more clouds than CUs, equal values": (lambda: np.repeat(inputs.lattice_grid(16, 16, 12)[None], 258, 0), 300, 5),
    "equal values, four per lane": (lambda: inputs.lattice_grid(16, 16, 8)[None], 2048, 1),
    "planes": (lambda: np.stack([inputs.planes_and_clusters(4001, i) for i in range(5)]), 1500, 1),
    "lattice, many equal values": (lambda: inputs.lattice_grid(16, 16, 12)[None], 2000, 0),
    "a line": (lambda: inputs.lattice_line(1500)[None], 1500, 0),
    "duplicates, fewer points than samples": (lambda: np.repeat(inputs.uniform_cube(300, 8), 4, axis=0)[None], 1000, 0),
    "one place": (lambda: np.ones((2, 600, 3), np.float32), 100, 3),
    "distances beyond fp32": (lambda: (inputs.uniform_cube(2000, 9) * 3e38).astype(np.float32)[None], 400, 0),
    "distances below the normal numbers": (lambda: (inputs.uniform_cube(2000, 9) * 3e-20).astype(np.float32)[None], 400, 0),
    "an outlier": (lambda: np.concatenate([inputs.uniform_cube(3000, 10), [[4e5, -3e5, 1e5]]]).astype(np.float32)[None], 900, 1),
}


@pytest.mark.parametrize("name", list(CASES))
def test_one_workgroup_gives_the_samples_of_the_greedy_loop(oracle, name):
    import torch

    import paper_2604_17720_amd.binding as fb
    make, m, start = CASES[name]
    x = np.ascontiguousarray(make(), dtype=np.float32)
    print(name, x.shape, m, start, flush=True)
    assert fb.ffps_describe_kernel(x.shape[0], x.shape[1], m) == fb.FFPS_KERNEL_BLOCK
    ws = fb.make_workspace(x.shape[0], x.shape[1], m)
    idx, md = fb.ffps_exact(torch.from_numpy(x).cuda(), m, start, return_maxdist=True, workspace=ws)
    assert fb.ffps_last_status(ws) == 0
    ref, rmd = oracle.fps_exact(x, m, start, return_maxdist=True)
    assert np.array_equal(idx.cpu().numpy(), ref.reshape(idx.shape))
    assert np.array_equal(md.cpu().numpy().view(np.uint32), rmd.reshape(md.shape).view(np.uint32))


@pytest.mark.parametrize("n,m", [(1, 1), (2, 2), (63, 63), (64, 64), (65, 65), (127, 64), (128, 128), (129, 65), (200, 50), (256, 256)])
def test_one_wave_gives_the_samples_of_the_greedy_loop(oracle, n, m):
    import torch

    import paper_2604_17720_amd.binding as fb
    x = np.round(_shape(3, max(n, 2))[:, :n] * 8) / 8 if n % 2 else _shape(3, n)  # odd sizes: many equal values
    x = np.ascontiguousarray(x, dtype=np.float32)
    ws = fb.make_workspace(3, n, m)
    ws.fill_(0x5A)  # whatever an earlier call left
    idx, md = fb.ffps_exact(torch.from_numpy(x).cuda(), m, n - 1, return_maxdist=True, workspace=ws)
    assert fb.ffps_last_status(ws) == 0 and fb.ffps_last_rounds(ws) == 0
    ref, rmd = oracle.fps_exact(x, m, n - 1, return_maxdist=True)
    assert np.array_equal(idx.cpu().numpy(), ref.reshape(idx.shape))
    assert np.array_equal(md.cpu().numpy().view(np.uint32), rmd.reshape(md.shape).view(np.uint32))


@pytest.mark.parametrize("b", [1, 3])
@pytest.mark.parametrize("n,stages", [(9000, (4608, 1024, 257, 256, 64, 5)), (300, (150, 150, 20, 1)), (20, (20, 7, 7, 2) + (1,) * 20)])
def test_stages_read_through_the_samples_of_the_one_before(oracle, b, n, stages):
    import torch

    import paper_2604_17720_amd.binding as fb
    x = np.ascontiguousarray(_shape(b, n), dtype=np.float32)
    for mode in (fb.FFPS_MODE_CHAIN, fb.FFPS_MODE_CACHED):
        for num, den, flags in ((1, 1, 0), (1, 2, fb.FFPS_FLAG_CP | fb.FFPS_FLAG_IP)):
            ws = fb.make_workspace(b, n, stages[0])
            ws.fill_(0x5A)
            print(b, n, stages, mode, num, den, flush=True)
            outs = fb.ffps_cached_stages(torch.from_numpy(x).cuda(), stages, mode, num, den, flags, n // 3, workspace=ws)
            assert fb.ffps_last_status(ws) == 0
            got = np.concatenate([o.cpu().numpy() for o in outs], axis=1)
            assert np.array_equal(got, oracle.fps_stages(x, stages, mode, num, den, flags, n // 3))
