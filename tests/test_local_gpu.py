"""The local-maximum kernel behind FFPS_VARIANT_AUTO and the two sorts around it, at the
sizes where they can go wrong, against the oracle bit for bit (indices and squared
pick distances are the same individually rounded numbers on both sides)."""
import numpy as np
import pytest

from paper_2604_17720_amd import inputs

pytestmark = pytest.mark.gpu


def _dup(n, seed):
    return np.repeat(inputs.uniform_cube(n // 4, seed), 4, axis=0)


def _outlier(n):
    return np.concatenate([inputs.uniform_cube(n, 10), [[4e5, -3e5, 1e5]]]).astype(np.float32)[None]


def _denser(n, seed):
    """A cube in which a tenth of the points lies in a corner a thousand times as small."""
    x = inputs.uniform_cube(n, seed)
    x[: n // 10] *= 1e-3
    return x


CASES = {
    # name: (clouds, M, start[, kernel, where it is another one]); a workgroup holds 512 points per row,
    # 256 workgroups are the most; points x samples of 2^25 (2^26 beyond 65,536 points, 12 x 2^25 with many
    # clouds) and about a hundred samples are the least, or a fifth (a third) of up to 8192 points
    "smallest": (lambda: inputs.uniform_cube(4609, 1)[None], 4609, 4608),
    "smallest with the work for it": (lambda: inputs.uniform_cube(5793, 1)[None], 5793, 5792),
    "half of a small cloud": (lambda: inputs.uniform_cube(8192, 1)[None], 4095, 0),
    "just short of it": (lambda: inputs.uniform_cube(30000, 1)[None], 1118, 0, "GRID"),
    "few samples, still enough": (lambda: inputs.uniform_cube(2097152, 5)[None], 128, 9),
    "too few samples": (lambda: inputs.uniform_cube(2097152, 5)[None], 127, 9, "GRID"),
    "twenty-four rows, exactly": (lambda: inputs.uniform_cube(3145728, 6)[None], 150, 3145727),
    "thirty-two rows": (lambda: inputs.uniform_cube(3145729, 6)[None], 90, 0),
    "forty rows": (lambda: inputs.room(4194305, 6)[None], 100, 77),
    "the most a device holds": (lambda: inputs.uniform_cube(5242880, 7)[None], 80, 5242879),
    "beyond it": (lambda: inputs.uniform_cube(5242881, 7)[None], 80, 5, "STREAM"),
    "a row of units and one point": (lambda: inputs.room(65537, 2)[None], 1100, 65536),
    "a row of units and one point, few samples": (lambda: inputs.room(65537, 2)[None], 513, 65536, "GRID"),
    "as many clouds as fit one launch": (lambda: np.stack([inputs.planes_and_clusters(9001, i) for i in range(15)]), 3728, 3),
    "two launches, the second one short": (lambda: np.stack([inputs.uniform_cube(380001, i) for i in range(14)]), 180, 4),
    "a launch per cloud": (lambda: np.stack([inputs.uniform_cube(2700001, i) for i in range(2)]), 150, 2700000),
    "a long line": (lambda: inputs.lattice_line(6000)[None], 6000, 0),
    "duplicates, fewer points than many samples": (lambda: _dup(16000, 8)[None], 5000, 0),
    "one row, exactly": (lambda: inputs.room(131072, 2)[None], 3000, 7),
    "one point more": (lambda: inputs.room(131073, 2)[None], 3000, 131072),
    "three rows and one point": (lambda: inputs.uniform_cube(393217, 3)[None], 500, 0),
    "many rows": (lambda: inputs.uniform_cube(1600001, 4)[None], 200, 5),
    "largest": (lambda: inputs.uniform_cube(3145728, 5)[None], 60, 9, "GRID"),
    "many clouds of few samples": (lambda: np.stack([inputs.uniform_cube(4700, i) for i in range(270)]), 90, 3, "BLOCK"),
    "clusters in many clouds": (lambda: np.stack([inputs.planes_and_clusters(5003, i) for i in range(37)]), 600, 1, "GRID"),
    "equal values, bins sorted in LDS": (lambda: inputs.lattice_grid(40, 40, 8)[None], 3000, 0),
    "as many small workgroups as there are, exactly": (lambda: inputs.room(11264, 5)[None], 3000, 7),
    "one point more than that": (lambda: inputs.room(11265, 5)[None], 3000, 11264),
    "half a row per unit for many samples": (lambda: inputs.planes_and_clusters(30001, 5)[None], 7501, 1),
    "a fifth of the smallest": (lambda: inputs.uniform_cube(4609, 1)[None], 922, 4608),
    "small, equal values": (lambda: inputs.lattice_grid(20, 20, 20)[None], 1600, 0),
    "small, a line": (lambda: inputs.lattice_line(5000)[None], 2000, 0),
    "small, one place": (lambda: np.ones((1, 6000, 3), np.float32), 1200, 3),
    "small, duplicates": (lambda: _dup(6000, 8)[None], 1600, 0),
    "fifteen small ones": (lambda: np.stack([inputs.planes_and_clusters(4999, 90 + i) for i in range(15)]), 1667, 3),
    "an outlier, small": (lambda: _outlier(8000), 1700, 1),
    "six rows, exactly": (lambda: inputs.uniform_cube(786432, 7)[None], 130, 786431),
    "eight rows": (lambda: inputs.room(786433, 7)[None], 131, 5),
    "twelve rows": (lambda: inputs.uniform_cube(1048577, 7)[None], 130, 0),
    "twelve rows, exactly": (lambda: inputs.room(1572864, 7)[None], 129, 9),
    "equal values in six rows": (lambda: inputs.lattice_grid(88, 88, 88)[None], 150, 0),
    "equal values in eight rows": (lambda: inputs.lattice_grid(100, 100, 100)[None], 150, 7),
    "equal values in twelve rows": (lambda: inputs.lattice_grid(112, 112, 112)[None], 150, 0),
    "equal values in sixteen rows": (lambda: inputs.lattice_grid(160, 128, 102)[None], 200, 0),
    "equal values in rows that are read again": (lambda: inputs.lattice_grid(160, 128, 108)[None], 200, 0),
    "clusters": (lambda: np.stack([inputs.planes_and_clusters(9001, 50 + i) for i in range(4)]), 4000, 1),
    "one pick": (lambda: inputs.uniform_cube(5000, 6)[None], 2, 0, "GRID"),
    "equal values, bins too large for one sort in LDS": (lambda: inputs.lattice_grid(60, 60, 12)[None], 20000, 0),
    "a line": (lambda: inputs.lattice_line(5000)[None], 5000, 0),
    "duplicates, fewer points than samples": (lambda: _dup(24000, 8)[None], 7000, 0),
    "one place, few samples": (lambda: np.ones((1, 6000, 3), np.float32), 100, 3, "GRID"),
    "one place": (lambda: np.ones((1, 6000, 3), np.float32), 5700, 3),
    "one place but for two points": (lambda: np.concatenate([np.zeros((6000, 3)), [[1, 2, 3], [-1, 0, 2]]]).astype(np.float32)[None], 5700, 3),
    "distances beyond fp32, few samples": (lambda: (inputs.uniform_cube(5000, 9) * 3e38).astype(np.float32)[None], 400, 0, "GRID"),
    "distances beyond fp32": (lambda: (inputs.uniform_cube(6000, 9) * 3e38).astype(np.float32)[None], 5700, 0),
    "some distances beyond fp32": (lambda: (inputs.uniform_cube(9000, 9) * 1.4e19).astype(np.float32)[None], 4000, 8),
    "distances below the normal numbers, few samples": (lambda: (inputs.uniform_cube(5000, 9) * 3e-20).astype(np.float32)[None], 400, 0, "GRID"),
    "distances below the normal numbers": (lambda: (inputs.uniform_cube(6000, 9) * 3e-20).astype(np.float32)[None], 5700, 0),
    "distances that round to 0": (lambda: (inputs.uniform_cube(6000, 9) * 1e-22).astype(np.float32)[None], 5700, 0),
    "an outlier, few samples": (lambda: _outlier(9000), 2000, 1, "GRID"),
    "an outlier": (lambda: _outlier(9000), 6000, 1),
    "an outlier, most points left": (lambda: _outlier(40000), 1000, 40000),
    "places of different density": (lambda: _denser(20000, 3)[None], 8000, 0),
}


@pytest.mark.parametrize("name", list(CASES))
def test_local_maxima_give_the_samples_of_the_greedy_loop(oracle, name):
    import torch

    import paper_2604_17720_amd.binding as fb
    make, m, start, *other = CASES[name]
    x = np.ascontiguousarray(make(), dtype=np.float32)
    print(name, x.shape, m, start, flush=True)
    assert fb.ffps_describe_kernel(x.shape[0], x.shape[1], m) == getattr(fb, "FFPS_KERNEL_" + (other[0] if other else "LOCAL"))
    ws = fb.make_workspace(x.shape[0], x.shape[1], m)
    idx, md = fb.ffps_exact(torch.from_numpy(x).cuda(), m, start, return_maxdist=True, workspace=ws)
    assert fb.ffps_last_status(ws) == 0
    ref, rmd = oracle.fps_exact(x, m, start, return_maxdist=True)
    assert np.array_equal(idx.cpu().numpy(), ref.reshape(idx.shape))
    assert np.array_equal(md.cpu().numpy().view(np.uint32), rmd.reshape(md.shape).view(np.uint32))


def test_more_clouds_than_workgroups(oracle):
    """258 clouds, one workgroup each: two launches.  All against the grid kernel, some against the oracle."""
    import torch

    import paper_2604_17720_amd.binding as fb
    b, n, m = 258, 20480, 19700
    assert fb.ffps_describe_kernel(b, n, m) == fb.FFPS_KERNEL_LOCAL
    x = np.stack([inputs.uniform_cube(n, 300 + i) if i % 2 else inputs.shape_cloud(n, 300 + i) for i in range(b)])
    xd, ws = torch.from_numpy(x).cuda(), fb.make_workspace(b, n, m)
    got, md = fb.ffps_exact(xd, m, 11, return_maxdist=True, workspace=ws)
    assert fb.ffps_last_status(ws) == 0
    ref, rmd = fb.ffps_exact(xd, m, 11, fb.FFPS_VARIANT_GRID, return_maxdist=True)
    assert torch.equal(got, ref) and torch.equal(md, rmd)
    for i in (0, 257):
        assert np.array_equal(got[i].cpu().numpy(), oracle.fps_exact(x[i], m, 11))


@pytest.mark.parametrize("flags", [3, 7])
def test_candidates_sampled_by_local_maxima(oracle, flags):
    """FPS-Prune whose candidates go to the kernel; drawn ones (7) have a first sample of their own per cloud."""
    import torch

    import paper_2604_17720_amd.binding as fb
    n, m = 24000, 6000
    assert fb.ffps_describe_kernel(3, n // 2, m // 2) == fb.FFPS_KERNEL_LOCAL
    x = np.stack([inputs.planes_and_clusters(n, 80 + i) for i in range(3)])
    ws = fb.make_workspace(3, n, m)
    got, k = fb.ffps_prune(torch.from_numpy(x).cuda(), m, 1, 2, flags, 777, workspace=ws, seed=5)
    assert fb.ffps_last_status(ws) == 0 and k == m // 2
    assert np.array_equal(got.cpu().numpy(), oracle.fps_prune(x, m, 1, 2, flags, 777, 5))


@pytest.mark.parametrize("n,m", [(45678, 1501), (400000, 170)])  # the kernel's area fits the library's array, and does not
def test_local_maxima_without_a_workspace(oracle, n, m):
    import torch

    import paper_2604_17720_amd.binding as fb
    assert fb.ffps_describe_kernel(1, n, m) == fb.FFPS_KERNEL_LOCAL
    x = inputs.room(n, 21)
    out = torch.empty((1, m), dtype=torch.int32, device="cuda")
    st = torch.empty(2, dtype=torch.int32, device="cuda")
    fb.ffps_exact_noalloc(torch.from_numpy(x).cuda(), m, out, 3, out_status=st)
    assert st[0].item() == 0 and st[1].item() > 0
    assert np.array_equal(out[0].cpu().numpy(), oracle.fps_exact(x, m, 3))


def test_auto_in_a_hip_graph(oracle):
    """Exact, pruned and chained calls of AUTO recorded in one graph, every replay against the oracle."""
    import torch

    import paper_2604_17720_amd.binding as fb
    x = np.stack([inputs.planes_and_clusters(12000, 70 + i) for i in range(2)])
    xd, m, st = torch.from_numpy(x).cuda(), 1500, (6000, 1500)
    ws = fb.make_workspace(2, 12000, 6000)
    e = torch.empty((2, m), dtype=torch.int32, device="cuda")
    p = torch.empty((2, 6000), dtype=torch.int32, device="cuda")
    c = torch.empty((2, sum(st)), dtype=torch.int32, device="cuda")
    fb.ffps_exact(xd, m, 0, workspace=ws, out=e)
    torch.cuda.synchronize()
    side, graph = torch.cuda.Stream(), torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=side):
        fb.ffps_exact(xd, m, 0, workspace=ws, out=e)
        fb.ffps_prune(xd, 6000, 1, 2, 3, 0, workspace=ws, out=p)
        fb.ffps_cached_stages(xd, st, 1, workspace=ws, out=c)
    for rep in range(3):
        print("replay", rep, flush=True)
        for t in (e, p, c):
            t.zero_()
        graph.replay()
        torch.cuda.synchronize()
        assert fb.ffps_last_status(ws) == 0
        assert np.array_equal(e.cpu().numpy(), oracle.fps_exact(x, m, 0))
        assert np.array_equal(p.cpu().numpy(), oracle.fps_prune(x, 6000, 1, 2, 3, 0))
        assert np.array_equal(c.cpu().numpy(), oracle.fps_stages(x, st, 1))
        eager = fb.ffps_exact(xd, m, 5, workspace=ws)
        torch.cuda.synchronize()
        assert np.array_equal(eager.cpu().numpy(), oracle.fps_exact(x, m, 5))


@pytest.mark.parametrize("n,m", [(60000, 1500), (9000, 8000)])
def test_give_up_path_of_local_maxima_ends_cleanly(oracle, n, m):
    """FFPS_ERR_TIMEOUT, forced from the host: a workgroup that misses a record at its first look gives
    up, all leave in the ordinary way, and the next call on the workspace is right again."""
    import torch

    import paper_2604_17720_amd.binding as fb
    x = inputs.room(n, 3)[None]
    assert fb.ffps_describe_kernel(1, n, m) == fb.FFPS_KERNEL_LOCAL
    xd, ws = torch.from_numpy(x).cuda(), fb.make_workspace(1, n, m)
    fb.ffps_exact(xd, m, 0, fb.FFPS_VARIANT_AUTO | fb.FFPS_VARIANT_TEST_NO_WAIT, workspace=ws)
    assert fb.ffps_last_status(ws) == fb.FFPS_ERR_TIMEOUT
    got = fb.ffps_exact(xd, m, 0, workspace=ws)
    assert fb.ffps_last_status(ws) == 0
    assert np.array_equal(got.cpu().numpy(), oracle.fps_exact(x, m, 0))


@pytest.mark.parametrize("n,m", [(1500, 700), (9000, 8000)])  # one workgroup, many
def test_a_coordinate_that_is_not_finite_is_reported(oracle, n, m):
    """Outputs are undefined then, but the call ends with FFPS_ERR_INTERNAL on either kernel (a point
    is picked again, which the kernels check themselves), and the workspace stays usable."""
    import torch

    import paper_2604_17720_amd.binding as fb
    x = inputs.uniform_cube(n, 4)[None]
    bad = x.copy()
    bad[0, n // 3, 1] = np.nan
    ws = fb.make_workspace(1, n, m)
    fb.ffps_exact(torch.from_numpy(bad).cuda(), m, 0, workspace=ws)
    assert fb.ffps_last_status(ws) == fb.FFPS_ERR_INTERNAL
    got = fb.ffps_exact(torch.from_numpy(x).cuda(), m, 0, workspace=ws)
    assert fb.ffps_last_status(ws) == 0
    assert np.array_equal(got.cpu().numpy(), oracle.fps_exact(x, m, 0))
