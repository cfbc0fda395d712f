"""The local-maximum kernel behind FFPS_VARIANT_AUTO and the two sorts around it, at the
sizes where they can go wrong, against the oracle bit for bit (indices and squared
pick distances are the same individually rounded numbers on both sides)."""
import numpy as np
import pytest

from paper_2604_17720_amd import inputs

pytestmark = pytest.mark.gpu


def _dup(n, seed):
    return np.repeat(inputs.uniform_cube(n // 4, seed), 4, axis=0)


CASES = {
    # name: (clouds, M, start); a workgroup holds 512 points per row, 256 workgroups are the most
    "smallest": (lambda: inputs.uniform_cube(4609, 1)[None], 4609, 4608),
    "smallest with the work for it": (lambda: inputs.uniform_cube(5793, 1)[None], 5793, 5792),
    "just short of it": (lambda: inputs.uniform_cube(8192, 1)[None], 4095, 0),
    "few samples, still enough": (lambda: inputs.uniform_cube(2097152, 5)[None], 128, 9),
    "too few samples": (lambda: inputs.uniform_cube(2097152, 5)[None], 127, 9),
    "twenty-four rows, exactly": (lambda: inputs.uniform_cube(3145728, 6)[None], 150, 3145727),
    "thirty-two rows": (lambda: inputs.uniform_cube(3145729, 6)[None], 90, 0),
    "forty rows": (lambda: inputs.room(4194305, 6)[None], 100, 77),
    "the most a device holds": (lambda: inputs.uniform_cube(5242880, 7)[None], 80, 5242879),
    "beyond it": (lambda: inputs.uniform_cube(5242881, 7)[None], 80, 5),
    "a row of units and one point": (lambda: inputs.room(65537, 2)[None], 513, 65536),
    "more clouds than a launch, enough work": (lambda: np.stack([inputs.planes_and_clusters(9001, i) for i in range(15)]), 3728, 3),
    "a long line": (lambda: inputs.lattice_line(6000)[None], 6000, 0),
    "duplicates, fewer points than many samples": (lambda: _dup(16000, 8)[None], 5000, 0),
    "one row, exactly": (lambda: inputs.room(131072, 2)[None], 3000, 7),
    "one point more": (lambda: inputs.room(131073, 2)[None], 3000, 131072),
    "three rows and one point": (lambda: inputs.uniform_cube(393217, 3)[None], 500, 0),
    "many rows": (lambda: inputs.uniform_cube(1600001, 4)[None], 200, 5),
    "largest": (lambda: inputs.uniform_cube(3145728, 5)[None], 60, 9),
    "more clouds than fit one launch": (lambda: np.stack([inputs.uniform_cube(4700, i) for i in range(270)]), 90, 3),
    "clusters": (lambda: np.stack([inputs.planes_and_clusters(5003, i) for i in range(37)]), 600, 1),
    "one pick": (lambda: inputs.uniform_cube(5000, 6)[None], 2, 0),
    "equal values, bins too large for one sort in LDS": (lambda: inputs.lattice_grid(60, 60, 12)[None], 20000, 0),
    "a line": (lambda: inputs.lattice_line(5000)[None], 5000, 0),
    "duplicates, fewer points than samples": (lambda: _dup(16000, 8)[None], 5000, 0),
    "one place": (lambda: np.ones((1, 6000, 3), np.float32), 100, 3),
    "distances beyond fp32": (lambda: (inputs.uniform_cube(5000, 9) * 3e38).astype(np.float32)[None], 400, 0),
    "distances below the normal numbers": (lambda: (inputs.uniform_cube(5000, 9) * 3e-20).astype(np.float32)[None], 400, 0),
    "an outlier": (lambda: np.concatenate([inputs.uniform_cube(9000, 10), [[4e5, -3e5, 1e5]]]).astype(np.float32)[None], 2000, 1),
}


@pytest.mark.parametrize("name", list(CASES))
def test_local_maxima_give_the_samples_of_the_greedy_loop(oracle, name):
    import torch

    import paper_2604_17720_amd.binding as fb
    make, m, start = CASES[name]
    x = np.ascontiguousarray(make(), dtype=np.float32)
    print(name, x.shape, m, start, flush=True)
    ws = fb.make_workspace(x.shape[0], x.shape[1], m)
    idx, md = fb.ffps_exact(torch.from_numpy(x).cuda(), m, start, return_maxdist=True, workspace=ws)
    assert fb.ffps_last_status(ws) == 0
    ref, rmd = oracle.fps_exact(x, m, start, return_maxdist=True)
    assert np.array_equal(idx.cpu().numpy(), ref.reshape(idx.shape))
    assert np.array_equal(md.cpu().numpy().view(np.uint32), rmd.reshape(md.shape).view(np.uint32))


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
