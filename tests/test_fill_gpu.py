"""Candidate sets and fills of FPS-Prune at the edges of their tiles (32,768 points of the bitmap where one block
fills, 8,192 where several do, 4,096 of the drawn candidates; 1,024 places of the seeded permutation; beyond
256 tiles of the bitmap a block takes several), whole numbers against the oracle."""
import numpy as np
import pytest

from paper_2604_17720_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,m,start,b", [(31, 9, 30, 3), (4096, 2048, 0, 2), (4097, 4097, 4096, 1), (32768, 900, 32767, 1),
                                         (32769, 3000, 32768, 2), (65537, 700, 5, 1), (1100003, 300, 1100002, 1),
                                         (8421377, 40, 8421376, 1)])
@pytest.mark.parametrize("flags", [3, 7])
def test_prune_at_the_edges_of_tiles(oracle, n, m, start, b, flags):
    import torch

    import paper_2604_17720_amd.binding as fb
    x = np.stack([inputs.uniform_cube(n, 50 + i) for i in range(b)])
    ws = fb.make_workspace(b, n, m)
    for kn, kd in ((1, 2), (2, 3)):
        print(n, m, start, flags, kn, kd, flush=True)
        got, k = fb.ffps_prune(torch.from_numpy(x).cuda(), m, kn, kd, flags, start, workspace=ws, seed=11)
        assert fb.ffps_last_status(ws) == 0
        for i in range(b):
            assert np.array_equal(got[i].cpu().numpy(), oracle.fps_prune(x[i], m, kn, kd, flags, start, 11 + i))


@pytest.mark.parametrize("n,m,start,b", [(40960, 1024, 40959, 2), (40961, 1025, 0, 1), (32767, 2049, 8, 3), (2097153, 60, 2097152, 1)])
@pytest.mark.parametrize("flags", [2, 3, 6, 7])  # with and without candidates of their own
def test_fill_at_the_edges_of_smaller_tiles(oracle, n, m, start, b, flags):
    import torch

    import paper_2604_17720_amd.binding as fb
    x = np.stack([inputs.uniform_cube(n, 150 + i) for i in range(b)])
    ws = fb.make_workspace(b, n, m)
    for rep in range(2):  # what a call leaves in the workspace does not matter to the next one
        print(n, m, start, flags, rep, flush=True)
        got, k = fb.ffps_prune(torch.from_numpy(x).cuda(), m, 1, 3, flags, start + rep if start < n - 1 else start, workspace=ws, seed=19 + rep)
        assert fb.ffps_last_status(ws) == 0
        for i in range(b):
            want = oracle.fps_prune(x[i], m, 1, 3, flags, start + rep if start < n - 1 else start, 19 + rep + i)
            assert np.array_equal(got[i].cpu().numpy(), want)


@pytest.mark.parametrize("stages", [(2000, 1000), (2000, 1001, 7), (2000,) * 3, tuple(2000 - 100 * i for i in range(20)), (2000, *range(1000, 980, -1))])
@pytest.mark.parametrize("flags", [1, 2, 3, 7])
def test_stages_that_are_prefixes(oracle, stages, flags):
    """Written with the first stage's samples where none is longer than those, by a launch of their own
    otherwise and beyond sixteen."""
    import torch

    import paper_2604_17720_amd.binding as fb
    x = np.stack([inputs.planes_and_clusters(6000, 250 + i) for i in range(2)])
    ws = fb.make_workspace(2, 6000, 2000)
    got = fb.ffps_cached_stages(torch.from_numpy(x).cuda(), stages, fb.FFPS_MODE_CACHED, 1, 2, flags, 77, workspace=ws, seed=3)
    assert fb.ffps_last_status(ws) == 0
    assert np.array_equal(torch.cat(got, 1).cpu().numpy(), oracle.fps_stages(x, stages, 0, 1, 2, flags, 77, 3))
