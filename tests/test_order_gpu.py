"""The order of the points before the kernels that pick local maxima, for clouds that do not fill their
bounding box: samples as on the kernels that need no order, bit for bit, and about as many rounds
as without what lies far away.  (The samples never depend on the order, the rounds do: with a plain
grid over the box they were 1.7 to 6 times as many.)"""
import numpy as np
import pytest

from paper_2604_17720_amd import inputs

pytestmark = pytest.mark.gpu

KINDS = {
    "one stray point": lambda x, r: np.concatenate([x[:-1], [[400.0, -350.0, 500.0]]]),
    "one just outside": lambda x, r: np.concatenate([x[:-1], [[7.0, 9.0, -8.0]]]),
    "eight strays": lambda x, r: np.concatenate([x[:-8], r.uniform(-60, 60, (8, 3))]),
    "a fifth at one place": lambda x, r: np.where((r.random(len(x)) < 0.2)[:, None], np.float32(3e5), x),
    "two parts": lambda x, r: x + np.where(np.arange(len(x)) % 2, 200.0, 0.0)[:, None],
}


@pytest.mark.parametrize("kind", list(KINDS))
@pytest.mark.parametrize("b,n,m", [(1, 1024, 512), (3, 4096, 1024), (2, 8193, 4100), (1, 45678, 5001), (1, 200000, 50000)])
def test_what_lies_far_away_leaves_the_rounds_alone(kind, b, n, m):
    import torch

    import paper_2604_17720_amd.binding as fb
    local = n > 4608
    assert fb.ffps_describe_kernel(b, n, m) == (fb.FFPS_KERNEL_LOCAL if local else fb.FFPS_KERNEL_BLOCK)
    x = np.stack([inputs.uniform_cube(n, 900 + i) for i in range(b)])
    far = np.stack([KINDS[kind](c, np.random.default_rng(31 + i)) for i, c in enumerate(x)]).astype(np.float32)
    ws = fb.make_workspace(b, n, m)
    rounds = []
    for c in (x, far):
        idx, md = fb.ffps_exact(torch.from_numpy(c).cuda(), m, 1, return_maxdist=True, workspace=ws)
        assert fb.ffps_last_status(ws) == 0
        rounds.append(fb.ffps_last_rounds(ws))
    ref, rmd = fb.ffps_exact(torch.from_numpy(far).cuda(), m, 1, fb.FFPS_VARIANT_GRID if local else fb.FFPS_VARIANT_WG,
                             return_maxdist=True)
    assert torch.equal(idx, ref) and torch.equal(md, rmd)
    print(kind, b, n, m, rounds, flush=True)
    assert rounds[1] <= 1.5 * rounds[0]


@pytest.mark.parametrize("n,m", [(2000, 700), (6000, 5700)])
@pytest.mark.parametrize("scale", [1e-30, 1.0, 3e34])
def test_keys_at_the_ends_of_fp32(oracle, n, m, scale):
    """Clusters and a stray point whose spread, extent or their reciprocals leave fp32."""
    import torch

    import paper_2604_17720_amd.binding as fb
    r = np.random.default_rng(5)
    x = r.uniform(-1, 1, (n, 3)) + np.where(np.arange(n) % 3 == 0, 300.0, 0.0)[:, None]
    x[n // 2] = 5e3
    x = (x * scale).astype(np.float32)
    assert np.isfinite(x).all()
    idx, md = fb.ffps_exact(torch.from_numpy(x).cuda(), m, 0, return_maxdist=True)
    ref, rmd = oracle.fps_exact(x, m, 0, return_maxdist=True)
    assert np.array_equal(idx[0].cpu().numpy(), ref) and np.array_equal(md[0].cpu().numpy().view(np.uint32), rmd.view(np.uint32))
