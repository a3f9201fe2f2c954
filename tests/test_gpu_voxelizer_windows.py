"""The voxelizer's binning over several windows of tiles: every chunk and
window, large Gaussians among them, against the FP64 oracle at voxels near the
Gaussians, and repeated bit for bit."""
import numpy as np
import pytest
import torch

import oracle
from paper_2503_22139_amd import ops, synth
from paper_2503_22139_amd.synth import Grid

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    ops.lib()
    oracle.build()
    yield


def T(a):
    return torch.from_numpy(np.ascontiguousarray(a, np.float32)).cuda()


# 12,321 tiles (33 in the second window), 24,649 (the third), 62,500 (six)
@pytest.mark.parametrize("n", [(888, 888, 2), (1256, 1256, 3), (2000, 2000, 2)])
@pytest.mark.parametrize("c,m", [(1, 3000), (1, 100), (3, 700)])
def test_windows(n, c, m):
    print(n, c, m, flush=True)
    grid = Grid(n, (1.0, 1.0, 1.0))
    rng = np.random.default_rng(m)
    gs = synth.gaussians(rng, m, grid, c=c, s_vox=(0.6, 2.0))
    gs.scale[::50] = 25.0                        # more than 32 tiles
    t = [T(a) for a in (gs.mean, gs.scale, gs.quat, gs.value)]
    got = ops.pmf_voxelize(*t, grid, 3.0)
    at = gs.mean + rng.normal(0, 1.5, gs.mean.shape)
    ix = [np.clip(np.round(at[:, a] + (n[a] - 1) / 2.0), 0, n[a] - 1).astype(np.int64) for a in range(3)]
    idx = np.unique((ix[0] * n[1] + ix[1]) * n[2] + ix[2])
    want = oracle.voxelize_points(gs, grid, 3.0, idx).T
    g = got.reshape(c, -1)[:, torch.from_numpy(idx).cuda()].cpu().numpy()
    assert np.linalg.norm(g - want) <= 1e-4 * np.linalg.norm(want)
    assert torch.equal(got, ops.pmf_voxelize(*t, grid, 3.0))
