"""Sets of three and nine channels that leave most tiles empty, on more tiles
than the splat takes (voxel owners): voxels that no Gaussian reaches are exact
zeros, the others as on the grid's own corner."""
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


# lists of one chunk, of exactly one, and of several
@pytest.mark.parametrize("c", [3, 9])
@pytest.mark.parametrize("m", [1, 60, 400])
def test_empty_tiles_are_zero(c, m):
    grid = Grid((112, 112, 112), (1.0, 1.1, 0.9))
    gs = synth.gaussians(np.random.default_rng(m), m, Grid((20, 20, 20), grid.h), c=c, s_vox=(0.5, 1.5))
    t = [T(a) for a in (gs.mean, gs.scale, gs.quat, gs.value)]
    got = ops.pmf_voxelize(*t, grid, 3.0).cpu().numpy()
    want = oracle.voxelize(gs, grid, 3.0)
    assert np.linalg.norm(got - want) <= 1e-4 * np.linalg.norm(want)
    far = np.ones(grid.n, bool)
    far[36:76, 36:76, 36:76] = False            # the body and its Gaussians' reach
    assert not got[:, far].any() and np.isfinite(got).all()
