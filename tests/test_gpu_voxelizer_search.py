"""Sets whose tiles search all Gaussians against the same ones by lists: the sums
are of integers with the same scales, so the same bits.  The set that takes the
lists has Gaussians far outside the grid more."""
import numpy as np
import pytest
import torch

from paper_2503_22139_amd import ops, synth
from paper_2503_22139_amd.synth import Grid

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    ops.lib()
    yield


def T(a):
    return torch.from_numpy(np.ascontiguousarray(a, np.float32)).cuda()


# up to 256 tiles 4,096 Gaussians are searched, up to 512 tiles 1,000
@pytest.mark.parametrize("n,m", [((64, 60, 56), 4096), ((128, 120, 61), 1000)])
@pytest.mark.parametrize("c", [1, 2, 3, 9])
def test_search_has_the_bits_of_lists(n, m, c):
    print(n, m, c, flush=True)
    grid = Grid(n, (1.0, 1.2, 0.9))
    gs = synth.gaussians(np.random.default_rng(m), m, grid, c=c, s_vox=(0.4, 1.5), value_sigma=1.0)
    gs.scale[::200] *= 12.0                     # some past the bins
    t = [T(gs.mean), T(gs.scale), T(gs.quat), T(gs.value)]
    far = [torch.cat([x, x[:1]]) for x in t]
    far[0][-1] += 1e4
    assert torch.equal(ops.pmf_voxelize(*t, grid), ops.pmf_voxelize(*far, grid))
