"""The one-channel voxelizer adjoint over boxes of different heights, whose columns
are walked in steps of 2, 4 and 8 voxels, against the FP64 oracle.

Bar: a voxel at the truncation surface may fall on either side of it, a term of
e^-4.5 of the largest in sums of some thousands: 1e-3 in norm.
"""
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


# heights of about 6 s: 5..8, 8..10, 14..19, the whole grid; grids cut at 2, 9
# and 17 voxels; untruncated sets
@pytest.mark.parametrize("n", [(40, 37, 61), (33, 30, 2), (33, 30, 9), (30, 33, 17)])
@pytest.mark.parametrize("s,k", [((0.8, 1.3), 3.0), ((1.2, 1.7), 3.0), ((2.2, 3.2), 3.0), ((8.0, 14.0), 3.0),
                                 ((3.0, 5.0), float("inf"))])
def test_heights(n, s, k):
    print(n, s, k, flush=True)
    grid = Grid(n, (1.5, 1.2, 2.0), (3.0, -1.0, 0.5))
    rng = np.random.default_rng(11)
    gs = synth.gaussians(rng, 60, grid, s_vox=s)
    g_vol = rng.normal(0, 1, n).astype(np.float32)
    got = ops.pmf_voxelize_bwd(T(gs.mean), T(gs.scale), T(gs.quat), T(gs.value), grid, k, T(g_vol))
    want = oracle.voxelize_bwd(gs, grid, k, g_vol)
    for name, a in zip(("mean", "scale", "quat", "value"), got):
        a = a.cpu().numpy().astype(np.float64)
        assert np.linalg.norm(a - want[name]) <= 1e-3 * np.linalg.norm(want[name]), name
