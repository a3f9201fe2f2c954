"""The voxelizer's binning and tiles at the edges of their chunks, windows and
layouts, against the FP64 oracle.

With unit values a (voxel, Gaussian) pair that a box, a column's range or the
binning dropped takes e^(-m/2) >= e^(-4.5) ~ 0.011 from its voxel.  m carries a
rounding error of about 30 2^-24 k^2 (s_max / s_min)^2 (`dm`), so pairs within
dm of the mask's edge may fall either side and a sum may be off by dm / 2 of
its terms, beside the volumes' float bar of 1e-4."""
import math

import numpy as np
import pytest
import torch

import oracle
from paper_2503_22139_amd import ops, synth
from paper_2503_22139_amd.synth import Grid

pytestmark = pytest.mark.gpu

K = 3.0


@pytest.fixture(scope="module", autouse=True)
def gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    ops.lib()
    yield


def T(a):
    return torch.from_numpy(np.ascontiguousarray(a, np.float32)).cuda()


def check(gs, grid, ratio=4.0):
    dm = 2e-5 * ratio * ratio
    t = [T(gs.mean), T(gs.scale), T(gs.quat), T(gs.value)]
    got = ops.pmf_voxelize(*t, grid, K).cpu().numpy().astype(np.float64)
    inner, edge, amb, absum = oracle.voxelize_band(gs, grid, K, dm)
    tol = (1e-4 + 0.5 * dm) * absum + 1e-7
    assert not (np.abs(got - inner) > amb + tol).any()
    # the adjoint takes the same pairs: its sum over <voxel gradient, value>
    # of unit gradients is the volume's sum
    ones = torch.ones((gs.c,) + tuple(grid.n), device="cuda")
    gv = ops.pmf_voxelize_bwd(*t, grid, K, ones)[3].double().sum().item()
    assert abs(gv - got.sum()) <= (amb + tol).sum() + 1e-5 * absum.sum()


def unit(rng, m, grid, **kw):
    gs = synth.gaussians(rng, m, grid, **kw)
    gs.value = np.ones_like(gs.value)
    return gs


# sizes around a chunk of 128 Gaussians and around 256 chunks
@pytest.mark.parametrize("m", [1, 127, 128, 129, 257, 32768, 32769])
def test_chunks(m):
    print(m, flush=True)
    grid = Grid((40, 33, 50), (1.0, 1.2, 0.9))
    check(unit(np.random.default_rng(m), m, grid, s_vox=(0.5, 1.0)), grid)


# 512 tiles (sixteen waves each) and 544 (four); three and nine channels'
# tiles; more tiles than one window of counts holds
@pytest.mark.parametrize("n,c,m", [((128, 128, 64), 1, 3000), ((136, 128, 64), 1, 3000),
                                   ((33, 47, 29), 3, 500), ((33, 47, 29), 9, 500),
                                   ((33, 47, 29), 2, 500), ((512, 384, 136), 1, 2000)])
def test_tiles(n, c, m):
    print(n, c, flush=True)
    grid = Grid(n, (1.0, 1.0, 1.3), (5.0, -3.0, 2.0))
    check(unit(np.random.default_rng(n[0] + c), m, grid, c=c, s_vox=(0.5, 2.0)), grid)


# boxes and column ranges: Gaussians thinner than a voxel, needles and discs,
# a grid far from the origin, large Gaussians (off the bins) among small ones
@pytest.mark.parametrize("s_vox,center,m", [((0.05, 0.2), (0.0, 0.0, 0.0), 2000),
                                            ((0.4, 4.0), (0.0, 0.0, 0.0), 300),
                                            ((0.4, 4.0), (900.0, -1200.0, 700.0), 300),
                                            ((1.5, 15.0), (3.0, 2.0, 1.0), 60)])
@pytest.mark.parametrize("c", [1, 3])
def test_boxes(s_vox, center, m, c):
    print(s_vox, center, c, flush=True)
    grid = Grid((96, 80, 72), (1.0, 1.2, 1.5), center)
    gs = unit(np.random.default_rng(m), m, grid, c=c, s_vox=s_vox)
    if center[0] > 100.0:
        # positions of a far grid carry 2^-24 of it: against a grid at the
        # origin the voxel centres agree to that only, so take exact ones
        gs.mean = np.round(gs.mean * 64.0).astype(np.float32) / 64.0
        grid = Grid((96, 80, 72), (1.0, 1.25, 1.5), center)
    check(gs, grid, ratio=s_vox[1] / s_vox[0])


def test_no_gaussians():
    grid = Grid((40, 33, 50), (1.0, 1.2, 0.9))
    z = np.zeros((0, 3), np.float32)
    out = ops.pmf_voxelize(T(z), T(z), T(np.zeros((0, 4))), T(np.zeros((0, 1))), grid, K)
    assert not out.any()


# the adjoint's walks: boxes of fewer and more than 64 columns and columns of
# more than a window of voxels, sets of one workgroup's size and around it
@pytest.mark.parametrize("c", [1, 2, 3, 9])
@pytest.mark.parametrize("m,s_vox,n", [(3, (6.0, 12.0), (40, 36, 90)), (4, (0.3, 0.6), (20, 21, 22)),
                                       (65, (0.5, 2.0), (20, 21, 22)), (130, (0.05, 3.0), (9, 70, 11))])
def test_adjoint_walks(m, s_vox, n, c):
    print(m, s_vox, n, c, flush=True)
    grid = Grid(n, (1.0, 1.2, 0.9), (1.0, 2.0, -3.0))
    gs = synth.gaussians(np.random.default_rng(m), m, grid, c=c, s_vox=s_vox, value_sigma=1.0)
    gv = synth.random_normal(m, (c,) + tuple(n))
    want = oracle.voxelize_bwd(gs, grid, K, gv)
    got = ops.pmf_voxelize_bwd(T(gs.mean), T(gs.scale), T(gs.quat), T(gs.value), grid, K, T(gv))
    for name, g in zip(("mean", "scale", "quat", "value"), got):
        w = want[name]
        e = np.linalg.norm(g.cpu().numpy().astype(np.float64) - w)
        assert e <= 1e-3 * np.linalg.norm(w), (name, e)


# the largest set whose tiles search all its Gaussians, and one more (lists),
# with large Gaussians among them
@pytest.mark.parametrize("m", [4096, 4097])
@pytest.mark.parametrize("c", [1, 2, 3])
def test_search_or_lists(m, c):
    print(m, c, flush=True)
    grid = Grid((64, 60, 56), (1.0, 1.2, 0.9))
    gs = unit(np.random.default_rng(m), m, grid, c=c, s_vox=(0.3, 0.6))
    gs.scale[::500] *= 20.0
    check(gs, grid, ratio=2.0)
