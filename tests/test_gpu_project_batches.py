"""A view's projection has the same bits alone and beside other views: up to
800,000 rays of a launch are shared by four waves, above they are marched
whole, in the plain and in the paired layout."""
import ctypes as C

import numpy as np
import pytest
import torch

from paper_2503_22139_amd import ops, synth
from paper_2503_22139_amd.synth import Cone, Grid

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    ops.lib()
    yield


def T(a):
    return torch.from_numpy(np.ascontiguousarray(a, np.float32)).cuda()


CONE = Cone(1000.0, 1500.0, 512, 384, 90.0 / 512, 70.0 / 384, off_u=0.3)
ANG = synth.scan_angle([3, 100, 222, 391, 500])


def plain(vol, stride, grid, cone, ang):
    out = torch.empty((ang.numel(), cone.nv, cone.nu), device="cuda")
    g, c = ops.make_grid(grid), ops.make_cone(cone)
    ops._check(ops.lib().pmf_project(ops._ptr(vol), stride, C.byref(g), C.byref(c), ops._ptr(ang), ang.numel(),
                                     ops._ptr(out), ops._stream()))
    return out


# rays of many samples, of a few, and of one
@pytest.mark.parametrize("n,step", [((33, 21, 18), 0.0), ((33, 21, 18), 30.0), ((2, 2, 2), 0.0), ((70, 40, 51), 0.3)])
@pytest.mark.parametrize("shared", [True, False])
def test_projection(n, step, shared):
    grid = Grid(n, (48.0 / n[0], 36.0 / n[1], 36.0 / n[2]), (3.0, -2.0, 1.0))
    cone = Cone(CONE.sad, CONE.sdd, CONE.nu, CONE.nv, CONE.du, CONE.dv, off_u=0.3, step=step)
    vol = T(synth.random_volume(8, n if shared else (5,) + n))
    ang = T(ANG)
    whole = ops.pmf_project(vol, grid, cone, ang, shared=shared)
    assert torch.equal(plain(vol, 0 if shared else grid.size, grid, cone, ang), whole)
    for v in range(5):
        one = vol if shared else vol[v].contiguous()
        assert torch.equal(ops.pmf_project(one, grid, cone, ang[v:v + 1], shared=True)[0], whole[v]), v
        assert torch.equal(plain(one, 0, grid, cone, ang[v:v + 1])[0], whole[v]), v


def test_motion_path():
    grid = Grid((40, 36, 32), (1.2, 1.2, 1.2))
    levels = synth.level_grids(grid, [(10, 9, 8), (40, 36, 32)])
    rng = np.random.default_rng(4)
    bases = [T(rng.normal(0, 1, (3,) + tuple(g.n))) for g in levels]
    coeff = T(rng.normal(0, 1, (5, 2, 1, 3)))
    ref, ang = T(synth.random_volume(9, grid.n)), T(ANG)
    all_ = ops.pmf_warp_project(ref, grid, bases, levels, coeff, CONE, ang)
    for v in range(5):
        one = ops.pmf_warp_project(ref, grid, bases, levels, coeff[v:v + 1], CONE, ang[v:v + 1])
        assert torch.equal(one[0], all_[v]), v
