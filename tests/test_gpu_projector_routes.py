"""The projector's routes by launch size: paired copies of the volumes, rays
shared by four waves, bricks and chunks by workgroup count, and the adjoint
summed over views in rounds.

Routes that only move data (paired copies) have to give the plain route's
bits; routes that reorder a float sum of n non-negative terms agree to
2 n 2^-24; the summed adjoint is the views' volumes added in order.
"""
import ctypes as C

import numpy as np
import pytest
import torch

import oracle
from paper_2503_22139_amd import ops, synth
from paper_2503_22139_amd.synth import Cone, Grid

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


def rel(a, b):
    a, b = a.double(), b.double()
    return float((a - b).norm() / b.norm().clamp(min=1e-300))


def plain(vol, stride, grid, cone, ang):
    out = torch.empty((ang.numel(), cone.nv, cone.nu), device="cuda")
    g, c = ops.make_grid(grid), ops.make_cone(cone)
    ops._check(ops.lib().pmf_project(ops._ptr(vol), stride, C.byref(g), C.byref(c), ops._ptr(ang),
                                     ang.numel(), ops._ptr(out), ops._stream()))
    return out


def workspace(grid, cone, V, stride):
    g, c = ops.make_grid(grid), ops.make_cone(cone)
    return ops.lib().pmf_project_workspace(C.byref(g), C.byref(c), V, stride)


GRID = Grid((33, 21, 18), (1.5, 1.7, 2.0), (3.0, -2.0, 1.0))


@pytest.mark.parametrize("nu,nv,V,shared,paired", [
    (512, 293, 1, True, True),        # 150,016 rays: the first paired size, odd rows
    (512, 292, 1, True, False),       # one row less
    (512, 293, 9, False, True),       # per-view volumes in rounds of 8 + 1
    (512, 293, 6, True, True),        # above 800,000 rays: whole rays per wave
    (131, 67, 3, True, False),        # few rays: plain, shared by four waves
])
def test_paired_copy_gives_the_plain_bits(nu, nv, V, shared, paired):
    print(nu, nv, V, shared, flush=True)
    cone = Cone(1000.0, 1500.0, nu, nv, 90.0 / nu, 70.0 / nv, off_u=0.3)
    ang = T(synth.scan_angle(np.arange(V) * 61))
    n = GRID.size
    vol = T(synth.random_volume(5, (1 if shared else V,) + GRID.n))
    assert (workspace(GRID, cone, V, 0 if shared else n) > 0) == paired
    got = ops.pmf_project(vol, GRID, cone, ang, shared=shared)
    want = plain(vol, 0 if shared else n, GRID, cone, ang)
    assert torch.equal(got, want)
    rng = np.random.default_rng(1)
    rays = np.stack([rng.integers(0, V, 300), rng.integers(0, nu, 300), rng.integers(0, nv, 300)], 1)
    if shared:
        ref = oracle.project_rays(vol[0].cpu().numpy(), GRID, cone, ang.cpu().numpy(), rays)
        g = got.cpu().numpy()[rays[:, 0], rays[:, 2], rays[:, 1]]
        assert np.linalg.norm(g - ref) < 1e-4 * np.linalg.norm(ref)


def test_project_needs_its_workspace():
    cone = Cone(1000.0, 1500.0, 512, 293, 0.2, 0.25)
    ang, vol = T([0.3]), T(synth.random_volume(5, GRID.n))
    need = workspace(GRID, cone, 1, 0)
    assert need == 8 * GRID.size
    out = torch.empty((1, 293, 512), device="cuda")
    g, c = ops.make_grid(GRID), ops.make_cone(cone)
    for ws, size in ((None, 0), (ops.workspace(need, "cuda"), need - 1)):
        rc = ops.lib().pmf_project_ws(ops._ptr(vol), 0, C.byref(g), C.byref(c), ops._ptr(ang), 1,
                                      ops._ptr(out), None if ws is None else C.c_void_p(ws.data_ptr()),
                                      size, ops._stream())
        assert rc == ops.PMF_EWORKSPACE


def test_shared_and_whole_rays_agree():
    """Five views are marched whole, each alone by four waves: the same
    samples in another order (at most 120 terms, all non-negative)."""
    cone = Cone(1000.0, 1500.0, 512, 320, 90.0 / 512, 70.0 / 320)
    ang = T(synth.scan_angle([3, 100, 222, 391, 500]))
    vol = T(synth.random_volume(8, GRID.n))
    whole = ops.pmf_project(vol, GRID, cone, ang, shared=True)
    parts = torch.cat([ops.pmf_project(vol, GRID, cone, ang[v:v + 1], shared=True) for v in range(5)])
    assert rel(parts, whole) < 2 * 120 * 2.0 ** -24


def in_order(vols):
    out = vols[0].clone()
    for v in vols[1:]:
        out += v
    return out


@pytest.mark.parametrize("n,V", [
    ((44, 20, 8), 2),          # one default brick: no pads
    ((45, 21, 9), 3),          # one voxel past a brick on every axis
    ((33, 17, 18), 4),         # the smaller brick's edges; rows of 2 at the top
    ((90, 65, 31), 5),         # scalar rows (n2 odd)
    ((130, 70, 64), 40),       # default brick, both orientations
])
def test_summed_adjoint_is_the_views_in_order(n, V):
    print(n, V, flush=True)
    grid = Grid(n, (1.5, 1.4, 2.0), (1.0, 2.0, -1.0))
    cone = Cone(1000.0, 1500.0, 96, 61, 3.1, 3.3, off_v=0.4)
    ang = T(synth.scan_angle((np.arange(V) * 660) // V + 7))
    gp = T(synth.random_normal(9, (V, cone.nv, cone.nu)))
    got = ops.pmf_project_bwd(gp, grid, cone, ang, shared=True)
    views = ops.pmf_project_bwd(gp, grid, cone, ang, shared=False)
    assert torch.equal(got, in_order(views))
    if V <= 5:
        want = oracle.project_bwd(gp.cpu().numpy(), grid, cone, ang.cpu().numpy(), shared=True)
        assert np.linalg.norm(got.cpu().numpy() - want) < 1e-4 * np.linalg.norm(want)


def test_summed_adjoint_in_rounds():
    """17 views of a 256x256x128 volume take two rounds (16 + 1); the last
    round's view alone takes other bricks, so its fixed point is rounded apart
    (each of the ~1e2 contributions of a voxel to 2^-31 of the view's bound)."""
    grid = Grid((256, 256, 128), (1.5, 1.5, 2.0))
    cone = Cone(1000.0, 1500.0, 64, 48, 512 * 0.776 / 64, 384 * 0.776 / 48)
    ang = T(synth.scan_angle(np.arange(17) * 38))
    gp = T(synth.random_normal(10, (17, cone.nv, cone.nu)))
    got = ops.pmf_project_bwd(gp, grid, cone, ang, shared=True)
    views = ops.pmf_project_bwd(gp, grid, cone, ang, shared=False)
    assert rel(got, in_order(views)) < 1e-5


# around the 131,072 rows of eight from which a thread sums whole rows: the last
# that takes them in pairs, the first whole ones, scalar and with wide loads
@pytest.mark.parametrize("n", [(128, 127, 64), (128, 127, 61), (128, 128, 64), (200, 90, 62)])
def test_summed_adjoint_by_rows_and_pairs(n):
    print(n, flush=True)
    grid = Grid(n, (1.5, 1.4, 2.0), (1.0, 2.0, -1.0))
    cone = Cone(1000.0, 1500.0, 96, 61, 3.1, 3.3, off_v=0.4)
    ang = T(synth.scan_angle([7, 180, 415]))
    gp = T(synth.random_normal(11, (3, cone.nv, cone.nu)))
    got = ops.pmf_project_bwd(gp, grid, cone, ang, shared=True)
    views = ops.pmf_project_bwd(gp, grid, cone, ang, shared=False)
    assert torch.equal(got, in_order(views))
