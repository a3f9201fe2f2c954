"""The FDK filter's transforms at the edges of their lengths, row slots and
row pairs, against the FP64 oracle (bar 1e-4, as for every volume)."""
import numpy as np
import pytest
import torch

from oracle import fdk as ofdk
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


def case(nu, nv, V=3, seed=1):
    grid = Grid((6, 5, 7), (3.0, 3.0, 3.0), (1.0, -2.0, 0.5))
    cone = Cone(1000.0, 1500.0, nu, nv, 40.0 / nu, 40.0 / nv, off_u=0.2, off_v=-0.3)
    ang = synth.evenly_spaced_angles(V)
    return grid, cone, ang, synth.projection_like(seed, V, nv, nu)


# rows that fill half a transform exactly, one pixel more (the next length),
# and the shortest; row counts around a slot's eight and odd ones
@pytest.mark.parametrize("nu,nv", [(1, 9), (2, 8), (32, 7), (33, 1), (64, 9), (65, 17), (128, 3), (129, 16),
                                   (256, 5), (257, 2), (512, 10), (513, 3), (1024, 4), (1025, 3),
                                   (2048, 2), (2049, 3), (4096, 5)])
def test_transform_lengths(nu, nv):
    print(nu, nv, flush=True)
    grid, cone, ang, proj = case(nu, nv)
    got = ops.pmf_fdk(T(proj), cone, T(ang), grid).cpu().numpy().astype(np.float64)
    want = ofdk.fdk(proj, cone, ang.astype(np.float64), grid)
    assert np.linalg.norm(got - want) <= 1e-4 * np.linalg.norm(want)


@pytest.mark.parametrize("bad", [np.nan, np.inf])
def test_a_bad_pixel_stays_in_its_row(bad):
    """A value that is not finite reaches what its own row reaches, not the
    row it shares a transform with."""
    grid, cone, ang, proj = case(96, 40, V=2)
    r = 21                                  # the second row of its pair
    proj[:, r] = 0.0
    clean = ops.pmf_fdk(T(proj), cone, T(ang), grid).cpu().numpy()
    proj[0, r, 50] = bad
    got = ops.pmf_fdk(T(proj), cone, T(ang), grid).cpu().numpy()
    fine = np.isfinite(got)
    # voxels that read row r in the first view: between rows r - 1 and r + 1
    tau_v = cone.dv * cone.sad / cone.sdd
    x, y, z = (np.asarray(grid.center[a]) + (np.arange(grid.n[a]) - (grid.n[a] - 1) / 2.0) * grid.h[a]
               for a in range(3))
    U = cone.sad - x * np.cos(ang[0])
    fv = (cone.sad * z[None, :] / U[:, None]) / tau_v + 0.5 * (cone.nv - 1) - cone.off_v
    reads = np.abs(fv - r) < 1.0
    assert not fine.all() and fine[:, 0, :][~reads].all()
    scale = np.abs(clean).max()
    assert np.abs(got[fine] - clean[fine]).max() <= 1e-5 * scale
