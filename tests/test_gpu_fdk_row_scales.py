"""Detector rows of unlike sizes that share one of the FDK filter's transforms:
each row's rounding errors follow its own largest value."""
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


# transforms by a part of a wave, a wave, and several waves
@pytest.mark.parametrize("nu", [20, 96, 512, 1100])
@pytest.mark.parametrize("first", [False, True])
@pytest.mark.parametrize("bright", [1e10, 1e20, float(np.finfo(np.float32).max)])
def test_a_bright_pixel_stays_in_its_row(nu, first, bright):
    """The other rows' filtered values change by a rounding to float at most:
    a few 2^-24 of the volume."""
    print(nu, first, bright, flush=True)
    nv, V = 40, 2
    grid = Grid((6, 5, 33), (3.0, 3.0, 0.2), (1.0, -2.0, 0.3))     # five samples per row
    cone = Cone(1000.0, 1500.0, nu, nv, 40.0 / nu, 40.0 / nv, off_u=0.2, off_v=-0.3)
    ang = synth.evenly_spaced_angles(V)
    proj = synth.projection_like(1, V, nv, nu)
    r = 20 if first else 21                 # the first, the second row of its pair
    proj[:, r] = 0.0
    clean = ops.pmf_fdk(T(proj), cone, T(ang), grid).cpu().numpy()
    proj[0, r, nu // 2] = bright
    got = ops.pmf_fdk(T(proj), cone, T(ang), grid).cpu().numpy()
    # voxels that read row r in the first view: between rows r - 1 and r + 1
    tau_v = cone.dv * cone.sad / cone.sdd
    x, y, z = (np.asarray(grid.center[a]) + (np.arange(grid.n[a]) - (grid.n[a] - 1) / 2.0) * grid.h[a]
               for a in range(3))
    U = cone.sad - (x[:, None] * np.cos(ang[0]) + y[None, :] * np.sin(ang[0]))
    fv = (cone.sad * z / U[..., None]) / tau_v + 0.5 * (nv - 1) - cone.off_v
    reads = np.abs(fv - r) < 1.001
    assert reads.any() and not reads.all()
    assert np.abs(got[~reads] - clean[~reads]).max() <= 1e-6 * np.abs(clean).max()


def test_a_row_of_zeros_stays_zero():
    """Beside a row of any size: the volume of one large row alone is zero where
    neither it nor its neighbours are read."""
    nu, nv = 96, 40
    grid = Grid((6, 5, 33), (3.0, 3.0, 0.2), (1.0, -2.0, 0.3))
    cone = Cone(1000.0, 1500.0, nu, nv, 40.0 / nu, 40.0 / nv, off_u=0.2, off_v=-0.3)
    ang = synth.evenly_spaced_angles(1)
    U = cone.sad - (np.asarray(grid.center[0]) + (np.arange(6) - 2.5) * 3.0)
    z = grid.center[2] + (np.arange(33) - 16) * 0.2
    fv = (cone.sad * z[None, :] / U[:, None]) / (cone.dv * cone.sad / cone.sdd) + 0.5 * (nv - 1) - cone.off_v
    for r in (20, 21):
        proj = np.zeros((1, nv, nu), np.float32)
        proj[0, r] = synth.projection_like(2, 1, nv, nu)[0, r] * np.float32(1e30)
        got = ops.pmf_fdk(T(proj), cone, T(ang), grid).cpu().numpy()
        reads = np.abs(fv - r) < 1.001
        assert got.any() and not got.transpose(0, 2, 1)[~reads].any()


def test_rows_of_unlike_sizes():
    """A volume of the small rows alone is that of the same rows beside large
    ones: the rows of even index filtered with the others 1e12 times as large."""
    nu, nv, V = 130, 24, 2
    grid = Grid((5, 5, 1 + 2 * 11), (2.0, 2.0, 40.0 / 24 * 1000.0 / 1500.0), (0.0, 0.0, 0.0))
    cone = Cone(1000.0, 1500.0, nu, nv, 40.0 / nu, 40.0 / nv)
    ang = T(synth.evenly_spaced_angles(V))
    proj = synth.projection_like(4, V, nv, nu)
    small = proj.copy()
    small[:, 1::2] = 0.0
    both = small.copy()
    both[:, 1::2] = proj[:, 1::2] * np.float32(1e12)
    large = both.copy()
    large[:, 0::2] = 0.0
    f = lambda p: ops.pmf_fdk(T(p), cone, ang, grid).double()
    a, b, c = f(small), f(both), f(large)
    # back-projection is linear up to float roundings of its largest terms
    assert float((b - c - a).norm()) <= 1e-5 * float(c.norm())
    assert float((f(small * np.float32(1e12)) - a * float(np.float32(1e12))).norm()) <= 1e-6 * 1e12 * float(a.norm())
