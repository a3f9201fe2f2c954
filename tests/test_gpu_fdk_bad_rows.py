"""Values that are not finite in the FDK filter's row pairs, of every kind and in
either row: the rows beside them keep their values, for transforms by a part of
a wave, a wave and several waves."""
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


def kinds(volume):
    return np.isnan(volume), np.isposinf(volume), np.isneginf(volume)


@pytest.mark.parametrize("nu", [20, 96, 512, 1100])
@pytest.mark.parametrize("bad", [np.inf, -np.inf, np.nan])
@pytest.mark.parametrize("rows", [(20,), (21,), (20, 21), (7, 12, 13)])
def test_other_rows_keep_their_values(nu, bad, rows):
    print(nu, bad, rows, flush=True)
    nv = 40
    grid = Grid((6, 5, 63), (3.0, 3.0, 0.3), (1.0, -2.0, 0.3))
    cone = Cone(1000.0, 1500.0, nu, nv, 40.0 / nu, 40.0 / nv, off_u=0.2, off_v=-0.3)
    ang = synth.evenly_spaced_angles(1)
    proj = synth.projection_like(1, 1, nv, nu)
    clean = ops.pmf_fdk(T(proj), cone, T(ang), grid).cpu().numpy()
    for r in rows:
        proj[0, r, nu // 3] = bad
        proj[0, r, nu // 2] = bad
    got = ops.pmf_fdk(T(proj), cone, T(ang), grid).cpu().numpy()
    x, z = (np.asarray(grid.center[a]) + (np.arange(grid.n[a]) - (grid.n[a] - 1) / 2.0) * grid.h[a] for a in (0, 2))
    fv = (cone.sad * z[None, :] / (cone.sad - x)[:, None]) / (cone.dv * cone.sad / cone.sdd) + 0.5 * (nv - 1) \
        - cone.off_v
    near = np.min([np.abs(fv - r) for r in rows], axis=0)
    got, clean = got.transpose(0, 2, 1), clean.transpose(0, 2, 1)
    assert np.abs(got[near > 1.001] - clean[near > 1.001]).max() <= 1e-6 * np.abs(clean).max()
    assert not np.isfinite(got[near < 0.999]).any()
