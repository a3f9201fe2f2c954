"""The FDK filter's slots of two rows (few rows in a call) and of eight: row
counts around a slot's eight, against each other."""
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


@pytest.mark.parametrize("nv", [13, 15, 16, 17])
@pytest.mark.parametrize("nu,more", [(512, 500), (900, 500), (96, 2400)])
def test_slots_of_two_and_of_eight(nv, nu, more):
    """Three views alone, and followed by views of zeros, which change the weight
    (pi / V) and the slots; a row's partner in the transform is the same."""
    print(nv, nu, flush=True)
    grid = Grid((9, 8, 21), (3.0, 3.0, 1.0), (1.0, -2.0, 0.3))
    cone = Cone(1000.0, 1500.0, nu, nv, 60.0 / nu, 40.0 / nv, off_u=0.2, off_v=-0.3)
    ang = synth.evenly_spaced_angles(3)
    proj = synth.projection_like(1, 3, nv, nu)
    few = ops.pmf_fdk(T(proj), cone, T(ang), grid).double()
    V = 3 + more * 8 * 6 // nv
    p = torch.zeros((V, nv, nu), device="cuda")
    p[:3] = T(proj)
    a = T(np.concatenate([ang, np.full(V - 3, 0.4)]))
    many = ops.pmf_fdk(p, cone, a, grid).double() * (V / 3.0)
    assert float(few.abs().max()) > 0
    assert float((many - few).abs().max()) <= 1e-6 * float(few.abs().max())
