"""The summed back-projection where its workspace with the views' volumes does not
fit: in more rounds, from the views' own parts."""
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


def test_without_room_for_the_volumes(monkeypatch):
    grid = Grid((64, 60, 56), (1.5, 1.4, 2.0))
    cone = Cone(1000.0, 1500.0, 96, 61, 1.9, 2.9)
    V = 6
    ang = torch.tensor(synth.scan_angle(np.arange(V) * 100), dtype=torch.float32, device="cuda")
    gp = torch.randn(V, cone.nv, cone.nu, device="cuda")
    want = ops.pmf_project_bwd(gp, grid, cone, ang, shared=True)
    g, c = ops.make_grid(grid), ops.make_cone(cone)
    need = ops.lib().pmf_project_bwd_workspace(C.byref(g), C.byref(c), V)
    asked = []

    def tight(nbytes, device):
        asked.append(nbytes)
        if nbytes > need:
            raise torch.cuda.OutOfMemoryError("no room")
        return torch.empty(nbytes, dtype=torch.uint8, device=device)

    monkeypatch.setattr(ops, "workspace", tight)
    got = ops.pmf_project_bwd(gp, grid, cone, ang, shared=True)
    assert len(asked) == 2 and asked[1] == need
    # (shorter rounds may take other bricks: 2^-31 of a view's bound per term)
    assert float((got - want).norm()) <= 1e-5 * float(want.norm())
