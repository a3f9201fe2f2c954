"""Workspaces that a call must not need more of: the sizes that the queries
returned when callers first sized their buffers by them (host arithmetic, no
GPU)."""
import ctypes as C
import os

import pytest

from paper_2503_22139_amd import ops
from paper_2503_22139_amd.synth import Cone, Grid


@pytest.fixture(scope="module")
def lib():
    if not os.path.exists(ops.LIB_PATH):
        from paper_2503_22139_amd import build
        build.build(verbose=False)
    return ops.lib()


@pytest.mark.parametrize("n,nu,nv,V,want", [
    ((256, 256, 128), 512, 384, 1, 52353536), ((256, 256, 128), 512, 384, 8, 418824704),
    ((64, 64, 64), 128, 96, 10, 25705472), ((33, 21, 18), 5, 3, 2, 717824),
    ((512, 512, 512), 64, 64, 4, 2717770240),
])
def test_back_projection(lib, n, nu, nv, V, want):
    """The views' parts alone, whether the call sums over views or not."""
    g, c = ops.make_grid(Grid(n, (0.5, 0.5, 0.5))), ops.make_cone(Cone(1000.0, 1500.0, nu, nv, 1.0, 1.0))
    assert lib.pmf_project_bwd_workspace(C.byref(g), C.byref(c), V) <= want


@pytest.mark.parametrize("n", [(256, 256, 128), (512, 512, 512), (1290, 1290, 1290), (32767, 32767, 2)])
def test_warp_adjoint(lib, n):
    """Eight bytes per voxel and at most 1 GiB, however large or flat the grid."""
    g = ops.make_grid(Grid(n, (0.01, 0.01, 0.01)))
    assert 0 < lib.pmf_warp_bwd_workspace(C.byref(g)) <= 8 * n[0] * n[1] * n[2] + (1 << 30) + 1024
