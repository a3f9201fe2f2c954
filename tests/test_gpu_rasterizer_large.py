"""The rasterizer beyond one grid dimension's 2^32 threads: a wave per splat
from 2^26 of them on, 1,024 threads per tile from 2^22 tiles on."""
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


GRID = Grid((64, 64, 32), (1.5, 1.5, 2.0))


def test_adjoint_of_2_to_26_splats():
    """2^20 Gaussians in 64 views against the sum of two calls of 32 views
    (doubles over a call's views, rounded to float once per call)."""
    m, V = 1 << 20, 64
    gs = synth.gaussians(np.random.default_rng(1), m, GRID, s_vox=(0.5, 1.0))
    g = [T(x) for x in (gs.mean, gs.scale, gs.quat, gs.value)]
    cone = Cone(1000.0, 1500.0, 16, 16, 9.0, 6.0)
    ang = T(synth.scan_angle(np.arange(V) * 10))
    gp = T(synth.random_normal(2, (V, 16, 16)))
    all_ = ops.pmf_rasterize_bwd(*g, cone, ang, 3.0, gp)
    h = V // 2
    a = ops.pmf_rasterize_bwd(*g, cone, ang[:h], 3.0, gp[:h])
    b = ops.pmf_rasterize_bwd(*g, cone, ang[h:].clone(), 3.0, gp[h:].clone())
    for x, y, z in zip(all_, a, b):
        want = y.double() + z.double()
        assert float(want.norm()) > 0
        assert float((x.double() - want).norm()) <= 1e-6 * float((y.double().abs() + z.double().abs()).norm())


def test_forward_of_2_to_22_tiles():
    """Views repeat, so their pixels do, bit for bit."""
    V = (1 << 22) + 3
    gs = synth.gaussians(np.random.default_rng(1), 4, GRID, s_vox=(4.0, 8.0))
    g = [T(x) for x in (gs.mean, gs.scale, gs.quat, gs.value)]
    cone = Cone(1000.0, 1500.0, 3, 2, 30.0, 30.0)
    base = T(synth.scan_angle(np.arange(7) * 90))
    few = ops.pmf_rasterize(*g, cone, base, 3.0)
    assert float(few.min()) >= 0 and float(few.max()) > 0
    at = torch.arange(V, device="cuda") % 7
    assert torch.equal(ops.pmf_rasterize(*g, cone, base[at], 3.0), few[at])
