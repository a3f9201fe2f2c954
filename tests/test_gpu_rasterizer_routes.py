"""The rasterizer at the edges of its chunks of Gaussians, windows of tiles,
tiles, pixel boxes and its list of large splats, against the FP64 oracle
(images 1e-4, gradients 1e-3, as for every rasterizer result; the image also
pixel by pixel, where a dropped splat takes e^(-4.5) ~ 0.011 of its
amplitude)."""
import numpy as np
import pytest
import torch

from oracle import rasterize as R
from paper_2503_22139_amd import ops
from paper_2503_22139_amd.synth import Cone, GaussSet

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    ops.lib()
    yield


def T(a):
    return torch.from_numpy(np.ascontiguousarray(a, np.float32)).cuda()


def N(t):
    return t.detach().cpu().numpy().astype(np.float64)


def splats(seed, m, extent, smin, smax):
    rng = np.random.default_rng(seed)
    c = lambda a: np.asarray(a, np.float32).astype(np.float64)
    return GaussSet(c(rng.uniform(-1.0, 1.0, (m, 3)) * np.asarray(extent)),
                    c(np.exp(rng.uniform(np.log(smin), np.log(smax), (m, 3)))),
                    c(rng.normal(size=(m, 4))), c(rng.uniform(0.02, 0.05, (m, 1))))


def check(gs, cone, angles, k=3.0, pixels=None):
    """Image and gradients, at `pixels` only when given."""
    t = [T(a) for a in (gs.mean, gs.scale, gs.quat, gs.value)]
    ang = T(angles)
    img = N(ops.pmf_rasterize(*t, cone, ang, k))
    V = len(angles)
    rng = np.random.default_rng(1)
    if pixels is None:
        iv, iu = np.meshgrid(np.arange(cone.nv), np.arange(cone.nu), indexing="ij")
        pixels = np.stack([iu.ravel(), iv.ravel()], -1)
    got = img.reshape(V, cone.nv, cone.nu)[:, pixels[:, 1], pixels[:, 0]]
    gp = rng.normal(size=got.shape).astype(np.float32)
    g_proj = np.zeros((V, cone.nv, cone.nu), np.float32)
    g_proj[:, pixels[:, 1], pixels[:, 0]] = gp
    grads = ops.pmf_rasterize_bwd(*t, cone, ang, k, T(g_proj))
    wt = [torch.tensor(a, dtype=torch.float64, requires_grad=True)
          for a in (gs.mean, gs.scale, gs.quat, gs.value)]
    p = R.rasterize_t(*wt, cone, list(angles), k, pixels=pixels)
    want = p.detach().numpy()
    (p * torch.tensor(gp.astype(np.float64))).sum().backward()
    nrm = max(np.linalg.norm(want), 1e-30)
    assert np.linalg.norm(got - want) <= 1e-4 * nrm
    for a, b in zip(grads, wt):
        b = b.grad.numpy()
        assert np.linalg.norm(N(a) - b) <= 1e-3 * np.linalg.norm(b) + 1e-12


# Gaussians around a chunk of 512; views
@pytest.mark.parametrize("m", [1, 511, 512, 513, 1030])
@pytest.mark.parametrize("V", [1, 3])
def test_chunks(m, V):
    print(m, V, flush=True)
    cone = Cone(1000.0, 1500.0, 40, 36, 1.5, 1.5)
    check(splats(m, m, (18, 18, 16), 0.5, 2.0), cone, np.linspace(0.2, 5.0, V))


# detectors around a tile of 16 and a block of 8
@pytest.mark.parametrize("nu,nv", [(1, 1), (8, 9), (15, 17), (16, 16), (33, 7), (7, 33)])
def test_detectors(nu, nv):
    print(nu, nv, flush=True)
    cone = Cone(1000.0, 1500.0, nu, nv, 40.0 / nu, 40.0 / nv, off_u=0.3, off_v=-0.2)
    check(splats(nu, 100, (12, 12, 12), 0.5, 3.0), cone, np.array([0.7, 3.9]))


# boxes: under a pixel, needles, 64 pixels wide and around it, around the
# sixteen tiles that make a splat large, and all pixels
@pytest.mark.parametrize("smin,smax,k", [(0.02, 0.1, 3.0), (0.3, 9.0, 3.0), (6.6, 7.4, 3.0), (6.0, 9.0, 3.0),
                                         (9.0, 25.0, 3.0), (0.5, 4.0, float("inf"))])
def test_boxes(smin, smax, k):
    print(smin, smax, k, flush=True)
    cone = Cone(1000.0, 1500.0, 150, 130, 1.0, 1.0)
    check(splats(3, 80, (40, 40, 35), smin, smax), cone, np.array([1.1]), k)


# a detector of more tiles than one window of counts holds
def test_windows():
    cone = Cone(1000.0, 1500.0, 1808, 1799, 0.25, 0.25)
    gs = splats(4, 600, (130, 130, 130), 0.5, 2.0)
    rng = np.random.default_rng(5)
    pix = np.unique(np.stack([rng.integers(0, cone.nu, 3000), rng.integers(0, cone.nv, 3000)], -1), axis=0)
    check(gs, cone, np.array([0.4]), pixels=pix)
