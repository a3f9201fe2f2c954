"""Many large splats (more than sixteen tiles each), which a tile stages 1,024 at
a time: around that count and over several views, with ordinary ones beside
them, against the FP64 oracle (images 1e-4, gradients 1e-3, as for every
rasterizer result)."""
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


@pytest.mark.parametrize("m,V,k", [(1023, 1, 3.0), (1025, 1, 3.0), (700, 3, 3.0), (600, 2, float("inf"))])
def test_many_large_splats(m, V, k):
    print(m, V, k, flush=True)
    rng = np.random.default_rng(m)
    c = lambda a: np.asarray(a, np.float32).astype(np.float64)
    s = np.exp(rng.uniform(np.log(14.0), np.log(25.0), (m, 3)))
    s[::7] *= 0.05                              # ordinary ones
    gs = [c(rng.uniform(-40.0, 40.0, (m, 3))), c(s), c(rng.normal(size=(m, 4))),
          c(rng.uniform(0.02, 0.05, (m, 1)))]
    cone = Cone(1000.0, 1500.0, 150, 131, 1.0, 1.0)
    angles = np.linspace(0.3, 4.0, V)
    pix = np.unique(np.stack([rng.integers(0, cone.nu, 600), rng.integers(0, cone.nv, 600)], -1), axis=0)
    t = [T(a) for a in gs]
    img = ops.pmf_rasterize(*t, cone, T(angles), k)
    got = N(img)[:, pix[:, 1], pix[:, 0]]
    gp = rng.normal(size=got.shape).astype(np.float32)
    g_proj = np.zeros((V, cone.nv, cone.nu), np.float32)
    g_proj[:, pix[:, 1], pix[:, 0]] = gp
    grads = ops.pmf_rasterize_bwd(*t, cone, T(angles), k, T(g_proj))
    wt = [torch.tensor(a, dtype=torch.float64, requires_grad=True) for a in gs]
    p = R.rasterize_t(*wt, cone, list(angles.astype(np.float32)), k, pixels=pix)
    want = p.detach().numpy()
    (p * torch.tensor(gp.astype(np.float64))).sum().backward()
    assert np.linalg.norm(got - want) <= 1e-4 * np.linalg.norm(want)
    for a, b in zip(grads, wt):
        b = b.grad.numpy()
        assert np.linalg.norm(N(a) - b) <= 1e-3 * np.linalg.norm(b) + 1e-12
    assert torch.equal(ops.pmf_rasterize(*t, cone, T(angles), k), img)
