"""A tile's splats in four parts or one: the same bits (the sums are of integers,
with a scale that does not depend on the parts), and tiles that no splat reaches."""
import numpy as np
import pytest
import torch

from oracle import rasterize as R
from paper_2503_22139_amd import ops
from paper_2503_22139_amd.synth import Cone

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    ops.lib()
    yield


def T(a):
    return torch.from_numpy(np.ascontiguousarray(a, np.float32)).cuda()


def splats(m, lo, hi):
    rng = np.random.default_rng(m)
    return [T(rng.uniform(lo, hi, (m, 3))), T(np.exp(rng.uniform(-1.0, 0.7, (m, 3)))), T(rng.normal(size=(m, 4))),
            T(rng.uniform(0.02, 0.05, (m, 1)))]


# 12 tiles a view: parts from 480 Gaussians and up to 85 views on
@pytest.mark.parametrize("m", [479, 480, 3000])
def test_a_view_alone_and_among_many(m):
    cone = Cone(1000.0, 1500.0, 61, 47, 1.0, 1.0)
    t = splats(m, -15.0, 15.0)
    angles = np.linspace(0.2, 6.0, 86)
    many = ops.pmf_rasterize(*t, cone, T(angles))
    for n in (1, 85):
        assert torch.equal(ops.pmf_rasterize(*t, cone, T(angles[:n])), many[:n])


@pytest.mark.parametrize("m", [20, 2000])
def test_empty_tiles(m):
    """Splats in one corner of the detector; the other tiles hold zeros."""
    cone = Cone(1000.0, 1500.0, 90, 70, 1.0, 1.0)
    t = splats(m, (-3.0, 18.0, 12.0), (3.0, 22.0, 16.0))
    img = ops.pmf_rasterize(*t, cone, T([0.0]), out=torch.full((1, 70, 90), 7.0, device="cuda"))
    want = R.rasterize_t(*(a.cpu().double() for a in t), cone, [0.0], 3.0).numpy().reshape(1, 70, 90)
    assert (want == 0).mean() > 0.5
    got = img.cpu().numpy().astype(np.float64)
    assert np.all(got[want == 0] == 0)
    assert np.linalg.norm(got - want) <= 1e-4 * np.linalg.norm(want)
