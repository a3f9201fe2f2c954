"""The motion path's adjoint at the edges of its rounds of 32 views and its
launches of 64, with displacements that stay inside the volume (waves that skip
the rim's cases), reach its rim, and vanish (samples on the voxel centres),
against the FP64 oracle (gradients 1e-3, as for every step)."""
import numpy as np
import pytest
import torch

import oracle
from paper_2503_22139_amd import ops, synth
from paper_2503_22139_amd.model import MotionModel

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    ops.lib()
    yield


def rel(a, b):
    a = a.detach().cpu().numpy().astype(np.float64)
    return np.linalg.norm(a - b) / max(np.linalg.norm(b), 1e-30)


@pytest.mark.parametrize("nviews", [1, 32, 33, 65])
@pytest.mark.parametrize("factor", [0.0, 0.1, 2.0])
def test_rounds(nviews, factor):
    print(nviews, factor, flush=True)
    w = synth.small_motion(seed=70 + nviews, n=(24, 22, 20), nbases=2, nviews=nviews,
                           level_dims=((6, 6, 5), (12, 11, 10), (24, 22, 20)), det=(24, 20), du=4.0)
    w.coeff = (w.coeff * np.float32(factor)).astype(np.float32)
    target = synth.add_target_noise(oracle.forward(synth.perturbed_truth(w)))
    want_loss, want = oracle.step(w, target)
    m = MotionModel(w)
    loss, got = m.step_batched(torch.from_numpy(np.ascontiguousarray(target, np.float32)).cuda())
    assert abs(float(loss) - want_loss) <= 1e-4 * want_loss
    for name in ("mean", "scale", "quat", "value"):
        assert rel(got["ref"][name], want["ref"][name]) < 1e-3, name
        for a, b in zip(got["mbc"], want["mbc"]):
            if factor > 0.0:
                assert rel(a[name], b[name]) < 1e-3, name
    if factor > 0.0:
        assert rel(got["coeff"], want["coeff"]) < 1e-3
