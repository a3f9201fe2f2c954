"""Gaussians past the bins' capacity, staged 64 at a time by every tile, against
the FP64 oracle.

Bar: an entry of Sigma^-1 carries a few 2^-24 (s_max / s_min)^2, below 4e-6 here,
of m <= 10 where a term counts, and at most 130 terms are added in float: 3e-5 in
norm.
"""
import numpy as np
import pytest
import torch

import oracle
from paper_2503_22139_amd import ops, synth
from paper_2503_22139_amd.synth import Grid

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    ops.lib()
    oracle.build()
    yield


def T(a):
    return torch.from_numpy(np.ascontiguousarray(a, np.float32)).cuda()


# grids of few small tiles, of few whole ones, and (three channels) of many; whole
# chunks and one more; channel counts with and without a kernel of their own
@pytest.mark.parametrize("n,c,m", [
    ((33, 30, 35), 1, 64), ((33, 30, 35), 1, 65), ((33, 30, 35), 3, 130), ((33, 30, 35), 9, 65),
    ((33, 30, 35), 2, 65), ((33, 30, 35), 16, 3), ((66, 130, 66), 1, 65), ((66, 130, 66), 3, 65),
    ((70, 130, 130), 3, 65), ((66, 70, 130), 9, 64),
])
def test_large_gaussians(n, c, m):
    print(n, c, m, flush=True)
    grid = Grid(n, (1.5, 1.2, 2.0), (3.0, -1.0, 0.5))
    rng = np.random.default_rng(13)
    big = synth.gaussians(rng, m, grid, s_vox=(14.0, 24.0), c=c, **({} if c == 1 else dict(value_sigma=1.0)))
    got = ops.pmf_voxelize(T(big.mean), T(big.scale), T(big.quat), T(big.value), grid, float("inf"))
    want = oracle.voxelize(big, grid, float("inf"))
    err = np.linalg.norm(got.cpu().numpy().astype(np.float64).reshape(-1) - np.asarray(want).reshape(-1))
    assert err <= 3e-5 * np.linalg.norm(want)
    again = ops.pmf_voxelize(T(big.mean), T(big.scale), T(big.quat), T(big.value), grid, float("inf"))
    assert torch.equal(got, again)
