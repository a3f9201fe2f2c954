"""The fixed-point sums of the warp adjoint's g_ref: both signs alike, and terms
far below the largest |g_out| to their own last kept bit, against the FP64
oracle."""
import numpy as np
import pytest
import torch

import oracle
from paper_2503_22139_amd import ops
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


GRID = Grid((26, 17, 37), (1.0, 1.2, 2.0))


def inputs(seed, size):
    rng = np.random.default_rng(seed)
    h = np.array(GRID.h)[None, :, None, None, None]
    dvf = (rng.uniform(-size, size, (2, 3) + GRID.n) * h).astype(np.float32)
    go = rng.normal(0, 1, (2,) + GRID.n).astype(np.float32)
    ref = rng.uniform(0.5, 1.5, GRID.n).astype(np.float32)
    return ref, dvf, go


# inside the bricks' boxes, and beyond them (the 64-bit volume's atomics)
@pytest.mark.parametrize("size", [0.8, 9.0])
def test_signs_are_alike(size):
    ref, dvf, go = inputs(1, size)
    a = ops.pmf_warp_bwd(T(ref), GRID, T(dvf), T(go))[0]
    b = ops.pmf_warp_bwd(T(ref), GRID, T(dvf), T(-go))[0]
    assert torch.equal(a, -b)


@pytest.mark.parametrize("small", [1e-7, 1e-8, 1e-9])
def test_small_terms_beside_a_large_one(small):
    """Every term is rounded to 2^-40 of the largest |g_out| (here 1, at one
    corner): with at most 16 terms per voxel of errors of either sign below 2^-41,
    beside float products of small size."""
    ref, dvf, go = inputs(2, 0.8)
    go *= np.float32(small)
    go[0, 0, 0, 0] = 1.0
    got = ops.pmf_warp_bwd(T(ref), GRID, T(dvf), T(go))[0].cpu().numpy().astype(np.float64)
    want = oracle.warp_bwd(ref, GRID, dvf, go)[0]
    far = (slice(4, None),) * 3             # displacements stay below one voxel
    err = np.linalg.norm(got[far] - want[far]) / np.linalg.norm(want[far])
    print(small, err, flush=True)
    assert err <= 16 * 2.0 ** -41 / small + 1e-6


def test_infinite_cotangent_gives_zeros():
    """No scale fits an infinite |g_out|: g_ref is zero; a NaN adds nothing."""
    ref, dvf, go = inputs(3, 0.8)
    go[1, 5, 5, 5] = np.nan
    clean = go.copy()
    clean[1, 5, 5, 5] = 0.0
    a = ops.pmf_warp_bwd(T(ref), GRID, T(dvf), T(go))[0]
    assert torch.equal(a, ops.pmf_warp_bwd(T(ref), GRID, T(dvf), T(clean))[0])
    go[0, 3, 3, 3] = -np.inf
    assert not ops.pmf_warp_bwd(T(ref), GRID, T(dvf), T(go))[0].any()
