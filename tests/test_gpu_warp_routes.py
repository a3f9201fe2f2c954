"""The warp adjoint on both sides of the lines between bricks and a voxel per
thread, and bricks that take several rounds."""
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


def rel(a, b):
    a = a.detach().cpu().numpy().astype(np.float64)
    return np.linalg.norm(a - b) / np.linalg.norm(b)


# eleven and twelve bricks; bricks of 3 and of 4 layers; ragged ones
@pytest.mark.parametrize("n", [(88, 8, 32), (90, 8, 32), (81, 60, 3), (81, 60, 4), (33, 31, 35)])
@pytest.mark.parametrize("size", [0.8, 9.0])
def test_routes(n, size):
    print(n, size, flush=True)
    grid = Grid(n, (1.5, 1.2, 2.0))
    rng = np.random.default_rng(7)
    ref = rng.uniform(0.5, 1.5, n).astype(np.float32)
    dvf = (rng.uniform(-size, size, (2, 3) + n) * np.array(grid.h)[None, :, None, None, None]).astype(np.float32)
    go = rng.uniform(0.1, 1.0, (2,) + n).astype(np.float32)
    gr, gd = ops.pmf_warp_bwd(T(ref), grid, T(dvf), T(go))
    wr, wd = oracle.warp_bwd(ref, grid, dvf, go)
    # non-negative terms of four float products each, summed exactly
    assert rel(gr, wr) < 8 * 2.0 ** -24
    assert rel(gd, wd) < 1e-5
    neg = ops.pmf_warp_bwd(T(ref), grid, T(dvf), T(-go))
    assert torch.equal(gr, -neg[0])


def test_rounds_give_the_bits_of_one():
    """138 x 138 bricks in two rounds against the first 88 planes of them in one
    (rows that displacements of up to 9 voxels from beyond the cut do not reach)."""
    n, cut = (1100, 1100, 4), 700
    gen = torch.Generator(device="cuda").manual_seed(3)
    u = lambda *s: torch.rand(s, device="cuda", generator=gen)
    ref = u(*n) + 0.5
    dvf = (2 * u(1, 3, *n) - 1) * 2.0
    dvf[:, 0, ::2] *= 4.5
    go = 2 * u(1, *n) - 1
    go[0, 5, 5, 1] = 1.5                        # the largest, on both grids
    whole = ops.pmf_warp_bwd(ref, Grid(n, (1.0, 1.0, 1.0)), dvf, go)
    part = ops.pmf_warp_bwd(ref[:cut].contiguous(), Grid((cut,) + n[1:], (1.0, 1.0, 1.0)),
                            dvf[:, :, :cut].contiguous(), go[:, :cut].contiguous())
    k = cut - 12
    assert torch.equal(whole[0][:k], part[0][:k])
    assert torch.equal(whole[1][:, :, :k], part[1][:, :, :k])
