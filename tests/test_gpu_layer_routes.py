"""The DVF and warp layers at the edges of their blocks and bricks, against the
FP64 oracle and against each other's routes.

Bars: a DVF entry is at most 4 x 4 x 3 fused terms of three lerps each
(48 x 2^-24 relative to their sizes, 3e-6 in norm); a basis or reference
gradient sums at most a few hundred float terms (2e-5); a coefficient gradient
sums every voxel with mixed signs (1e-4).
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


def rel(a, b):
    a = a.detach().cpu().numpy().astype(np.float64).reshape(-1)
    b = np.asarray(b, np.float64).reshape(-1)
    return np.linalg.norm(a - b) / max(np.linalg.norm(b), 1e-300)


# output size, level sizes (same field of view unless given as a Grid), B
LEVELS = {
    "ratios 4, 2, 1": ((32, 24, 128), [(8, 6, 64), (16, 12, 128), (32, 24, 128)], 3),
    "ragged": ((37, 30, 67), [(9, 7, 33), (18, 15, 67), (37, 30, 67)], 1),
    "one voxel past a block": ((33, 29, 65), [(8, 7, 32), (33, 29, 65)], 2),
    "smallest": ((2, 2, 2), [(2, 2, 2)], 1),
    "coarse by 1.3": ((26, 26, 20), [(20, 20, 15), (25, 26, 20)], 2),
    "finer than the output": ((12, 10, 9), [(24, 20, 18), (6, 5, 9)], 1),
    "smaller than the output": ((28, 24, 20), [Grid((7, 6, 5), (3.0, 3.0, 4.0), (4.0, -3.0, 2.0)),
                                                Grid((14, 12, 20), (3.0, 3.0, 2.0))], 1),
    "own spacing, shifted": ((20, 18, 16), [Grid((20, 18, 16), (1.5, 1.5, 2.0), (0.7, 0.2, -0.9))], 4),
}


def setup(name, V, seed=3):
    n, lv, B = LEVELS[name]
    grid = Grid(n, (1.5, 1.5, 2.0))
    levels = [g if isinstance(g, Grid) else synth.level_grids(grid, [g])[0] for g in lv]
    rng = np.random.default_rng(seed)
    bases = [rng.normal(0, 2, (3 * B,) + tuple(g.n)).astype(np.float32) for g in levels]
    coeff = rng.normal(0, 1, (V, len(levels), B, 3)).astype(np.float32)
    g_dvf = rng.normal(0, 1, (V, 3) + n).astype(np.float32)
    return grid, levels, bases, coeff, g_dvf


@pytest.mark.parametrize("V", [1, 2, 3])
@pytest.mark.parametrize("name", sorted(LEVELS))
def test_dvf_and_its_adjoint(name, V):
    print(name, V, flush=True)
    grid, levels, bases, coeff, g_dvf = setup(name, V)
    tb = [T(b) for b in bases]
    dvf = ops.pmf_combine_dvf(tb, levels, T(coeff), grid)
    assert rel(dvf, oracle.combine(bases, levels, coeff, grid)) < 3e-6
    gb, gc = ops.pmf_combine_dvf_bwd(tb, levels, T(coeff), grid, T(g_dvf))
    wb, wc = oracle.combine_bwd(bases, levels, coeff, grid, g_dvf)
    assert rel(gc, wc) < 1e-4
    for a, b in zip(gb, wb):
        assert rel(a, b) < 2e-5


@pytest.mark.parametrize("name", sorted(LEVELS))
def test_blocks_give_the_per_voxel_bits(name):
    """One and two views take the block kernel, three the per-voxel one."""
    grid, levels, bases, coeff, _ = setup(name, 3)
    tb = [T(b) for b in bases]
    three = ops.pmf_combine_dvf(tb, levels, T(coeff), grid)
    for v in range(3):
        one = ops.pmf_combine_dvf(tb, levels, T(coeff[v:v + 1]), grid)
        assert torch.equal(one[0], three[v]), v
    assert torch.equal(ops.pmf_combine_dvf(tb, levels, T(coeff[:2]), grid), three[:2])


def test_sample_on_a_voxel_ignores_its_neighbours():
    """On a level's own grid an interior voxel is read alone, whatever its
    neighbours hold."""
    grid = Grid((12, 10, 70), (1.5, 1.5, 2.0))
    b = np.ones((3,) + grid.n, np.float32)
    b[:, 5, 5, 30] = np.inf
    b[:, 2, 7, 64] = np.nan
    dvf = ops.pmf_combine_dvf([T(b)], [grid], T(np.ones((1, 1, 1, 3))), grid)[0].cpu().numpy()
    inner = dvf[:, :-1, :-1, :-1]
    assert np.isinf(inner).sum() == 3 and np.isnan(inner).sum() == 3
    assert np.all(inner[np.isfinite(inner)] == 1.0)


# sizes at the edges of the 8 x 8 x 32 bricks; displacements in voxels: inside
# the 3-voxel halo, at it, and beyond it
@pytest.mark.parametrize("n", [(2, 2, 2), (8, 8, 32), (9, 9, 33), (7, 17, 31), (16, 24, 70)])
@pytest.mark.parametrize("size", [0.8, 3.0, 9.0])
def test_warp_adjoint(n, size):
    print(n, size, flush=True)
    grid = Grid(n, (1.5, 1.2, 2.0), (3.0, 0.0, 1.0))
    V = 3
    rng = np.random.default_rng(7)
    ref = rng.uniform(0.5, 1.5, n).astype(np.float32)
    dvf = (rng.uniform(-size, size, (V, 3) + n) * np.array(grid.h)[None, :, None, None, None]).astype(np.float32)
    go = rng.uniform(0.1, 1.0, (V,) + n).astype(np.float32)
    gr, gd = ops.pmf_warp_bwd(T(ref), grid, T(dvf), T(go))
    wr, wd = oracle.warp_bwd(ref, grid, dvf, go)
    # non-negative terms of four float products each, summed exactly
    assert rel(gr, wr) < 8 * 2.0 ** -24
    assert rel(gd, wd) < 1e-5
    again = ops.pmf_warp_bwd(T(ref), grid, T(dvf), T(go))
    assert torch.equal(gr, again[0]) and torch.equal(gd, again[1])


@pytest.mark.parametrize("scale", [0.0, 1e-30, 1e30])
def test_warp_adjoint_scale(scale):
    """The fixed-point scale follows the largest |g_out| over its whole range."""
    grid = Grid((9, 8, 40), (1.0, 1.0, 1.0))
    rng = np.random.default_rng(9)
    dvf = rng.uniform(-1, 1, (1, 3) + grid.n).astype(np.float32)
    go = rng.uniform(0.1, 1.0, (1,) + grid.n).astype(np.float32)
    ref = T(rng.uniform(0.5, 1.5, grid.n))
    one = ops.pmf_warp_bwd(ref, grid, T(dvf), T(go))[0].double()
    got = ops.pmf_warp_bwd(ref, grid, T(dvf), T(go * np.float32(scale)))[0].double()
    want = one * float(np.float32(scale))
    assert float((got - want).norm()) <= 8 * 2.0 ** -24 * float(want.norm())
