"""The DVF layers on both sides of the lines between blocks of outputs and a voxel
per thread, against the FP64 oracle.

Bars: a DVF entry is at most 2 x 3 x 3 fused terms of three lerps (2e-6 in norm), a
basis gradient a sum of at most a few hundred float terms (2e-5), a coefficient
gradient one of every voxel with mixed signs (1e-4).
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


@pytest.mark.parametrize("n,B,V", [
    ((113, 111, 60), 1, 1),     # blocks, one basis
    ((113, 111, 60), 1, 2),
    ((113, 110, 45), 1, 1),     # too few outputs per block forward, enough backward
    ((90, 87, 61), 2, 1),       # blocks, several bases, ragged on every axis
    ((90, 87, 61), 3, 3),       # blocks backward only
    ((90, 87, 30), 2, 1),       # half-empty blocks: a voxel per thread
    ((70, 61, 64), 3, 2),       # few blocks: backward by the views' number
    ((300, 300, 2), 3, 2),      # a thin grid
])
def test_both_routes(n, B, V):
    grid = Grid(n, (1.5, 1.5, 2.0))
    sizes = [tuple(max(2, x // 4) for x in n[:2]) + (max(2, n[2] // 2),), n]
    levels = synth.level_grids(grid, sizes)
    rng = np.random.default_rng(5)
    bases = [rng.normal(0, 2, (3 * B,) + s).astype(np.float32) for s in sizes]
    coeff = rng.normal(0, 1, (V, 2, B, 3)).astype(np.float32)
    g_dvf = rng.normal(0, 1, (V, 3) + n).astype(np.float32)
    tb = [T(b) for b in bases]
    assert rel(ops.pmf_combine_dvf(tb, levels, T(coeff), grid),
               oracle.combine(bases, levels, coeff, grid)) < 2e-6
    gb, gc = ops.pmf_combine_dvf_bwd(tb, levels, T(coeff), grid, T(g_dvf))
    wb, wc = oracle.combine_bwd(bases, levels, coeff, grid, g_dvf)
    assert rel(gc, wc) < 1e-4
    for a, b in zip(gb, wb):
        assert rel(a, b) < 2e-5


@pytest.mark.parametrize("ratio", [4.0, 2.0, 1.2])
def test_blocks_over_a_level_that_goes_on_past_the_output(ratio):
    """What a level holds past a ragged grid of whole and cut blocks changes no bit."""
    grid = Grid((90, 87, 61), (1.0, 1.0, 1.0))
    n = tuple(int(np.ceil((s + 16) / ratio)) for s in grid.n)
    level = Grid(n, (ratio,) * 3, (0.3, -0.2, 0.1))
    rng = np.random.default_rng(1)
    base = rng.normal(0, 1, (6,) + n).astype(np.float32)
    coeff = rng.normal(0, 1, (1, 1, 2, 3)).astype(np.float32)
    g_dvf = rng.normal(0, 1, (1, 3) + grid.n).astype(np.float32)
    keep = np.ones(n, bool)         # the cells that output voxels sample
    for a in range(3):
        x = (np.arange(grid.n[a]) - (grid.n[a] - 1) / 2.0) - level.center[a]
        u = x / ratio + (n[a] - 1) / 2.0
        idx = np.zeros(n[a], bool)
        idx[int(np.floor(u[0] - 0.01)):int(np.floor(u[-1] + 0.01)) + 2] = True
        keep &= idx.reshape([-1 if b == a else 1 for b in range(3)])
    assert not keep.all()
    bad = base.copy()
    bad[:, ~keep] = np.inf
    kept, got = ([ops.pmf_combine_dvf([T(b)], [level], T(coeff), grid),
                 ops.pmf_combine_dvf_bwd([T(b)], [level], T(coeff), grid, T(g_dvf))[1]] for b in (base, bad))
    assert torch.equal(kept[0], got[0])
    assert torch.equal(kept[1], got[1])
