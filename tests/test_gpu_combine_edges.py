"""The DVF layers past the edges of the output grid: level values that no output
voxel samples, and the largest flat grid."""
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


@pytest.mark.parametrize("ratio", [4.0, 2.0, 1.2])
@pytest.mark.parametrize("V", [1, 3])
def test_a_level_that_goes_on_past_the_output(ratio, V):
    """Blocks of four outputs reach past a grid of 5 x 6 x 7; what the level holds
    there stays out of the coefficients' gradient."""
    grid = Grid((5, 6, 7), (1.0, 1.0, 1.0))
    n = tuple(int(np.ceil(24 / ratio)) for _ in range(3))
    level = Grid(n, (ratio,) * 3, (0.3, -0.2, 0.1))
    rng = np.random.default_rng(1)
    base = rng.normal(0, 1, (3,) + n).astype(np.float32)
    coeff = rng.normal(0, 1, (V, 1, 1, 3)).astype(np.float32)
    g_dvf = rng.normal(0, 1, (V, 3) + grid.n).astype(np.float32)
    # the cells that output voxels sample
    keep = np.ones(n, bool)
    for a in range(3):
        x = (np.arange(grid.n[a]) - (grid.n[a] - 1) / 2.0) - level.center[a]
        u = x / ratio + (n[a] - 1) / 2.0
        idx = np.zeros(n[a], bool)
        idx[int(np.floor(u[0] - 0.01)):int(np.floor(u[-1] + 0.01)) + 2] = True
        keep &= idx.reshape([-1 if b == a else 1 for b in range(3)])
    assert not keep.all()
    bad = base.copy()
    bad[:, ~keep] = np.inf
    want = oracle.combine_bwd([base], [level], coeff, grid, g_dvf)[1]
    got = ops.pmf_combine_dvf_bwd([T(bad)], [level], T(coeff), grid, T(g_dvf))[1].cpu().numpy()
    assert np.linalg.norm(got - want) <= 1e-4 * np.linalg.norm(want)
    dvf = ops.pmf_combine_dvf([T(bad)], [level], T(coeff), grid).cpu().numpy()
    ref = oracle.combine([base], [level], coeff, grid)
    assert np.linalg.norm(dvf - ref) <= 3e-6 * np.linalg.norm(ref)


def test_the_largest_flat_grid():
    """2^26 blocks of output columns: a linear field over 32767 x 32767 x 2."""
    n = 32767
    grid = Grid((n, n, 2), (1.0, 1.0, 1.0))
    level = Grid((2, 2, 2), (n - 1.0, n - 1.0, 1.0))
    x = np.array([0.0, 1.0], np.float32)
    base = np.stack([np.broadcast_to(x[:, None, None], (2, 2, 2)), np.broadcast_to(x[None, :, None], (2, 2, 2)),
                     np.broadcast_to(x[None, None, :], (2, 2, 2))])
    dvf = ops.pmf_combine_dvf([T(base)], [level], T(np.ones((1, 1, 1, 3))), grid)[0]
    rng = np.random.default_rng(2)
    i, j = (torch.from_numpy(np.concatenate([rng.integers(0, n, 4000), [0, n - 1]])).cuda() for _ in range(2))
    for k in range(2):
        for a, at in enumerate((i, j)):
            want = at.double() / (n - 1)
            assert float((dvf[a, i, j, k].double() - want).abs().max()) <= 1e-3
        assert float((dvf[2, i, j, k] - k).abs().max()) <= 1e-3
