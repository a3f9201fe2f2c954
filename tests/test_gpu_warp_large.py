"""The warp adjoint of grids whose bricks take several rounds."""
import numpy as np
import pytest
import torch

from paper_2503_22139_amd import ops
from paper_2503_22139_amd.synth import Grid

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    ops.lib()
    yield


def test_rounds_give_the_bits_of_one():
    """138 x 138 bricks in two rounds against the first 88 planes of them in one:
    integer sums with one scale, so equal bits up to the rows that displacements
    from beyond the cut can reach (at most 9 voxels); inside the boxes' halo and
    beyond it."""
    n, cut = (1100, 1100, 2), 700
    gen = torch.Generator(device="cuda").manual_seed(3)
    u = lambda *s: torch.rand(s, device="cuda", generator=gen)
    ref = u(*n) + 0.5
    dvf = (2 * u(2, 3, *n) - 1) * 2.0
    dvf[1] *= 4.5
    go = 2 * u(2, *n) - 1
    go[0, 5, 5, 1] = 1.5                        # the largest, on both grids
    whole = ops.pmf_warp_bwd(ref, Grid(n, (1.0, 1.0, 1.0)), dvf, go)
    c = (cut,) + n[1:]
    part = ops.pmf_warp_bwd(ref[:cut].contiguous(), Grid(c, (1.0, 1.0, 1.0)), dvf[:, :, :cut].contiguous(),
                            go[:, :cut].contiguous())
    k = cut - 12
    assert torch.equal(whole[0][:k], part[0][:k])
    assert torch.equal(whole[1][:, :, :k], part[1][:, :, :k])
    # the rows past the first round, as the first ones of a grid of their own
    lo = 600
    go[0, n[0] - 5, 5, 1] = 1.5
    whole = ops.pmf_warp_bwd(ref, Grid(n, (1.0, 1.0, 1.0)), dvf, go)
    part = ops.pmf_warp_bwd(ref[lo:].contiguous(), Grid((n[0] - lo,) + n[1:], (1.0, 1.0, 1.0)),
                            dvf[:, :, lo:].contiguous(), go[:, lo:].contiguous())
    assert torch.equal(whole[0][lo + 12:], part[0][12:])
