"""Projections whose calls overlap: a recorded one replayed among eager calls
that take more scratch, and two host threads on one stream."""
import threading

import numpy as np
import pytest
import torch

from paper_2503_22139_amd import ops, synth
from paper_2503_22139_amd.synth import Cone, Grid

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    ops.lib()
    yield


def T(a):
    return torch.from_numpy(np.ascontiguousarray(a, np.float32)).cuda()


GRID = Grid((33, 21, 18), (1.5, 1.7, 2.0), (3.0, -2.0, 1.0))
BIG = Grid((130, 110, 64), (0.5, 0.5, 0.9))
CONE = Cone(1000.0, 1500.0, 512, 293, 90.0 / 512, 70.0 / 293, off_u=0.3)


def test_replay_among_larger_eager_calls():
    ang, vol = T([0.3]), T(synth.random_volume(5, GRID.n))
    big = T(synth.random_volume(6, (4,) + BIG.n))
    angs = T([0.1, 0.7, 1.9, 3.0])
    stream = torch.cuda.Stream()
    stream.wait_stream(torch.cuda.current_stream())
    arena = ops.Arena()
    with torch.cuda.stream(stream):
        with ops.use_arena(arena):
            ops.pmf_project(vol, GRID, CONE, ang)
        arena.freeze()
        stream.synchronize()
        res = {}

        def record():
            with ops.use_arena(arena):
                res["out"] = ops.pmf_project(vol, GRID, CONE, ang)

        graph = ops.Graph(record, stream)
        want_big = ops.pmf_project(big, BIG, CONE, angs).clone()
        for k in range(4):
            vol.copy_(T(synth.random_volume(10 + k, GRID.n)))
            eager = ops.pmf_project(vol, GRID, CONE, ang).clone()
            res["out"].zero_()
            ops.workspace((k + 1) << 22, vol.device)    # the stream's buffer is replaced
            graph.replay()
            assert torch.equal(ops.pmf_project(big, BIG, CONE, angs), want_big)
            stream.synchronize()
            assert torch.equal(res["out"], eager), k
        graph.close()


def test_two_threads_on_one_stream():
    ang = T([0.3])
    vols = [T(synth.random_volume(20 + i, GRID.n)) for i in range(2)]
    want = [ops.pmf_project(v, GRID, CONE, ang).clone() for v in vols]
    torch.cuda.synchronize()
    stream = torch.cuda.Stream()
    bad = []

    def run(i):
        with torch.cuda.stream(stream):
            outs = [ops.pmf_project(vols[i], GRID, CONE, ang) for _ in range(50)]
        stream.synchronize()
        bad.extend(k for k, o in enumerate(outs) if not torch.equal(o, want[i]))

    ts = [threading.Thread(target=run, args=(i,)) for i in range(2)]
    for t in ts:
        t.start()
    for t in ts:
        t.join()
    assert not bad
