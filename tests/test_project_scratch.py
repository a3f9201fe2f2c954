"""The scratch of ops.pmf_project on the CPU, with a stand-in for the library's
two projection calls: every call has scratch of its own, and none while the
stream is captured or where it does not fit."""
import ctypes as C
import os
import threading

import pytest
import torch

from paper_2503_22139_amd import ops, synth
from paper_2503_22139_amd.synth import Cone, Grid

GRID = Grid((33, 21, 18), (1.5, 1.7, 2.0))
CONE = Cone(1000.0, 1500.0, 512, 293, 0.2, 0.25)       # enough rays for a paired copy


class Lib:
    """The library's host queries, and a record of the projections."""

    def __init__(self, real, meet=None):
        self.real, self.meet, self.calls = real, meet, []

    def __getattr__(self, name):
        return getattr(self.real, name)

    def pmf_project(self, *a):
        self.calls.append(None)
        return ops.PMF_OK

    def pmf_project_ws(self, *a):
        self.calls.append(a[7].value)
        if self.meet:
            self.meet.wait(20)
        return ops.PMF_OK


@pytest.fixture
def project(monkeypatch):
    if not os.path.exists(ops.LIB_PATH):
        from paper_2503_22139_amd import build
        build.build(verbose=False)
    real = ops.lib()

    class Stream:
        cuda_stream = 0

    state = {"capturing": False}
    monkeypatch.setattr(torch.cuda, "current_stream", lambda *a: Stream())
    monkeypatch.setattr(torch.cuda, "is_current_stream_capturing", lambda: state["capturing"])
    monkeypatch.setattr(ops, "_ptr", lambda t: C.c_void_p(t.data_ptr()))
    monkeypatch.setattr(ops, "_ws_cache", {})

    def make(meet=None):
        lib = Lib(real, meet)
        monkeypatch.setattr(ops, "lib", lambda: lib)
        return lib

    vol, ang = torch.zeros(GRID.n), torch.zeros(1)
    return make, lambda: ops.pmf_project(vol, GRID, CONE, ang, shared=True), state


def test_capture_keeps_no_scratch(project):
    """A recorded call holds no address of a buffer that a later call may replace."""
    make, run, state = project
    lib = make()
    ops.workspace(1 << 20, torch.device("cpu"))         # large enough, and at hand
    run()
    assert lib.calls[0] is not None
    state["capturing"] = True
    run()
    assert lib.calls[1] is None


def test_threads_on_one_stream_have_scratch_of_their_own(project):
    make, run, _ = project
    lib = make(threading.Barrier(2))
    ts = [threading.Thread(target=run) for _ in range(2)]
    for t in ts:
        t.start()
    for t in ts:
        t.join()
    assert None not in lib.calls and len(set(lib.calls)) == 2


def test_without_room_the_plain_route_runs(project, monkeypatch):
    make, run, _ = project
    lib = make()
    empty = torch.empty

    def short(*a, **k):
        if k.get("dtype") == torch.uint8:
            raise torch.cuda.OutOfMemoryError("no room")
        return empty(*a, **k)

    monkeypatch.setattr(torch, "empty", short)
    run()
    assert lib.calls == [None]


def test_copies_of_large_volumes_are_bounded(project):
    """Eight at a time, fewer where they would take more than 1 GiB, never below one."""
    make, _, _ = project
    lib = make().real
    for n, copies in (((64, 64, 64), 8), ((512, 512, 256), 2), ((800, 800, 512), 1)):
        g, c = ops.make_grid(Grid(n, (0.5, 0.5, 0.5))), ops.make_cone(Cone(1000.0, 1500.0, 4096, 4096, 0.1, 0.1))
        N = n[0] * n[1] * n[2]
        assert lib.pmf_project_workspace(C.byref(g), C.byref(c), 20, N) == 8 * N * copies
        assert lib.pmf_project_workspace(C.byref(g), C.byref(c), 20, 0) == 8 * N
