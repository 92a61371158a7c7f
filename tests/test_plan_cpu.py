"""The workspace plans (host-only).  No GPU."""
import ctypes
import os
import time

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def size():
    lib = ctypes.CDLL(os.path.join(ROOT, "paper_2007_01088_amd", "libcc3.so"))
    f = lib.cc3_workspace_size
    f.argtypes = [ctypes.c_int] * 4 + [ctypes.c_uint, ctypes.POINTER(ctypes.c_size_t)]

    def call(no, nv, prec=0, flags=0):
        n = ctypes.c_size_t(0)
        assert f(no, nv, 3 * (no + nv), prec, flags, ctypes.byref(n)) == 0
        return n.value
    return call


def test_planning_time_does_not_follow_the_batch(size):
    """Every call plans at least once, before its first launch.  The plan goes over the batch
    sizes of the loop (up to 160 at 31/16, one at 1/16), and the rules that do not depend on the
    batch are evaluated once: 1.6 us more, where evaluating them per batch size took 12."""
    def best(no, nv):
        t = []
        for _ in range(30):
            t0 = time.perf_counter()
            for _ in range(200):
                size(no, nv)
            t.append(time.perf_counter() - t0)
        return min(t) / 200
    assert best(31, 16) - best(1, 16) < 5e-6


# (no, nv, cube budget in MiB): bytes of the plan at nchol = 3 (no + nv) in FP64 with five cube
# slots per triple; a server's requests, whose budget is a share of its arena, fit where they did
SMALL_BUDGET = {
    (3, 119, 128): 427615488, (4, 95, 128): 547965696, (8, 43, 128): 312605184,
    (10, 53, 128): 455077888, (3, 190, 512): 1373221120, (6, 302, 4096): 11227156992}


@pytest.mark.parametrize("no,nv,mb", sorted(SMALL_BUDGET))
def test_small_cube_budget_bounds_the_plan(size, monkeypatch, no, nv, mb):
    monkeypatch.setenv("CC3_CUBE_BUDGET_MB", str(mb))
    assert size(no, nv) <= SMALL_BUDGET[no, nv, mb]
