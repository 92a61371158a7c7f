"""The workspace plans (host-only).  No GPU."""
import ctypes
import os
import time

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SCRATCH = 256 << 20      # the allocation-free call's array
CALLER_STREAM = 1 << 30  # the plan of that call (PLAN_CALLER_STREAM)


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


NO = (2, 3, 4, 6, 8, 10, 12, 16, 18, 24, 31, 40, 63)
# Largest nv per no, at nchol = 3 (no + nv), of a loop on two streams with five cubes per
# triple and integral blocks without padding; every smaller nv fitted too.
TAKEN = {
    (0, 0): (104, 101, 97, 91, 86, 81, 77, 69, 66, 56, 46, 36, 19),
    (1, 0): (103, 98, 95, 88, 82, 77, 73, 65, 62, 53, 43, 33, 17),
    (1, 8): (98, 95, 90, 83, 78, 72, 68, 61, 58, 49, 41, 32, 17),
    (2, 0): (103, 98, 95, 88, 82, 77, 73, 65, 62, 53, 43, 33, 17),
    (2, 8): (96, 92, 88, 81, 76, 72, 67, 61, 57, 48, 40, 32, 16),
    (3, 0): (102, 97, 94, 87, 81, 75, 71, 64, 61, 51, 42, 32, 16),
    (3, 8): (94, 88, 85, 79, 72, 68, 64, 57, 55, 46, 38, 29, 16)}


@pytest.mark.parametrize("prec,flags", sorted(TAKEN))
def test_allocation_free_call_takes_these_sizes(size, monkeypatch, prec, flags):
    monkeypatch.setenv("CC3_BATCH", "1")  # one triple per batch: the least it can do with
    for no, top in zip(NO, TAKEN[prec, flags]):
        for nv in range(1, top + 1):
            assert size(no, nv, prec, flags | CALLER_STREAM) <= SCRATCH, (no, nv)


def test_transition_density_sizes():
    lib = ctypes.CDLL(os.path.join(ROOT, "paper_2007_01088_amd", "libcc3.so"))
    best, least = ctypes.c_size_t(0), ctypes.c_size_t(0)
    fb, fl = lib.cc3_transition_density_workspace_size, lib.cc3_transition_density_workspace_min
    for f in (fb, fl):
        f.argtypes = [ctypes.c_int] * 3 + [ctypes.POINTER(ctypes.c_size_t)]
    for no, nv in ((1, 64), (2, 9), (12, 120), (16, 150), (40, 60), (63, 400)):
        assert fb(no, nv, 3 * (no + nv), ctypes.byref(best)) == 0
        assert fl(no, nv, 3 * (no + nv), ctypes.byref(least)) == 0
        if no in (1, 63):  # nothing to keep between pairs; cubes beyond 64 GiB
            assert least.value == best.value
        else:
            assert least.value < best.value
    # the loop by pairs at 12/120: 1.1 GB
    assert fl(12, 120, 400, ctypes.byref(least)) == 0 and least.value < 1.2e9
    for bad in ((0, 9, 9), (4, 401, 9), (4, 9, 0)):
        assert fl(*bad, ctypes.byref(least)) == -1
    assert fl(4, 9, 9, None) == -1
