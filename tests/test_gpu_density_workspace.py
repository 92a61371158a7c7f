"""The transition density with less memory than its fastest loop wants: the least workspace
that the library reports is enough, the binding takes it where the device has no more, and a
large buffer does not stay with the Context.  Both loops sum the same FP64 terms in other orders:
the parity bar, 1e-11."""
import weakref

import numpy as np
import pytest
import torch

from paper_2007_01088_amd import cc3
from paper_2007_01088_amd.synth import make_inputs, make_left_inputs

pytestmark = pytest.mark.gpu
TOL = 1e-11


def inputs(no, nv, nJ):
    d, lf = make_inputs(no, nv, nJ, tag=51), make_left_inputs(no, nv, tag=51)
    g = [torch.from_numpy(np.ascontiguousarray(d[k])).cuda() for k in ("eps", "L", "t1", "t2")]
    return g + [torch.from_numpy(lf[k]).cuda() for k in ("l1", "l2")], lf["omega"]


def sizes(no, nv, nJ):
    out = []
    for f in (cc3._lib.cc3_transition_density_workspace_size,
              cc3._lib.cc3_transition_density_workspace_min):
        n = cc3._c_size(0)
        assert f(no, nv, nJ, cc3.ctypes.byref(n)) == cc3.OK
        out.append(n.value)
    return out


def same(a, b):
    for x, y in zip(a, b):
        assert float((x - y).norm()) <= TOL * float(y.norm())


@pytest.mark.parametrize("no,nv,nJ", [(2, 9, 12), (4, 20, 30), (7, 33, 40), (17, 12, 24)])
def test_least_workspace(no, nv, nJ):
    g, omega = inputs(no, nv, nJ)
    ctx = cc3.Context(0)
    ref = ctx.transition_density(*g, omega, want_yo=True)
    best, least = sizes(no, nv, nJ)
    assert least < best
    ws = torch.empty(least, dtype=torch.uint8, device="cuda")
    out = [torch.full_like(x, float("nan")) for x in ref]
    call = [ctx._h, no, nv, nJ] + [x.data_ptr() for x in g] + [float(omega)]
    call += [x.data_ptr() for x in out] + [0, ws.data_ptr()]
    st = torch.cuda.current_stream().cuda_stream
    assert cc3._td(*call, least - 1, st) == cc3.E_NOMEM
    assert cc3._td(*call, least, st) == cc3.OK, cc3.last_error()
    same(out, ref)
    ctx.close()


@pytest.mark.parametrize("fails", ["reported", "allocation"])
def test_binding_takes_the_least_where_memory_is_short(fails, monkeypatch):
    no, nv, nJ = 5, 21, 30
    g, omega = inputs(no, nv, nJ)
    ref = cc3.Context(0).transition_density(*g, omega, want_yo=True)
    best, least = sizes(no, nv, nJ)
    ctx = cc3.Context(0)
    if fails == "reported":
        held = torch.cuda.memory_reserved(0) - torch.cuda.memory_allocated(0)
        monkeypatch.setattr(torch.cuda, "mem_get_info", lambda d: (best - held - 1, 1 << 40))
    else:
        real = cc3.Context.workspace

        def workspace(self, n):
            if n >= best:
                self._ws = None
                raise torch.OutOfMemoryError("no piece of that size")
            return real(self, n)
        monkeypatch.setattr(cc3.Context, "workspace", workspace)
    got = ctx.transition_density(*g, omega, want_yo=True)
    assert ctx._ws.numel() < best
    same(got, ref)


def test_large_buffer_is_given_back(monkeypatch):
    no, nv, nJ = 6, 40, 60
    g, omega = inputs(no, nv, nJ)
    ctx = cc3.Context(0)
    ref = ctx.transition_density(*g, omega, want_yo=True)
    assert ctx._ws is not None  # small enough to keep
    monkeypatch.setattr(cc3, "KEEP_WORKSPACE", 1 << 20)
    side = torch.cuda.Stream()
    for stream in (None, side, side.cuda_stream):
        c2 = cc3.Context(0)
        torch.cuda.synchronize()
        got = c2.transition_density(*g, omega, want_yo=True, stream=stream)
        assert c2._ws is None
        # memory of that size, handed out at once on this stream, is not the buffer while
        # `stream` still works in it
        torch.full((sizes(no, nv, nJ)[0] // 8,), float("nan"), dtype=torch.float64, device="cuda")
        torch.cuda.synchronize()
        same(got, ref)
    # a buffer that was there before the call stays
    keep = ctx._ws
    ctx.transition_density(*g, omega)
    assert ctx._ws is keep


def test_outgrown_buffer_is_freed_first(monkeypatch):
    no, nv, nJ = 5, 21, 30
    g, omega = inputs(no, nv, nJ)
    ctx = cc3.Context(0)
    old = weakref.ref(ctx.workspace(4096))
    alive = []
    empty = torch.empty

    def spy(*a, **k):
        if k.get("dtype") is torch.uint8:
            alive.append(old() is not None)
        return empty(*a, **k)
    monkeypatch.setattr(torch, "empty", spy)
    ctx.transition_density(*g, omega)
    assert alive == [False]
