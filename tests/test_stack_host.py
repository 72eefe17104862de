"""What SliceStack hands to the library, looked at without a GPU: CPU tensors pass for device tensors and a recording
stand-in takes the calls, so arguments can be checked that must never reach a kernel."""
import ctypes
import types

import pytest
import torch

from paper_2408_11500_amd import binding as B
from paper_2408_11500_amd.stack import SliceStack

N, K, FIRST, HS, L = 70, 3, 40, 32, 2


class Recorder:
    """Stands in for the loaded library: workspace queries give 256 bytes, every other call is recorded and succeeds."""

    def __init__(self):
        self.calls = []

    def __getattr__(self, name):
        if name.endswith("_workspace_bytes"):
            return lambda *a: 256

        def call(*a):
            if name in ("slicegcn_layers_fwd", "slicegcn_layers_bwd"):
                group = B.LayerGroup.from_buffer_copy(a[1]._obj)
                io = (B.LayerIo * group.count).from_address(ctypes.addressof(a[2]._obj) + self.first * ctypes.sizeof(B.LayerIo))
                self.calls.append((name, group, [B.LayerIo.from_buffer_copy(x) for x in io]))
            else:
                self.calls.append((name, a))
            return 0
        return call

    def layers(self, name):
        return [(g, io) for n, g, io in [c for c in self.calls if c[0] == f"slicegcn_layers_{name}"]]


@pytest.fixture
def rec(monkeypatch):
    r = Recorder()
    monkeypatch.setattr(torch.Tensor, "is_cuda", True)
    monkeypatch.setattr(B, "lib", lambda: r)
    monkeypatch.setattr(B, "_stream", lambda: 0)
    for name in ("slicegcn_layers_fwd", "slicegcn_layers_bwd"):   # byref(io, offset) does not tell its offset

        def wrapped(g, group, io, first, ws, inner=getattr(B, name)):
            r.first = first
            inner(g, group, io, first, ws)
        monkeypatch.setattr(B, name, wrapped)
    return r


def stack(**kw):
    g = types.SimpleNamespace(handle=1, view=lambda: types.SimpleNamespace(nnz=10))
    st = SliceStack(g, N, kw.pop("k", K), FIRST, HS, kw.pop("layers", L), device="cpu", **kw)
    for i in range(st.k):
        for l, (wi, wo) in enumerate(st.widths):
            st.set_params(i, l, torch.randn(wi, wo), torch.randn(wo), torch.randn(wi, wo), torch.randn(wo))
    return st


def test_backward_checks_every_gradient(rec):
    """A gradient at the address and row stride of the one before it is looked at all the same."""
    st, w = stack(), K * HS
    st.forward()
    buf = torch.randn(N, 2 * w)
    st.backward(buf[:, :w])
    good = len(rec.calls)
    for bad in (buf[:, ::2],                                # the columns of another matrix
                buf.view(torch.int32)[:, :w],               # whole numbers
                buf.view(torch.bfloat16).as_strided((N, w), (2 * w, 1))):   # half the bytes
        assert bad.data_ptr() == buf.data_ptr()
        with pytest.raises(TypeError):
            st.backward(bad)
    assert len(rec.calls) == good
    st.backward(buf[:, w:])
    group, io = rec.layers("bwd")[-L]                       # the last layer runs first
    assert group.ldgo == 2 * w
    assert [x.dHout for x in io] == [buf[:, w:].data_ptr() + 4 * i * HS for i in range(K)]
