"""What SliceStack hands to the library, looked at without a GPU: CPU tensors pass for device tensors and a recording
stand-in takes the calls, so arguments can be checked that must never reach a kernel."""
import contextlib
import ctypes
import types

import pytest
import torch

from paper_2408_11500_amd import binding as B
from paper_2408_11500_amd import stack as stack_module
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
            elif name == "slicegcn_accumulate_many":   # the list of sources ends with the call
                self.calls.append((name, a[0], list((ctypes.c_void_p * a[3]).from_address(a[2]))))
            else:
                self.calls.append((name, a))
            return 0
        return call

    def layers(self, name):
        return [c[1:] for c in self.calls if c[0] == f"slicegcn_layers_{name}"]


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


def replace(st, name, change):
    """Puts change(tensor) in the place of one of the stack's tensors (same address)."""
    holder, key = {"Z": (st.Z[-1], 0), "H": (st.H[-1], 0), "mask": (st.mask[-1], 1), "X": (st.X, -1), "W_self": (st.params[-1][1], "W_self"),
                   "b": (st.params[-1][1], "b"), "dW_agg": (st.grads[-1][1], "dW_agg"), "Hcat": (st.__dict__, "Hcat"),
                   "E": (st.__dict__, "E"), "dbuf": (st.dbuf[-1], 1)}[name]
    old = holder[key]
    holder[key] = change(old)
    assert holder[key].data_ptr() == old.data_ptr()
    return holder[key]


@pytest.fixture(params=[True, False], ids=["guards", "tuples"])
def comparison(request, monkeypatch):
    """The two ways the stack compares its tensors' layouts."""
    if not request.param:
        monkeypatch.setattr(stack_module, "TensorGuards", None)


@pytest.mark.parametrize("name", ["Z", "H", "X", "W_self", "b", "dW_agg", "Hcat", "E", "dbuf", "mask"])
def test_plan_sees_another_type_at_the_same_address(rec, comparison, name):
    st = stack()
    st.forward()
    st.backward(torch.randn(N, K * HS))
    replace(st, name, lambda t: t.view(torch.float32 if t.dtype == torch.int32 else torch.int32))
    good = len(rec.calls)
    if name not in ("dW_agg", "dbuf"):
        with pytest.raises(TypeError):
            st.forward()
    if name not in ("b", "Hcat", "E"):
        with pytest.raises(TypeError):
            st.backward(torch.randn(N, K * HS))
    assert len(rec.calls) == good


@pytest.mark.parametrize("name", ["W_self", "dW_agg", "Hcat", "X"])
def test_plan_sees_other_strides_at_the_same_address(rec, comparison, name):
    st = stack()
    st.forward()
    st.backward(torch.randn(N, K * HS))
    replace(st, name, lambda t: t.t() if t.shape[0] == t.shape[1] else t.as_strided((N, t.shape[1] // 2), (t.stride(0), 2)))
    with pytest.raises(TypeError):
        st.backward(torch.randn(N, K * HS)) if name == "dW_agg" else st.forward()


def test_plan_follows_leading_dimensions(rec, comparison):
    st = stack(k=1)
    st.forward()
    replace(st, "Hcat", lambda t: t.as_strided((N // 2, HS), (2 * HS, 1)))
    st.forward()
    assert [g.ldo for g, _ in rec.layers("fwd")] == [HS, HS, HS, 2 * HS]


@pytest.mark.parametrize("what", ["W_agg", "W_self"])
def test_plan_sees_another_shape_at_the_same_address(rec, comparison, what):
    st = stack()
    st.forward()
    st.params[0][0][what] = st.params[0][0][what].view(HS, FIRST)
    with pytest.raises(ValueError):
        st.forward()


def test_plan_sees_which_parameter_is_missing(rec, comparison):
    st = stack()
    p = st.params[0][0]
    p["b_self"] = None
    st.forward()
    p["b"], p["b_self"] = None, p["b"]
    st.forward()
    first, second = rec.layers("fwd")[0][1][0], rec.layers("fwd")[L][1][0]
    assert first.params.b and not first.params.b_self
    assert second.params.b_self == first.params.b and not second.params.b


def test_plan_is_kept_while_nothing_changes(rec, comparison, monkeypatch):
    """Also where a tensor stands in several places (shared inputs, shared weights, absent biases)."""
    st = stack(shared_input=torch.zeros(N, 64))
    for p in st.params:
        p[0].update(st.params[0][0], b=None)
    st.forward()
    st.backward(torch.randn(N, K * HS))
    made = []
    monkeypatch.setattr(B, "_LayerDesc", lambda *a, inner=B._LayerDesc: made.append(a) or inner(*a))
    st.forward()
    st.backward(torch.randn(N, K * HS))
    assert not made
    st.params[1][0]["W_agg"] = st.params[1][0]["W_agg"].clone()
    st.forward()
    assert made


def test_flags_changed_after_a_pass_take_effect(rec):
    """fuse_encoding, act_last and the layers' flags are what they are at the call, as the encoding pass looks at them."""
    st = stack()
    st.forward()
    st.backward(torch.randn(N, K * HS))
    assert all(x.enc for x in rec.layers("fwd")[L - 1][1]) and all(x.denc for x in rec.layers("bwd")[0][1])
    assert "slicegcn_concat" not in [c[0] for c in rec.calls]
    st.fuse_encoding, st.act_last = False, B.ACT_NONE
    st.layout[1] |= B.LAYER_OUT_SCALED
    del rec.calls[:]
    st.forward()
    st.backward(torch.randn(N, K * HS))
    (first, _), (last, io) = rec.layers("fwd")
    (last_b, io_b), _ = rec.layers("bwd")
    assert not any(x.enc or x.denc for x in io + io_b)     # the encoding is added once, by the pass of its own
    assert [c[0] for c in rec.calls].count("slicegcn_concat") == 1 and [c[0] for c in rec.calls].count("slicegcn_concat_bwd") == 1
    assert (first.desc.act, last.desc.act, last_b.desc.act) == (B.ACT_RELU, B.ACT_NONE, B.ACT_NONE)
    assert last.desc.flags == last_b.desc.flags == B.LAYER_OUT_SCALED


@pytest.mark.parametrize("what", ["leading dimension", "self term"])
def test_slices_that_differ_run_on_their_own(rec, what):
    """Slices whose layers share no launch (another padding of the features, no self term) run one after the other."""
    st = stack(layers=1, slice_encoding=False)
    if what == "self term":
        st.params[1][0].update(W_self=None, b_self=None)
    else:
        st.X[1] = torch.zeros(N, 96)
    st.forward()
    st.backward(torch.randn(N, K * HS))
    for way in ("fwd", "bwd"):
        got = rec.layers(way)
        assert [g.count for g, _ in got] == [1] * K
        assert [g.ldi for g, _ in got] == ([64] * K if what == "self term" else [64, 96, 64])
        assert [io[0].Hin for _, io in got] == [x.data_ptr() for x in st.X]
        assert [bool(io[0].params.W_self) for _, io in got] == [True, what != "self term", True]
    assert [g.ldgo for g, _ in rec.layers("bwd")] == [K * HS] * K


@pytest.mark.parametrize("streams,k,group", [(1, 1, 1), (1, 3, 1), (1, 3, 2), (1, 8, 8), (1, 19, 8), (1, 9, 8), (1, 20, 3), (4, 6, 1)])
def test_shared_input_gradients_alive(rec, monkeypatch, streams, k, group):
    """With feature fusion only the input gradients of the slices that run together are kept, and they are added in slice
    order, the first slice's being where the sum is formed."""
    monkeypatch.setattr(stack_module, "GROUP_BYTES", group * N * 20 * 64)
    if streams > 1:
        monkeypatch.setattr(torch.cuda, "Stream", lambda device=None: types.SimpleNamespace(wait_stream=lambda s: None))
        monkeypatch.setattr(torch.cuda, "current_stream", lambda: types.SimpleNamespace(wait_stream=lambda s: None))
        monkeypatch.setattr(torch.cuda, "stream", lambda s: contextlib.nullcontext())
    st = stack(k=k, shared_input=torch.zeros(N, 64), streams=streams)
    assert st.group == group
    together = k if streams > 1 else min(group, k)
    assert sum(t.numel() for t in st.dXs) <= (together if k > together else k - 1) * N * 64
    st.forward()
    del rec.calls[:]
    st.backward(torch.randn(N, k * HS))
    pending, order = {}, []
    for name, *a in rec.calls:
        if name == "slicegcn_layers_bwd" and a[0].desc.w_in == FIRST:
            for x in a[1]:
                slot = len(order) + len(pending)
                assert x.dHin not in pending, "a gradient is overwritten before it was added"
                if slot == 0:
                    assert x.dHin == st.dXin.data_ptr()
                    order.append(0)
                else:
                    pending[x.dHin] = slot
        elif name == "slicegcn_accumulate_many":
            assert a[0] == st.dXin.data_ptr() and 1 <= len(a[1]) <= B.MAX_GROUP
            order += [pending.pop(p) for p in a[1]]
    assert not pending and order == list(range(k))


@pytest.mark.parametrize("shared", [False, True])
def test_each_direction_looks_at_its_own_tensors(rec, comparison, shared):
    """Inference needs no gradient buffers (they may be gone, or of another type); a backward pass needs no biases."""
    st = stack(shared_input=torch.zeros(N, 64) if shared else None)
    grads, dE, dbuf, dXin, dXs = st.grads, st.dE, st.dbuf, st.dXin, st.dXs
    st.grads = st.dE = st.dbuf = st.dXin = st.dXs = None
    st.forward()
    st.forward()
    assert len(rec.layers("fwd")) == 2 * L
    st.grads, st.dE, st.dbuf, st.dXin, st.dXs = grads, dE, dbuf, dXin, dXs
    for per_slice in st.params:
        for p in per_slice:
            p["b"] = p["b"].double()
    st.backward(torch.randn(N, K * HS))
    assert len(rec.layers("bwd")) == L
    with pytest.raises(TypeError):
        st.forward()


def test_one_slice_runs_before_the_others_have_parameters(rec):
    st = stack(fuse_encoding=False)
    others, st.params[1:] = st.params[1:], [[None] * L for _ in range(K - 1)]
    st.forward_slice(0)
    assert [g.count for g, _ in rec.layers("fwd")] == [1] * L
    st.params[1:] = others
    st.forward()
    assert [g.count for g, _ in rec.layers("fwd")] == [1] * L + [K] * L
