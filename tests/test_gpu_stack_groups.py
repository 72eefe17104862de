"""Slice models in groups: more slices than share one set of launches, gradients of another layout from call to call, and
features padded differently, against slices that run one after the other (the same bits)."""
import numpy as np
import pytest
import torch

import paper_2408_11500_amd as sg
from paper_2408_11500_amd import stack as stack_module
from paper_2408_11500_amd.stack import SliceStack
from gpu_util import dev, messy_edges

pytestmark = pytest.mark.gpu

N, FIRST, HS, L = 3001, 37, 40, 2


@pytest.fixture(scope="module")
def graph():
    src, dst = messy_edges(N, 9000, np.random.default_rng(3))
    g = sg.slicegcn_build_norm_csr(dev(src, torch.int64), dev(dst, torch.int64), N)
    yield g
    g.destroy()


def make(g, k, shared, seed=1):
    gen = torch.Generator(device="cuda").manual_seed(seed)
    r = lambda *s: torch.randn(s, generator=gen, device="cuda")
    X = torch.zeros((N, 64), device="cuda")
    X[:, :FIRST] = r(N, FIRST)
    st = SliceStack(g, N, k, FIRST, HS, L, shared_input=X if shared else None)
    st.E.copy_(r(k, HS))
    for i in range(k):
        if not shared:
            st.X[i][:, :FIRST] = r(N, FIRST)
        for l, (wi, wo) in enumerate(st.widths):
            st.set_params(i, l, r(wi, wo) * 0.1, r(wo), r(wi, wo) * 0.1, r(wo))
    return st, r(N, 2 * k * HS + 5)


def outputs(st):
    out = [st.Hcat.clone(), st.dE.clone()] + ([st.dXin[:, :FIRST].clone()] if st.shared else [])
    return out + [gr[key].clone() for per_slice in st.grads for gr in per_slice for key in ("dW_agg", "db", "dW_self", "db_self")]


@pytest.mark.parametrize("k", [9, 17])
@pytest.mark.parametrize("shared", [False, True])
def test_more_slices_than_one_group(graph, monkeypatch, k, shared):
    runs = []
    for limit in (stack_module.GROUP_BYTES, 0):
        monkeypatch.setattr(stack_module, "GROUP_BYTES", limit)
        st, dH = make(graph, k, shared)
        assert st.group == (8 if limit else 1) and len(st.dXs) == (st.group if shared else 0)
        for _ in range(2):   # the second pass meets buffers that hold the first one's
            st.forward()
            st.backward(dH[:, :k * HS])
        runs.append(outputs(st))
    assert all(torch.isfinite(t).all() for t in runs[0])
    for a, b in zip(*runs):
        assert torch.equal(a, b)


def test_gradients_of_another_layout(graph):
    k = 3
    st, buf = make(graph, k, True)
    st.forward()
    w = k * HS
    views = [buf[:, :w], buf[:, w:2 * w], buf[:, 3:3 + w], buf[:, :w].contiguous(), buf[:, :w].t().contiguous().t().contiguous()]
    got = []
    for v in views:
        st.backward(v)
        got.append(outputs(st))
    for a, b, c in zip(got[0], got[3], got[4]):
        assert torch.equal(a, b) and torch.equal(a, c)
    for v, want in zip(views, got):
        st2, _ = make(graph, k, True)
        st2.forward()
        st2.backward(v.contiguous())
        for a, b in zip(want, outputs(st2)):
            assert torch.equal(a, b)
    before = outputs(st)
    for bad in (buf[:, ::2][:, :w], buf[:, :w].double(), buf[:, :w].t()):
        with pytest.raises(TypeError):
            st.backward(bad)
    for a, b in zip(before, outputs(st)):
        assert torch.equal(a, b)


def test_features_padded_differently(graph):
    """Slices whose leading dimensions differ share no launch and give the same bits."""
    k = 3
    runs = []
    for ld in (64, 96):
        st, dH = make(graph, k, False)
        if ld != 64:
            X = torch.zeros((N, ld), device="cuda")
            X[:, :FIRST] = st.X[1][:, :FIRST]
            st.X[1] = X
        st.forward()
        st.backward(dH[:, :k * HS])
        runs.append(outputs(st))
    for a, b in zip(*runs):
        assert torch.equal(a, b)


def test_encoding_fused_or_not_after_a_pass(graph):
    """fuse_encoding cleared between passes: the encoding is still added once."""
    st, dH = make(graph, 3, False)
    st.forward()
    st.backward(dH[:, :3 * HS])
    fused = outputs(st)
    st.fuse_encoding = False
    st.forward()
    st.backward(dH[:, :3 * HS])
    for a, b in zip(fused, outputs(st)):
        # the same sums in another order: one addition more per element forward, column sums of N rows backward
        assert float((a - b).abs().max()) <= 3e-6 * float(a.abs().max()) * (1 if a.shape[0] == N else 16)


def in_a_group_and_alone(monkeypatch, n, k, first, hs, self_term=True):
    rng = np.random.default_rng(first)
    g = sg.slicegcn_build_norm_csr(dev(rng.integers(0, n, 3 * n), torch.int64), dev(rng.integers(0, n, 3 * n), torch.int64), n)
    runs = []
    for limit in (stack_module.GROUP_BYTES, 0):
        monkeypatch.setattr(stack_module, "GROUP_BYTES", limit)
        gen = torch.Generator(device="cuda").manual_seed(first)
        r = lambda *s: torch.randn(s, generator=gen, device="cuda")
        X = torch.zeros((n, 64), device="cuda")
        X[:, :first] = r(n, first)
        st = SliceStack(g, n, k, first, hs, L, shared_input=X)
        st.E.copy_(r(k, hs))
        for i in range(k):
            for l, (wi, wo) in enumerate(st.widths):
                st.set_params(i, l, r(wi, wo) * 0.1, r(wo), *((r(wi, wo) * 0.1, r(wo)) if self_term else (None, None)))
        assert st.group == (k if limit else 1)
        dH = r(n, k * hs)
        st.forward()
        st.backward(dH)
        runs.append([st.Hcat.clone(), st.dE.clone(), st.dXin[:, :first].clone()] +
                    [gr[key].clone() for per_slice in st.grads for gr in per_slice for key in ("dW_agg", "db", "dW_self", "db_self") if gr[key] is not None])
    g.destroy()
    for a, b in zip(*runs):
        assert bool(torch.isfinite(a).all()) and torch.equal(a, b)


@pytest.mark.parametrize("first,hs", [(37, 64), (64, 40), (30, 30)])
def test_group_takes_the_strip_kernels_and_one_slice_does_not(monkeypatch, first, hs):
    """Together the slices of a launch have rows enough for the strip kernels, one alone has not: the same bits."""
    in_a_group_and_alone(monkeypatch, 66_003, 4, first, hs)


@pytest.mark.parametrize("n,first,hs,self_term", [(20_011, 64, 64, True), (20_011, 37, 40, True), (20_011, 5, 64, True), (20_011, 30, 31, True),
                                                  (66_003, 64, 64, False), (66_003, 37, 40, False), (66_003, 5, 64, False)])
def test_weight_gradients_of_a_group_in_strips_and_of_one_slice_in_tiles(monkeypatch, n, first, hs, self_term):
    """Blocks of 256 rows: pairs of products go to the strips from 160 of them on (79 a slice), single products from 512 on (258 a slice)."""
    in_a_group_and_alone(monkeypatch, n, 4, first, hs, self_term)


@pytest.mark.parametrize("n,k,first,hs", [(87_403, 3, 37, 100), (66_003, 4, 64, 96), (35_011, 8, 40, 164), (52_451, 2, 47, 260)])
def test_group_takes_the_wide_products_and_one_slice_does_not(monkeypatch, n, k, first, hs):
    """Input gradients of wide layers: together the slices of a launch have strips enough for pair_wide_kernel, which forms the two products of each one
    after the other; alone a slice goes to the general kernel: the same bits."""
    in_a_group_and_alone(monkeypatch, n, k, first, hs)


def test_group_with_more_column_tiles_than_fill_the_chip(monkeypatch):
    """Ten tiles of columns by eight slices and by six: the general kernel and the wide one."""
    in_a_group_and_alone(monkeypatch, 9_001, 8, 20, 320)
    in_a_group_and_alone(monkeypatch, 9_001, 6, 20, 320)
