"""Products in place: a gradient or an output in the rows of the operand it comes from is bitwise what it is in memory of its
own, at the widths and row counts where the kernels change their tiles; wider calls are refused."""
import numpy as np
import pytest
import torch

import paper_2408_11500_amd as sg
from paper_2408_11500_amd import binding as B
from gpu_util import dev, messy_edges

pytestmark = pytest.mark.gpu


def rows_of(gen, n, w, ld):
    return torch.randn((n, ld), generator=gen, device="cuda")[:, :w]


@pytest.mark.parametrize("n", [1, 129, 5003, 300_007])
@pytest.mark.parametrize("w_in,w_out", [(33, 33), (64, 64), (65, 65), (96, 96), (97, 97), (128, 128), (128, 40), (40, 128), (100, 300)])
def test_linear_bwd_in_place(n, w_in, w_out):
    gen = torch.Generator(device="cuda").manual_seed(n + w_in)
    ld = max(w_in, w_out) + 3
    X, dY, W = rows_of(gen, n, w_in, w_in), rows_of(gen, n, max(w_in, w_out), ld), rows_of(gen, w_in, w_out, w_out)
    mask = torch.randint(-2**31, 2**31, (n, (w_out + 31) // 32), generator=gen, device="cuda").to(torch.int32)
    ws = torch.empty(B.slicegcn_linear_bwd_full_workspace_bytes(n, w_in, w_out), dtype=torch.uint8, device="cuda")
    got = []
    for here in (False, True):
        g = torch.empty((n, ld), device="cuda")[:, :dY.shape[1]].copy_(dY)
        dX = g[:, :w_in] if here else torch.empty((n, w_in), device="cuda")
        dW, db = torch.empty_like(W), torch.empty(w_out, device="cuda")
        B.slicegcn_linear_bwd(X, W, mask, g[:, :w_out], dX, dW, db, ws, act=B.ACT_RELU)
        got.append((dX.clone(), dW, db))
    for a, b in zip(*got):
        assert torch.equal(a, b)


def test_wider_calls_are_refused_and_neighbours_are_not():
    n, w = 500, 160
    buf, W = torch.randn((n, 2 * w), device="cuda"), torch.randn((w, w), device="cuda")
    X, out = torch.randn((n, w), device="cuda"), torch.empty((n, w), device="cuda")
    before = buf.clone()
    with pytest.raises(B.SliceGCNError) as e:
        B.slicegcn_linear_bwd(X, W, None, buf[:, :w], buf[:, :w], None, None, None, act=B.ACT_NONE)
    assert e.value.status == B.EINVAL and torch.equal(buf, before)
    B.slicegcn_linear_bwd(X, W, None, buf[:, :w], out, None, None, None, act=B.ACT_NONE)
    B.slicegcn_linear_bwd(X, W, None, buf[:, :w], buf[:, w:], None, None, None, act=B.ACT_NONE)   # columns beside it
    assert torch.equal(buf[:, w:], out) and torch.equal(buf[:, :w], before[:, :w])


@pytest.mark.parametrize("order", [0, B.LAYER_TRANSFORM_FIRST])
@pytest.mark.parametrize("n", [70, 6001, 270_001])
@pytest.mark.parametrize("w", [20, 33, 64, 65, 96, 97])
def test_layer_in_place(order, n, w):
    gen = torch.Generator(device="cuda").manual_seed(n + w)
    src, dst = messy_edges(n, 3 * n, np.random.default_rng(n))
    g = sg.slicegcn_build_norm_csr(dev(src, torch.int64), dev(dst, torch.int64), n)
    ld = w + 1
    Hin, dHout = rows_of(gen, n, w, ld), rows_of(gen, n, w, ld)
    Wa, Ws, b, bs = rows_of(gen, w, w, w), rows_of(gen, w, w, w), rows_of(gen, 1, w, w)[0], rows_of(gen, 1, w, w)[0]
    Z = None if order else torch.empty((n, (w + 3) // 4 * 4), device="cuda")[:, :w]
    mask = torch.zeros((n, (w + 31) // 32), dtype=torch.int32, device="cuda")
    ws = torch.empty(B.slicegcn_layer_bwd_workspace_bytes(g, w, w, True, order), dtype=torch.uint8, device="cuda")
    out, dHin = torch.empty((n, w), device="cuda"), torch.empty((n, w), device="cuda")
    grads = [torch.empty_like(t) for t in (Wa, b, Ws, bs)]
    B.slicegcn_layer_fwd(g, Hin, Wa, b, Ws, bs, out, Z, mask, order=order)
    B.slicegcn_layer_bwd(g, Hin, Wa, Ws, Z, mask, dHout, dHin, *grads, ws, order=order)
    same_grads, same_dH = [torch.empty_like(t) for t in grads], torch.empty((n, ld), device="cuda")[:, :w].copy_(dHout)
    same_H = torch.empty((n, ld), device="cuda")[:, :w].copy_(Hin)
    if w > 96:
        with pytest.raises(B.SliceGCNError) as e:
            B.slicegcn_layer_bwd(g, Hin, Wa, Ws, Z, mask, same_dH, same_dH, *same_grads, ws, order=order)
        assert e.value.status == B.EINVAL and torch.equal(same_dH, dHout)
    else:
        B.slicegcn_layer_bwd(g, Hin, Wa, Ws, Z, mask, same_dH, same_dH, *same_grads, ws, order=order)
        assert torch.equal(same_dH, dHin) and all(map(torch.equal, grads, same_grads))
        B.slicegcn_layer_fwd(g, same_H, Wa, b, Ws, bs, same_H, Z, mask, order=order)
        assert torch.equal(same_H, out)
    g.destroy()
