"""Backward passes on few rows form weight gradients and input gradients in one launch: the same bits as one after the other, and the separate
launches where the input gradient takes memory that the weight gradients read."""
import pytest
import torch

from paper_2408_11500_amd import binding as B

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 33, 1000, 5001, 20_011, 140_001])
@pytest.mark.parametrize("w_in,w_out", [(1, 1), (64, 8), (31, 32), (32, 33), (64, 64), (65, 64), (96, 96), (100, 7), (7, 100), (130, 129), (256, 40), (300, 200)])
def test_linear_bwd_together_and_apart(n, w_in, w_out):
    gen = torch.Generator(device="cuda").manual_seed(n + w_in)
    X, dY, W = (torch.randn(s, generator=gen, device="cuda") for s in ((n, w_in), (n, w_out), (w_in, w_out)))
    mask = torch.randint(-2**31, 2**31, (n, (w_out + 31) // 32), generator=gen, device="cuda").to(torch.int32)
    ws = torch.empty(B.slicegcn_linear_bwd_full_workspace_bytes(n, w_in, w_out), dtype=torch.uint8, device="cuda")

    def run(X, dX, grads=True):
        dW, db = (torch.empty_like(W), torch.empty(w_out, device="cuda")) if grads else (None, None)
        B.slicegcn_linear_bwd(X, W, mask, dY, dX, dW, db, ws, act=B.ACT_RELU)
        return dW, db

    dX, alone = torch.full((n, w_in + 1), 7.0, device="cuda"), torch.empty((n, w_in), device="cuda")
    got = run(X, dX[:, :w_in])
    want = run(X, None)
    run(X, alone, grads=False)
    assert torch.equal(dX[:, :w_in], alone) and bool((dX[:, w_in] == 7.0).all()) and all(map(torch.equal, got, want))
    over = X.clone()
    got = run(over, over)                                # in place of the layer's input, which the weight gradients read
    assert torch.equal(over, alone) and all(map(torch.equal, got, want))


@pytest.mark.parametrize("n,w_in,w_out", [(262_149, 128, 40), (562_501, 128, 40), (281_251, 256, 33), (281_249, 256, 64), (140_700, 512, 40)])
def test_linear_bwd_of_many_rows(n, w_in, w_out):
    """Below and above the length from which the input gradient goes to the kernel of wide products instead, at 72 M elements."""
    test_linear_bwd_together_and_apart(n, w_in, w_out)


@pytest.mark.parametrize("n", [1, 40, 3001, 70_001])
@pytest.mark.parametrize("w_in,w_out", [(1, 5), (3, 64), (4, 4), (33, 32), (64, 64), (100, 20), (128, 9), (130, 33), (301, 64)])
@pytest.mark.parametrize("self_term", [True, False])
def test_layer_gradients_beside_the_aggregation(n, w_in, w_out, self_term):
    """The final sums of the weight gradients, formed in the launch of the input gradient's aggregation, or in their own without one."""
    gen = torch.Generator(device="cuda").manual_seed(n + w_in)
    src, dst = (torch.randint(0, n, (4 * n,), generator=gen, device="cuda") for _ in range(2))
    g = B.slicegcn_build_norm_csr(src, dst, n)
    X, G = (torch.randn((n, w), generator=gen, device="cuda") for w in (w_in, w_out))
    W, Ws = (torch.randn((w_in, w_out), generator=gen, device="cuda") for _ in range(2))
    b = torch.zeros(w_out, device="cuda")
    Ws, bs = (Ws, b) if self_term else (None, None)
    Z, H = torch.empty((n, (w_in + 3) // 4 * 4), device="cuda")[:, :w_in], torch.empty((n, w_out), device="cuda")
    words = torch.zeros((n, (w_out + 31) // 32), dtype=torch.int32, device="cuda")
    B.slicegcn_layer_fwd(g, X, W, b, Ws, bs, H, Z, words)
    got = []
    for dX in (torch.empty_like(X), None):
        grads = [torch.full_like(t, 7.0) if t is not None else None for t in (W, b, Ws, bs)]
        ws = torch.empty(B.slicegcn_layer_bwd_workspace_bytes(g, w_in, w_out, dX is not None), dtype=torch.uint8, device="cuda")
        B.slicegcn_layer_bwd(g, X, W, Ws, Z, words, G, dX, *grads, ws)
        got.append([t for t in grads if t is not None])
    assert all(map(torch.equal, *got)) and not any(bool((t == 7.0).any()) for t in got[0])
    g.destroy()
