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
