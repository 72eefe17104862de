"""Slice layers through the strip kernels (many rows, widths up to 64): widths that fill the kernels' tiles, end inside a 16-byte access or are
narrower than one, a last strip that is not whole, rows on any boundary with NaN behind them, with and without self term."""
import pytest
import torch

from paper_2408_11500_amd import binding as B

pytestmark = pytest.mark.gpu

# From 2^16 rows on the weight gradients, and the products with 9 to 31 columns in, of the 32-wide kernels; from 2^18 on the products with 4 to 8
# and with 32 columns in as well; from 2^21 on all of the 64-wide ones.
ROWS32, ROWS32_ALL, ROWS64 = 65_536 + 21, (1 << 18) + 21, (1 << 21) + 13


@pytest.fixture(scope="module")
def graphs():
    """No edges but the diagonal: the aggregation copies, so that the products stand alone."""
    none = torch.empty(0, dtype=torch.int64, device="cuda")
    made = {n: B.slicegcn_build_norm_csr(none, none, n) for n in (ROWS32, ROWS32_ALL, ROWS64)}
    yield made
    for g in made.values():
        g.destroy()


def operand(gen, rows, cols, pad):
    full = torch.full((rows, cols + pad), float("nan"), device="cuda")
    full[:, :cols] = torch.randn((rows, cols), generator=gen, device="cuda")
    return full[:, :cols]


def assert_fp32(got, want, scale, what):
    """Within 3e-6 of the sum of the products' magnitudes, element by element: what chains of some thousand fp32 products stay below."""
    assert bool(torch.isfinite(got).all()), what
    worst = ((got.double() - want).abs() / scale.clamp_min(1e-300)).max().item()
    assert worst <= 3e-6, f"{what}: {worst:.2e}"


CASES = [(ROWS32, i, o, self_term, pad) for i, o in ((32, 32), (25, 32), (32, 25), (4, 4), (5, 31), (3, 32), (32, 2), (1, 1), (30, 7))
         for self_term, pad in ((True, 0), (True, 3), (False, 1))]
CASES += [(ROWS32_ALL, i, o, self_term, pad) for i, o in ((32, 32), (25, 32), (32, 25), (32, 2), (4, 4), (5, 31), (31, 7))
          for self_term, pad in ((True, 0), (True, 3), (False, 1))]
CASES += [(ROWS64, i, o, self_term, pad) for i, o, self_term, pad in ((64, 64, True, 3), (25, 64, True, 3), (40, 30, True, 0), (40, 30, False, 1),
                                                                     (2, 50, True, 3), (2, 50, False, 0), (61, 3, True, 3), (64, 64, False, 0))]


@pytest.mark.parametrize("n,w_in,w_out,self_term,pad", CASES)
def test_layer_matches_fp64(graphs, n, w_in, w_out, self_term, pad):
    gen = torch.Generator(device="cuda").manual_seed(w_in + 7 * w_out + pad)
    X, G = operand(gen, n, w_in, pad), operand(gen, n, w_out, pad)
    W, Ws = (torch.randn((w_in, w_out), generator=gen, device="cuda") for _ in range(2))
    b, bs = (torch.randn(w_out, generator=gen, device="cuda") for _ in range(2))
    if not self_term:
        Ws = bs = None
    Z = torch.full((n, (w_in + 3) // 4 * 4), float("nan"), device="cuda")[:, :w_in]   # rows on 16-byte boundaries, as the call asks
    H = torch.full((n, w_out + 1), 7.0, device="cuda")
    words = torch.zeros((n, (w_out + 31) // 32), dtype=torch.int32, device="cuda")
    B.slicegcn_layer_fwd(graphs[n], X, W, b, Ws, bs, H[:, :w_out], Z, words)
    assert torch.equal(Z, X) and bool((H[:, w_out] == 7.0).all())
    on = torch.stack([(words >> j) & 1 for j in range(32)], dim=2).reshape(n, -1)
    assert not bool(on[:, w_out:].any())
    on = on[:, :w_out].bool()
    pre, size = X.double() @ W.double() + b.double(), X.double().abs() @ W.double().abs() + b.double().abs()
    assert bool((on == (pre > 0))[pre.abs() > 3e-6 * size].all())
    want = torch.where(on, pre, 0.)
    if self_term:
        want, size = want + X.double() @ Ws.double() + bs.double(), size + X.double().abs() @ Ws.double().abs() + bs.double().abs()
    assert_fp32(H[:, :w_out], want, size, "H")
    del pre, size, want

    for input_gradient in (True, False):
        dX = torch.full((n, w_in + 1), 7.0, device="cuda") if input_gradient else None
        dW, db = torch.empty_like(W), torch.empty_like(b)
        dWs, dbs = (torch.empty_like(W), torch.empty_like(b)) if self_term else (None, None)
        ws = torch.empty(B.slicegcn_layer_bwd_workspace_bytes(graphs[n], w_in, w_out, input_gradient), dtype=torch.uint8, device="cuda")
        B.slicegcn_layer_bwd(graphs[n], X, W, Ws, Z, words, G, dX[:, :w_in] if input_gradient else None, dW, db, dWs, dbs, ws)
        P, Gd, Xd = torch.where(on, G, 0.).double(), G.double(), X.double()
        if input_gradient:
            want, size = P @ W.double().t(), P.abs() @ W.double().abs().t()
            if self_term:
                want, size = want + Gd @ Ws.double().t(), size + Gd.abs() @ Ws.double().abs().t()
            assert bool((dX[:, w_in] == 7.0).all())
            assert_fp32(dX[:, :w_in], want, size, "dHin")
            first = dW.clone()
        else:
            assert torch.equal(first, dW)   # the same sums with and without the input gradient
        assert_fp32(dW, Xd.t() @ P, Xd.abs().t() @ P.abs(), "dW_agg")
        assert_fp32(db, P.sum(0), P.abs().sum(0), "db")
        if self_term:
            assert_fp32(dWs, Xd.t() @ Gd, Xd.abs().t() @ Gd.abs(), "dW_self")
            assert_fp32(dbs, Gd.sum(0), Gd.abs().sum(0), "db_self")


@pytest.mark.parametrize("w_in", [32, 8, 7, 4])
@pytest.mark.parametrize("w_out", [32, 20])
@pytest.mark.parametrize("self_term", [True, False])
def test_rows_and_strips_have_the_same_bits(w_in, w_out, self_term):
    """4 to 8 and 32 columns in: strips from 2^18 rows on, the general kernel below; the last call has one row less."""
    n = 1 << 18
    gen = torch.Generator(device="cuda").manual_seed(w_out)
    X, G, W, Ws = (torch.randn(s, generator=gen, device="cuda") for s in ((n, w_in), (n, w_out), (w_in, w_out), (w_in, w_out)))
    b, bs = (torch.randn(w_out, generator=gen, device="cuda") for _ in range(2))
    if not self_term:
        Ws = bs = None
    none, got = torch.empty(0, dtype=torch.int64, device="cuda"), []
    for rows in (n, n - 1):
        g = B.slicegcn_build_norm_csr(none, none, rows)
        Z, H, words = torch.empty((rows, (w_in + 3) // 4 * 4), device="cuda")[:, :w_in], torch.empty((rows, w_out), device="cuda"), torch.zeros((rows, 1), dtype=torch.int32, device="cuda")
        B.slicegcn_layer_fwd(g, X[:rows], W, b, Ws, bs, H, Z, words)
        Y, bits = torch.empty((rows, w_out), device="cuda"), torch.zeros((rows, 1), dtype=torch.int32, device="cuda")
        B.slicegcn_linear_fwd(X[:rows], W, b, Y, bits, act=B.ACT_RELU)
        dX = torch.empty((rows, w_out), device="cuda")   # backward: the product with w_in columns in is that of a layer w_out -> w_in
        B.slicegcn_linear_bwd(G[:rows], W.t().contiguous(), None, X[:rows], dX, None, None, None, act=B.ACT_NONE)
        got.append([t[:n - 1] for t in (H, words, Y, bits, dX)])
        g.destroy()
    assert all(map(torch.equal, *got))


@pytest.mark.parametrize("w_in,w_out", [(25, 40), (32, 33), (4, 63), (17, 34), (33, 4), (40, 5), (64, 30), (64, 3), (64, 47), (61, 62), (34, 33)])
def test_rows_and_strips_up_to_64_wide_have_the_same_bits(w_in, w_out):
    """Columns out that do not fill the tiles: lanes at a row's end store its last four columns once more.  Strips from 2^18 rows on, the last
    one not whole; the general kernel below.  Rows on any boundary, NaN and guards behind them."""
    n = (1 << 18) + 21
    gen = torch.Generator(device="cuda").manual_seed(w_in + 64 * w_out)
    X, (W, Ws, b, bs) = operand(gen, n, w_in, 1), (torch.randn(s, generator=gen, device="cuda") for s in ((w_in, w_out), (w_in, w_out), (w_out,), (w_out,)))
    none, got = torch.empty(0, dtype=torch.int64, device="cuda"), []
    for rows in (n, (1 << 18) - 1):
        g = B.slicegcn_build_norm_csr(none, none, rows)
        Z = torch.empty((rows, (w_in + 3) // 4 * 4), device="cuda")[:, :w_in]
        H, Y, P, dX = (torch.full((rows, w_out + 1), 7.0, device="cuda") for _ in range(4))
        words, bits = (torch.zeros((rows, (w_out + 31) // 32), dtype=torch.int32, device="cuda") for _ in range(2))
        B.slicegcn_layer_fwd(g, X[:rows], W, b, Ws, bs, H[:, :w_out], Z, words)
        B.slicegcn_linear_fwd(X[:rows], W, b, Y[:, :w_out], bits, act=B.ACT_RELU)
        B.slicegcn_linear_fwd(X[:rows], W, b, P[:, :w_out])
        # backward: the product with w_in columns in is that of a layer w_out -> w_in
        B.slicegcn_linear_bwd(P[:, :w_out], W.t().contiguous(), None, X[:rows], dX[:, :w_out], None, None, None, act=B.ACT_NONE)
        assert all(bool((t[:, w_out] == 7.0).all()) for t in (H, Y, P, dX))
        got.append([t[:(1 << 18) - 1].clone() for t in (H, words, Y, bits, P, dX)])
        tail = [t[(1 << 18) - 1:] for t in (P, dX)]
        if rows == n:   # the last strips, against fp64
            Xd = X[(1 << 18) - 1:].double()
            for t, c in ((tail[0], b.double()), (tail[1], 0.)):
                assert_fp32(t[:, :w_out], Xd @ W.double() + c, Xd.abs() @ W.double().abs() + (c.abs() if torch.is_tensor(c) else 0.), "tail")
        g.destroy()
    assert all(map(torch.equal, *got))


@pytest.mark.parametrize("n", [300, 20_032])
@pytest.mark.parametrize("w_in,w_out", [(70, 1), (70, 3), (93, 7), (159, 21), (65, 31), (96, 34), (130, 67), (257, 35), (288, 97), (3, 99)])
def test_last_columns_of_the_general_kernel(n, w_in, w_out):
    """Output tiles that are not full, in strips of 32 rows and in a last one that is not: last columns stored once more, rows of up to three columns
    by a lane each.  Against fp64, guards behind the rows."""
    gen = torch.Generator(device="cuda").manual_seed(w_in + w_out)
    X, W, b = operand(gen, n, w_in, 1), *(torch.randn(s, generator=gen, device="cuda") for s in ((w_in, w_out), (w_out,)))
    Y, P, dX = (torch.full((n, w_out + 1), 7.0, device="cuda") for _ in range(3))
    words = torch.zeros((n, (w_out + 31) // 32), dtype=torch.int32, device="cuda")
    B.slicegcn_linear_fwd(X, W, b, P[:, :w_out])
    B.slicegcn_linear_fwd(X, W, b, Y[:, :w_out], words, act=B.ACT_RELU)
    B.slicegcn_linear_bwd(P[:, :w_out], W.t().contiguous(), None, X, dX[:, :w_out], None, None, None, act=B.ACT_NONE)
    assert all(bool((t[:, w_out] == 7.0).all()) for t in (Y, P, dX))
    want, size = X.double() @ W.double(), X.double().abs() @ W.double().abs()
    assert_fp32(P[:, :w_out], want + b.double(), size + b.double().abs(), "Y")
    assert torch.equal(Y[:, :w_out], P[:, :w_out].clamp_min(0.))
    assert_fp32(dX[:, :w_out], want, size, "dX")
