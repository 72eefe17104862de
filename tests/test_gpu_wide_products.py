"""Products of wide layers on many rows (pair_wide_kernel; where one of the two widths is narrow, the direction that has it as its columns may be another
kernel's): bit for bit what the same rows give a few at a time, which takes the general kernel, and within an fp32 sum's bound of fp64."""
import pytest
import torch

import paper_2408_11500_amd as sg
from paper_2408_11500_amd import binding as B

pytestmark = pytest.mark.gpu

# rows, columns in, columns out: odd and whole chunks of k, one to many of them, full and partial tiles of columns and strips of rows
SIZES = [(262_144, 256, 64), (131_073, 4, 160), (87_390, 47, 288), (262_177, 64, 36), (131_101, 65, 256), (65_536, 301, 253), (262_145, 511, 63),
         (87_401, 33, 269), (131_100, 100, 229),
         (262_145, 333, 96), (262_145, 96, 333)]  # three tiles whose weights fill LDS to the last group of k
# two, three and four tiles of columns a workgroup, two and four chunks ahead, whole and partial last chunks, each forward and as an input gradient
SIZES += [(262_177, 128, 100), (262_146, 64, 96), (262_149, 96, 40), (262_155, 128, 96), (262_158, 96, 64), (262_155, 96, 128), (262_159, 64, 100),
          (262_151, 40, 100), (262_157, 40, 96)]
# several workgroups along the columns, five with two tiles each and up to two chunks of k among them, and beside them shorter products, which go to the general kernel
SIZES += [(52_452, 47, 310), (52_453, 320, 64), (131_105, 48, 160), (87_390, 100, 288), (65_570, 40, 512), (52_450, 128, 320), (52_451, 310, 47), (52_450, 64, 320)]
# less than a chunk of k, into whole lines (five columns of padding): with activation bits from four steps on, without from eight
SIZES += [(262_150, 5, 91), (262_151, 91, 6), (131_091, 9, 251), (131_092, 251, 14)]
FEW = 4096


def _in_pieces(n, f):
    for a in range(0, n, FEW):
        f(slice(a, min(n, a + FEW)))


@pytest.mark.parametrize("n,w_in,w_out", SIZES)
def test_wide_products_same_bits_as_few_rows(n, w_in, w_out):
    gen = torch.Generator(device="cuda").manual_seed(n)
    rand = lambda *s: torch.randn(s, generator=gen, device="cuda")
    X, W, b, pad = rand(n, w_in + 3)[:, :w_in], rand(w_in, w_out), rand(w_out), 5
    words = (w_out + 31) // 32
    for act in (B.ACT_RELU, B.ACT_NONE):
        Y, Y2 = (torch.full((n, w_out + pad), 7.0, device="cuda") for _ in range(2))
        M, M2 = (torch.full((n, words + 1), -3, dtype=torch.int32, device="cuda") for _ in range(2))
        B.slicegcn_linear_fwd(X, W, b, Y[:, :w_out], M[:, :words], act=act)
        _in_pieces(n, lambda r: B.slicegcn_linear_fwd(X[r], W, b, Y2[r, :w_out], M2[r, :words], act=act))
        assert torch.equal(Y, Y2) and torch.equal(M, M2)  # the padding too
    some = torch.cat([torch.arange(40), torch.arange(n - 40, n)]).cuda()
    want, size = X[some].double() @ W.double() + b.double(), X[some].double().abs() @ W.double().abs() + b.double().abs()
    assert bool(((Y[some, :w_out].double() - want).abs() <= (w_in + 2) * 2.0 ** -24 * size).all())

    dY = rand(n, w_out)
    mask = torch.randint(-2 ** 31, 2 ** 31 - 1, (n, words), generator=gen, device="cuda", dtype=torch.int32)
    ws = torch.empty(256, dtype=torch.uint8, device="cuda")
    for m, act in ((mask, B.ACT_RELU), (None, B.ACT_NONE)):
        D, D2 = (torch.full((n, w_in + pad), 7.0, device="cuda") for _ in range(2))
        B.slicegcn_linear_bwd(X, W, m, dY, D[:, :w_in], None, None, ws, act=act)
        _in_pieces(n, lambda r: B.slicegcn_linear_bwd(X[r], W, None if m is None else m[r], dY[r], D2[r, :w_in], None, None, ws, act=act))
        assert torch.equal(D, D2)


def test_wide_product_keeps_rows_with_infinities_apart():
    n = 131_072
    gen = torch.Generator(device="cuda").manual_seed(1)
    X, W = torch.randn((n, 96), generator=gen, device="cuda"), torch.randn((96, 256), generator=gen, device="cuda")
    b, Y = torch.zeros(256, device="cuda"), torch.empty((n, 256), device="cuda")
    B.slicegcn_linear_fwd(X, W, b, Y, None)
    X[5, 95], X[n - 1, 0] = float("inf"), float("nan")
    Z = torch.empty_like(Y)
    B.slicegcn_linear_fwd(X, W, b, Z, None)
    assert bool(Z[5].isinf().all()) and bool(Z[n - 1].isnan().all())
    Z[5], Z[n - 1] = Y[5], Y[n - 1]
    assert torch.equal(Y, Z)


@pytest.mark.parametrize("n,w_in,w_out", [(262_177, 128, 128), (262_150, 96, 65), (262_151, 70, 36), (131_080, 301, 33), (87_400, 260, 100), (131_081, 250, 9), (262_161, 90, 4)])
def test_wide_input_gradients_of_a_layer_same_bits_as_few_rows(n, w_in, w_out):
    """A graph of pairs and single nodes: its rows can be worked on a few at a time.  dZ takes row factors and the activation bits, T neither."""
    gen = torch.Generator(device="cuda").manual_seed(n)
    rand = lambda *s: torch.randn(s, generator=gen, device="cuda")

    def graph(count):
        a = torch.arange(0, count - 1, 6, device="cuda")
        return sg.slicegcn_build_norm_csr(a, a + 1, count, B.SYMMETRIZE | B.ADD_SELF_LOOPS)

    Wa, Ws, words = rand(w_in, w_out), rand(w_in, w_out), (w_out + 31) // 32
    Hin, Z, dH = rand(n, w_in), rand(n, (w_in + 3) // 4 * 4)[:, :w_in], rand(n, w_out + 1)[:, :w_out]
    mask = torch.randint(-2 ** 31, 2 ** 31 - 1, (n, words), generator=gen, device="cuda", dtype=torch.int32)

    def backward(g, r):
        dHin, grads = torch.empty((len(Hin[r]), w_in), device="cuda"), [torch.empty_like(x) for x in (Wa, Wa[0], Wa, Wa[0])]
        ws = torch.empty(B.slicegcn_layer_bwd_workspace_bytes(g, w_in, w_out, True), dtype=torch.uint8, device="cuda")
        B.slicegcn_layer_bwd(g, Hin[r], Wa, Ws, Z[r], mask[r], dH[r], dHin, *grads, ws)
        return dHin

    step = FEW - FEW % 6
    whole, piece, last = graph(n), graph(step), graph(n % step)
    got = backward(whole, slice(0, n))
    for a in range(0, n, step):
        r = slice(a, min(n, a + step))
        assert torch.equal(got[r], backward(piece if a + step <= n else last, r))
