"""The whole rows of 5 to 64 entries are dealt to the column classes in stretches whose length depends on how many there are:
every row is formed exactly once at the list lengths where the stretch grows, and where the last stretch is not full."""
import numpy as np
import pytest
import torch

import paper_2408_11500_amd as sg
from gpu_util import dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("width", [32, 64, 128])   # 32, 16 and 8 rows per chunk
@pytest.mark.parametrize("chunks", [4, 127, 128, 129, 513, 2047, 2048, 2305])
def test_every_row_once(width, chunks):
    rows = 4 * (64 // (width // 4)) * chunks - 3          # the last chunk is not full
    n = rows                                              # more than 22: the seven columns of a row differ
    v = np.arange(n)
    src = np.concatenate([v] * 3)
    dst = np.concatenate([(v + 1) % n, (v + 5) % n, (v + 11) % n])   # six neighbours and the diagonal: 7 entries per row
    X = torch.randn((n, width), generator=torch.Generator(device="cuda").manual_seed(chunks), device="cuda")
    for flags in (0, sg.binding.REORDER_BFS):
        g = sg.slicegcn_build_norm_csr(dev(src, torch.int64), dev(dst, torch.int64), n,
                                       sg.binding.SYMMETRIZE | sg.binding.ADD_SELF_LOOPS | sg.binding.SCHED_LONG_ITEMS | flags)
        Y = torch.full((n, width), float("nan"), device="cuda")
        sg.slicegcn_spmm_slice(g, X, Y)
        want = torch.zeros((n, width), dtype=torch.float64, device="cuda")
        for s in (0, 1, 5, 11, -1, -5, -11):
            want += torch.roll(X.double(), -s, 0)
        # fp32: three roundings of a stored value, one of its product, six of the sum, of terms that add up to at most max|X|
        assert float((Y.double() - want / 7).abs().max()) <= 11 * 2.0 ** -24 * float(X.abs().max())
        g.destroy()


def test_more_workgroups_than_one_grid():
    """Whole rows beyond the 2^32 threads of one grid: eight 128-column rows a workgroup, 2^27 rows and some.  Every row is formed."""
    n = 2 ** 27 + 4099
    v = torch.arange(n, device="cuda")
    src, dst = torch.cat([v, v]), torch.cat([(v + 1) % n, (v + 5) % n])     # four neighbours and the diagonal
    g = sg.slicegcn_build_norm_csr(src, dst, n)
    del src, dst
    x = (v % 61).float()
    del v
    torch.cuda.empty_cache()
    X = torch.empty((n, 128), device="cuda").copy_(x[:, None])
    Y = torch.full((n, 128), float("nan"), device="cuda")
    sg.slicegcn_spmm_slice(g, X, Y)
    want = (x + sum(torch.roll(x, s) for s in (1, 5, -1, -5))) / 5
    for i in range(0, n, 2 ** 22):
        # whole numbers up to 60 times 1/5 in fp32: three roundings of the stored value, one of each product, four of the sum
        assert float((Y[i:i + 2 ** 22] - want[i:i + 2 ** 22, None]).abs().max()) <= 8 * 2.0 ** -24 * 60
    g.destroy()
    del X, Y
    torch.cuda.empty_cache()


@pytest.fixture(scope="module", params=["symmetric", "directed", "breadth first", "few columns"])
def band(request):
    """Columns within 200 of the row, 1 to 32 entries and more, and a few rows of about 280 entries that are cut; or columns below 70 and the
    diagonal: graphs numbered like this take several items per lane group."""
    n, rng = 70_003, np.random.default_rng(7)
    deg = rng.integers(0, 16, n)
    src = np.repeat(np.arange(n), deg)
    dst = rng.integers(0, 70, src.size) if request.param == "few columns" else np.clip(src + rng.integers(-200, 201, src.size), 0, n - 1)
    hubs = rng.integers(0, n, 6)
    src = np.concatenate([src, np.repeat(hubs, 280)])
    dst = np.concatenate([dst, rng.integers(0, n, 6 * 280)])
    flags = {"symmetric": sg.binding.SYMMETRIZE, "directed": 0, "few columns": 0, "breadth first": sg.binding.SYMMETRIZE | sg.binding.REORDER_BFS}[request.param]
    g = sg.slicegcn_build_norm_csr(dev(src, torch.int64), dev(dst, torch.int64), n, flags | sg.binding.ADD_SELF_LOOPS)
    h = g.to_host()
    rows = torch.as_tensor(np.repeat(np.arange(n), np.diff(h["rowptr"]))).cuda()
    yield g, n, rows, torch.as_tensor(h["colidx"]).long().cuda(), torch.as_tensor(h["vals"]).double().cuda(), torch.as_tensor(h["dinv"]).cuda(), flags == 0
    g.destroy()


def aggregated(band, X, transpose):
    """A X and |A| |X| in 64 bits."""
    g, n, rows, cols, vals, dinv, _ = band
    if transpose:
        rows, cols = cols, rows
    return [torch.zeros((n, X.shape[1]), dtype=torch.float64, device="cuda").index_add_(0, rows, vals[:, None] * x[cols]) for x in (X.double(), X.double().abs())]


@pytest.mark.parametrize("width,ld", [(3, 3), (25, 25), (25, 32), (32, 32), (64, 64), (100, 101), (128, 128), (300, 304)])   # 2 to 8 items per lane group
@pytest.mark.parametrize("prescaled", [False, True])
def test_several_items_per_lane_group(band, width, ld, prescaled):
    g, n, dinv, directed = band[0], band[1], band[5], band[6]
    X = torch.full((n, ld), float("nan"), device="cuda")
    X[:, :width] = torch.randn((n, width), generator=torch.Generator(device="cuda").manual_seed(width), device="cuda")
    given = X * dinv[:, None] if prescaled else X
    for transpose in (False, True) if directed else (False,):
        Y = torch.full((n, ld + 1), 7.0, device="cuda")
        sg.slicegcn_spmm_slice(g, given[:, :width], Y[:, :width], transpose=transpose, prescaled=prescaled)
        want, size = aggregated(band, X[:, :width], transpose)
        # fp32 sums of at most 600 terms, and four roundings of a value, its factors and the product
        assert bool(((Y[:, :width].double() - want).abs() <= 604 * 2.0 ** -24 * size).all()) and bool((Y[:, width:] == 7.0).all())


@pytest.mark.parametrize("w_in,w_out", [(32, 20), (64, 33), (128, 16)])
def test_several_items_per_lane_group_beside_final_sums(band, w_in, w_out):
    """A layer's input gradient, in whose launch the final sums of its weight gradients are formed."""
    g, n, directed = band[0], band[1], band[6]
    gen = torch.Generator(device="cuda").manual_seed(w_in)
    X, Z, G, W, Ws = (torch.randn(s, generator=gen, device="cuda") for s in ((n, w_in), (n, w_in), (n, w_out), (w_in, w_out), (w_in, w_out)))
    got = []
    for dX in (torch.empty((n, w_in), device="cuda"), None):
        grads = [torch.full(s, 7.0, device="cuda") for s in ((w_in, w_out), (w_out,), (w_in, w_out), (w_out,))]
        ws = torch.empty(sg.binding.slicegcn_layer_bwd_workspace_bytes(g, w_in, w_out, dX is not None), dtype=torch.uint8, device="cuda")
        sg.binding.slicegcn_layer_bwd(g, X, W, Ws, Z, None, G, dX, *grads, ws, act=sg.binding.ACT_NONE)
        got.append(grads)
        if dX is not None:
            want = aggregated(band, G.double() @ W.double().t(), directed)[0] + G.double() @ Ws.double().t()
            size = aggregated(band, G.double().abs() @ W.double().abs().t(), directed)[0] + G.double().abs() @ Ws.double().abs().t()
            assert bool(((dX.double() - want).abs() <= (604 + 2 * w_out) * 2.0 ** -24 * size).all())
    assert all(map(torch.equal, *got))
