"""The lists that the aggregation takes its rows from: short rows of 0 to 4 entries, rows at the edges of the ranges that long
rows are taken in, graphs in which a list is empty."""
import numpy as np
import pytest
import torch

import oracle
import paper_2408_11500_amd as sg
from gpu_util import assert_close, dev

pytestmark = pytest.mark.gpu

N = 20_000
EDGES = [1, 2, 3, 4, 5, 64, 65, 256, 257, 512, 513, 1024, 1025, 2048, 2049, 4096, 4097, 8192, 8193]  # entries of a row with its diagonal


def star_rows(degrees, rng):
    """Directed pairs: row v has degrees[v] entries (other columns, drawn at random), the other rows none."""
    src = [np.full(d, v) for v, d in degrees]
    dst = [rng.permutation(N - 1)[:d] for v, d in degrees]
    dst = [np.where(x >= v, x + 1, x) for (v, _), x in zip(degrees, dst)]
    return np.concatenate(src + [[]]).astype(np.int64), np.concatenate(dst + [[]]).astype(np.int64)


@pytest.mark.parametrize("sched", [sg.binding.SCHED_SHORT_ITEMS, sg.binding.SCHED_LONG_ITEMS])
@pytest.mark.parametrize("loops", [False, True])
@pytest.mark.parametrize("which", ["all", "short", "none short", "empty"])
def test_rows_of_every_length(which, loops, sched):
    rng = np.random.default_rng(11)
    if which == "all":
        deg = [(int(v), d - loops) for v, d in zip(rng.permutation(N)[: 3 * len(EDGES)], EDGES * 3)]
    elif which == "short":
        deg = [(int(v), int(d)) for v, d in zip(rng.permutation(N)[:9_999], rng.integers(1, 4, 9_999))]
    elif which == "none short":
        deg = [(v, 6) for v in range(N)]
    else:
        deg = []
    src, dst = star_rows([(v, d) for v, d in deg if d > 0], rng)
    flags = sched | (sg.binding.ADD_SELF_LOOPS if loops else 0)
    o = oracle.build_norm_csr(src, dst, N, oracle.ADD_SELF_LOOPS if loops else 0)
    assert set(d + loops for _, d in deg) <= set(np.diff(o.rowptr))
    g = sg.slicegcn_build_norm_csr(dev(src, torch.int64), dev(dst, torch.int64), N, flags)
    for width in (5, 32, 64, 160):
        X = rng.standard_normal((N, width)).astype(np.float32)
        want = oracle.spmm(o, X)
        for pre in (False, True):
            Y = torch.full((N, width), float("nan"), device="cuda")
            sg.slicegcn_spmm_slice(g, dev(X * o.dinv[:, None].astype(np.float32) if pre else X), Y, prescaled=pre)
            assert_close(Y.cpu().numpy(), want, f"{which}, width {width}")
    g.destroy()
