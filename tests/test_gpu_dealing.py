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
