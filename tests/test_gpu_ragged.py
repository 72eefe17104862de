"""Aggregation of operands whose rows are not on 16-byte boundaries: the lane that owns a row's last columns loads the
last four of them and shifts its sums, so nothing outside the operand is read."""
import numpy as np
import pytest
import torch

import oracle
import paper_2408_11500_amd as sg
from gpu_util import assert_close, dev, hub_edges

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def graph():
    rng = np.random.default_rng(7)
    n = 9001
    src, dst = hub_edges(n, 30000, hubs=[0, 4000, n - 1], hub_deg=3000, rng=rng)   # items of all three kinds, cut rows
    o = oracle.build_norm_csr(src, dst, n)
    g = sg.slicegcn_build_norm_csr(dev(src, torch.int64), dev(dst, torch.int64), n)
    yield n, o, g
    g.destroy()


@pytest.mark.parametrize("width", [1, 2, 3, 4, 5, 7, 25, 31, 33, 66, 129, 130, 131, 259])
@pytest.mark.parametrize("offset", [0, 1])
def test_spmm_contiguous_rows(graph, width, offset):
    n, o, g = graph
    rng = np.random.default_rng(width)
    X = rng.standard_normal((n, width)).astype(np.float32)
    flat = torch.full((offset + n * width,), float("nan"), device="cuda")   # ends with the last element of the last row
    flat[offset:] = torch.as_tensor(X).reshape(-1).cuda()
    Y = torch.full((n, width + 1), float("nan"), device="cuda")
    want = oracle.spmm(o, X)
    for pre in (False, True):
        if pre:
            flat[offset:] = torch.as_tensor(X * o.dinv[:, None].astype(np.float32)).reshape(-1).cuda()
        sg.slicegcn_spmm_slice(g, flat[offset:].view(n, width), Y[:, :width], prescaled=pre)
        assert_close(Y[:, :width].cpu().numpy(), want, f"contiguous w={width}")
        assert bool(torch.isnan(Y[:, width]).all())                            # nothing written past width


@pytest.mark.parametrize("width", [129, 200, 301])
@pytest.mark.parametrize("pre", [False, True])
def test_wide_operand_with_the_workspace_of_one_pass(graph, width, pre):
    """On a cache-resident graph all passes of 128 columns share a launch where the workspace holds their partial sums, and
    follow each other in the workspace of one pass otherwise: the same bits."""
    n, o, g = graph
    X = torch.randn((n, width), generator=torch.Generator(device="cuda").manual_seed(width), device="cuda")
    full, least = sg.slicegcn_spmm_workspace_bytes(g, width), sg.slicegcn_spmm_workspace_bytes(g, 128)
    assert 0 < least < full
    got = []
    for size in (full, full - 256, least):
        Y = torch.full((n, width), float("nan"), device="cuda")
        sg.slicegcn_spmm_slice(g, X, Y, ws=torch.empty(size, dtype=torch.uint8, device="cuda"), prescaled=pre)
        got.append(Y)
    assert torch.equal(got[0], got[1]) and torch.equal(got[0], got[2])
    want = oracle.spmm(o, X.cpu().numpy() * (1 / o.dinv[:, None] if pre else 1))
    assert_close(got[0].cpu().numpy(), want, f"w={width}")
    with pytest.raises(sg.binding.SliceGCNError) as e:
        sg.slicegcn_spmm_slice(g, X, Y, ws=torch.empty(least - 256, dtype=torch.uint8, device="cuda"), prescaled=pre)
    assert e.value.status == sg.binding.EWORKSPACE
