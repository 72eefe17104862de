"""Graph construction at the edges of its key formats and chunks: 32-bit keys up to 65 535 nodes, 1024 keys per
wavefront; memory from torch's allocator and from the library itself."""
import ctypes

import numpy as np
import pytest
import torch

import oracle
import paper_2408_11500_amd as sg
from paper_2408_11500_amd import binding as B
from gpu_util import dev, hub_edges, messy_edges

pytestmark = pytest.mark.gpu


def check(o, g):
    h = g.to_host()
    assert h["nnz"] == o.nnz and np.array_equal(h["rowptr"].astype(np.int64), o.rowptr)
    assert np.array_equal(h["colidx"], o.colidx) and np.array_equal(h["deg"], o.deg)
    assert np.max(np.abs(h["vals"] / o.vals - 1.0), initial=0.0) <= 1e-6


@pytest.mark.parametrize("flags", [3, 2, 0])
@pytest.mark.parametrize("n,m", [(1, 3), (32767, 1024), (65535, 1023), (65536, 1025), (65537, 70000), (3, 4096), (1024, 0)])
def test_key_widths_and_chunks(n, m, flags):
    rng = np.random.default_rng(n + m + flags)
    src, dst = messy_edges(n, m, rng)
    if m > 4:
        src[:2], dst[:2] = n - 1, [0, n - 1]     # the largest key of a row, and a self pair beside the sentinel
    o = oracle.build_norm_csr(src, dst, n, flags)
    g = sg.slicegcn_build_norm_csr(dev(src, torch.int64), dev(dst, torch.int64), n, flags)
    check(o, g)
    g.destroy()


@pytest.mark.parametrize("flags", [3, 2])
def test_library_owned_memory(flags):
    rng = np.random.default_rng(5)
    n, w = 20011, 32
    src, dst = hub_edges(n, 50000, hubs=[0, n - 1], hub_deg=5000, rng=rng)
    o = oracle.build_norm_csr(src, dst, n, flags)
    s, d = dev(src, torch.int64), dev(dst, torch.int64)
    h = ctypes.c_void_p(0)
    assert B.lib().slicegcn_build_norm_csr(s.data_ptr(), d.data_ptr(), s.numel(), n, flags, None, ctypes.byref(h)) == 0
    g = B.Graph(h.value)
    check(o, g)
    X = rng.standard_normal((n, w)).astype(np.float32)
    Y = torch.empty((n, w), device="cuda")
    for transpose in (False, True):
        sg.slicegcn_spmm_slice(g, dev(X), Y, transpose=transpose)
        want = oracle.spmm(o, X, transpose=transpose)
        assert np.max(np.abs(Y.cpu().numpy() - want)) <= 1e-5 * np.max(np.abs(want))
    g.destroy()
