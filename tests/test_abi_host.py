"""Host-side checks of the C ABI that need no GPU: the library loads, exports every symbol the
header declares, the host-only slice strategy equals the oracle, and argument validation
returns error codes before any device work."""
import ctypes
import os
import re
import types

import pytest
import torch

import oracle
from paper_2408_11500_amd import binding

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def L():
    if not os.path.exists(binding.LIB_PATH):
        from paper_2408_11500_amd import build
        build.build(verbose=False)
    return binding.lib()


def declared_symbols(header="slicegcn.h"):
    text = open(os.path.join(ROOT, "include", header)).read()
    text = re.sub(r"/\*.*?\*/", "", text, flags=re.S)
    return sorted(set(re.findall(r"\b(slicegcn_[a-z_]+)\s*\(", text)))


def test_every_declared_symbol_is_exported(L):
    names = declared_symbols()
    assert len(names) == 29 and set(names) == set(binding.EXPORTS)
    for n in names:
        assert getattr(L, n) is not None


def test_the_native_header_is_exported_too(L):
    names = set(declared_symbols("slicegcn_native.h"))
    assert {"slicegcn_build_norm_csr_with", "slicegcn_layers_fwd", "slicegcn_layers_bwd", "slicegcn_accumulate_many"} <= names
    for n in names:
        assert getattr(L, n).argtypes is not None


def test_slice_strategy_matches_oracle(L):
    for d in range(1, 80):
        for p in range(1, d + 1):
            assert binding.slicegcn_slice_strategy(d, p) == oracle.slice_strategy(d, p)
    for d, p, s in [(100, 4, 0.5), (100, 4, 1.5), (301, 3, 1.0), (602, 2, 1.0), (7, 2, 1.7)]:
        assert binding.slicegcn_slice_strategy(d, p, s) == oracle.slice_strategy(d, p, s)


@pytest.mark.parametrize("args", [(0, 1, 1.0), (4, 0, 1.0), (4, 5, 1.0), (4, 2, 0.0), (4, 2, -1.0), (4, 2, 0.1), (4, 2, 3.0)])
def test_slice_strategy_rejects(L, args):
    with pytest.raises(binding.SliceGCNError) as e:
        binding.slicegcn_slice_strategy(*args)
    assert e.value.status == binding.EINVAL
    with pytest.raises(ValueError):
        oracle.slice_strategy(*args)


def test_cosine_lr_matches_oracle(L):
    for t in range(0, 51, 5):
        assert abs(binding.slicegcn_cosine_lr(0.01, 1e-4, t, 50) - oracle.cosine_lr(0.01, 1e-4, t, 50)) < 1e-15
    assert binding.slicegcn_cosine_lr(0.01, 0.0, 3, 0) == 0.01


def test_null_and_size_errors_return_codes(L):
    h = ctypes.c_void_p(0)
    assert L.slicegcn_build_norm_csr(None, None, 0, 0, 3, None, ctypes.byref(h)) == binding.EINVAL      # n_nodes < 1
    assert L.slicegcn_build_norm_csr(None, None, 5, 10, 3, None, ctypes.byref(h)) == binding.EINVAL     # NULL edges
    assert L.slicegcn_build_norm_csr(None, None, 0, 10, 1 << 20, None, ctypes.byref(h)) == binding.EINVAL  # unknown flag
    assert L.slicegcn_build_norm_csr(None, None, 0, 10, 3 | 16 | 32, None, ctypes.byref(h)) == binding.EINVAL  # both item limits
    assert L.slicegcn_build_norm_csr(None, None, 0, 1 << 31, 3, None, ctypes.byref(h)) == binding.ERANGE
    assert L.slicegcn_build_norm_csr(None, None, 0, 10, 3, None, None) == binding.EINVAL
    assert L.slicegcn_spmm_slice(None, 0, None, 4, 4, None, 4, None, 0, None) == binding.EINVAL
    assert L.slicegcn_spmm_workspace_bytes(None, 0, 32) == 0 and L.slicegcn_layer_fwd_workspace_bytes(None, None) == 0
    assert L.slicegcn_slice_feature(None, 4, 4, 0, 2, None, 2, None) == binding.EINVAL
    assert L.slicegcn_graph_destroy(None) == binding.OK
    assert L.slicegcn_layer_bwd_workspace_bytes(None, None, 1) == 0
    assert b"NULL" in L.slicegcn_last_error()
    assert L.slicegcn_strerror(binding.EWORKSPACE) == b"workspace missing or too small"
    assert L.slicegcn_strerror(-99) == b"unknown status"


def test_widened_entry_points_validate_before_device_work(L):
    vp = ctypes.c_void_p
    one = vp(256)  # a non-NULL dummy pointer: validation must fail before anything dereferences it
    assert L.slicegcn_linear_fwd(None, 4, 4, 4, 4, None, None, 0, None, 4, None, 0, None) == binding.EINVAL
    assert L.slicegcn_linear_fwd(one, 3, 4, 4, 4, one, None, 0, one, 4, None, 0, None) == binding.EINVAL      # ldx < w_in
    assert L.slicegcn_linear_fwd(one, 4, 4, 4, 4, one, None, 1, one, 4, None, 0, None) == binding.EINVAL      # ReLU, no mask
    assert L.slicegcn_linear_fwd(one, 4, 4, 4, 4, one, None, 7, one, 4, None, 0, None) == binding.EINVAL      # unknown act
    assert L.slicegcn_linear_bwd(one, 4, 4, 4, 4, one, 0, None, 0, one, 4, None, 0, one, None, None, 0, None) == binding.EWORKSPACE
    assert L.slicegcn_linear_bwd_workspace_bytes(0, 4, 4) == 0
    assert L.slicegcn_linear_bwd_workspace_bytes(5000, 25, 64) == -(-(5 * (25 * 64 + 64) * 4) // 256) * 256
    assert L.slicegcn_softmax_ce(None, 4, 4, 4, None, None, None, 0, None, 0, None) == binding.EINVAL
    assert L.slicegcn_softmax_ce(one, 3, 4, 4, one, one, None, 0, one, 4096, None) == binding.EINVAL          # ld < classes
    assert L.slicegcn_softmax_ce(one, 4, 4, 4, one, one, None, 0, None, 0, None) == binding.EWORKSPACE
    assert L.slicegcn_softmax_ce_workspace_bytes(0) == 0 and L.slicegcn_softmax_ce_workspace_bytes(1000) == 256
    assert L.slicegcn_accumulate(None, 4, None, 4, 4, 4, None) == binding.EINVAL
    assert L.slicegcn_accumulate(one, 3, one, 4, 4, 4, None) == binding.EINVAL
    assert L.slicegcn_adam_step(None, None, None, None, 4, 1e-3, 0.9, 0.999, 1e-8, 0.0, 1, None) == binding.EINVAL
    assert L.slicegcn_adam_step(one, one, one, one, 4, 1e-3, 0.9, 0.999, 1e-8, 0.0, 0, None) == binding.EINVAL  # step < 1
    assert L.slicegcn_adam_step(one, one, one, one, 4, 1e-3, 1.0, 0.999, 1e-8, 0.0, 1, None) == binding.EINVAL  # beta1 = 1


def test_gradients_in_place_are_refused_where_rows_are_shared(L):
    """dX in dY's rows: one workgroup forms whole rows up to 128 columns; wider ones are formed by several, of which one
    would store before another has read.  Columns beside each other in one buffer are no overlap."""
    vp, base = ctypes.c_void_p, 1 << 20
    W = vp(256)

    def bwd(w, dX, ld):
        return L.slicegcn_linear_bwd(W, w, 64, w, w, W, 0, None, 0, vp(base), ld, vp(dX), ld, None, None, None, 0, None)
    for w, dX, ld in ((129, base, 129), (200, base, 256), (200, base + 400, 256), (1000, base - 40, 1024)):
        assert bwd(w, dX, ld) == binding.EINVAL, (w, dX, ld)
        assert b"in place" in L.slicegcn_last_error()


class _Destroys:
    def __init__(self):
        self.handles = []

    def slicegcn_graph_destroy(self, h):
        self.handles.append(h)


def test_destroy_waits_for_the_handles_device_and_frees_it_all_the_same(monkeypatch):
    """The memory of a handle goes back to the allocator once its own device has finished, whichever one is current; if the
    wait fails the handle is freed nevertheless."""
    lib, waits = _Destroys(), []
    monkeypatch.setattr(binding, "lib", lambda: lib)
    monkeypatch.setattr(torch.cuda, "synchronize", lambda device=None: waits.append(device))
    block = types.SimpleNamespace(device=torch.device("cuda", 3))
    g = binding.Graph(11, [block])
    g.destroy()
    assert waits == [torch.device("cuda", 3)] and lib.handles == [11] and g._memory == []

    def broken(device=None):
        raise RuntimeError("device lost")
    monkeypatch.setattr(torch.cuda, "synchronize", broken)
    g = binding.Graph(12, [block])
    with pytest.raises(RuntimeError, match="device lost"):
        g.destroy()
    assert lib.handles == [11, 12] and g._memory == [] and g._ws is None
    with pytest.raises(ValueError):
        g.handle


def test_build_workspace_of_a_refused_build_is_zero(L):
    """What the build would refuse needs no workspace: the caller then gets the build's own error, not one of its allocator."""
    size, big = L.slicegcn_build_workspace_bytes, 2**31 - 1
    assert size(1000, 100, 3) > 8000
    assert size(2**30, 1000, 3) == 0            # both directions of 2^30 edges exceed int32
    assert size(2**30 - 500, 1000, 3) == 0      # ... and these with the self loops
    assert size(2**30 - 501, 1000, 3) > 0
    assert size(big, big, 0) > 0 and size(big, big, 2) == 0 and size(big, 2**31, 0) == 0
    for flags in (1 << 20, 4 | 8, 16 | 32):
        assert size(1000, 100, flags) == 0


def test_build_out_of_memory_is_the_librarys_error(L, monkeypatch):
    def full(*a, **k):
        raise torch.OutOfMemoryError("tried to allocate 60 GiB")
    monkeypatch.setattr(torch, "empty", full)
    none = torch.zeros(0, dtype=torch.int64)
    with pytest.raises(binding.SliceGCNError) as e:
        binding.slicegcn_build_norm_csr(none, none, 100)
    assert e.value.status == binding.ENOMEM and "60 GiB" in str(e.value)
