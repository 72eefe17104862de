"""The builder's distribution and sort at the sizes where they change their way: one tile of edges, one and two distributing passes, buckets sorted with 4 to 32
keys per thread, buckets cut once more (and parts of theirs that go through a bitmap: repeats), 64-bit keys, empty rows."""
import numpy as np
import pytest
import torch

import paper_2408_11500_amd as sg

pytestmark = pytest.mark.gpu


class _Array:
    def __init__(self, ptr, count, typestr):
        self.__cuda_array_interface__ = dict(data=(ptr, False), shape=(count,), typestr=typestr, strides=None, version=2)


def arrays(g):
    v = g.view()
    take = lambda p, c, t: torch.as_tensor(_Array(p, c, t), device="cuda").clone()
    return (take(v.rowptr, v.n_nodes + 1, "<i4"), take(v.colidx, v.nnz, "<i4") if v.nnz else torch.empty(0, dtype=torch.int32, device="cuda"),
            take(v.deg, v.n_nodes, "<i4"), take(v.dinv, v.n_nodes, "<f4"), take(v.vals, v.nnz, "<f4") if v.nnz else torch.empty(0, device="cuda"))


def reference(src, dst, n, flags):
    """Rows and columns by torch.unique over row * n + col."""
    keep = src != dst
    u, v = src[keep], dst[keep]
    keys = [u * n + v]
    if flags & sg.binding.SYMMETRIZE:
        keys.append(v * n + u)
    if flags & sg.binding.ADD_SELF_LOOPS:
        d = torch.arange(n, device="cuda")
        keys.append(d * n + d)
    k = torch.unique(torch.cat(keys))
    row, col = k // n, k % n
    deg = torch.bincount(row, minlength=n)
    rowptr = torch.cat([torch.zeros(1, dtype=torch.int64, device="cuda"), deg.cumsum(0)])
    # 1 / sqrt in fp64, rounded: off by at most one unit where torch's and the library's fp64 roots differ
    dinv = (1.0 / torch.sqrt(deg.clamp(min=1).double())).float()
    return rowptr, row, col, deg, dinv


def check(src, dst, n, flags):
    src, dst = (torch.as_tensor(a, dtype=torch.int64).cuda() for a in (src, dst))
    g = sg.slicegcn_build_norm_csr(src, dst, n, flags)
    rowptr, colidx, deg, dinv, vals = arrays(g)
    w_rowptr, row, col, w_deg, w_dinv = reference(src, dst, n, flags)
    assert torch.equal(rowptr.long(), w_rowptr) and torch.equal(colidx.long(), col) and torch.equal(deg.long(), w_deg)
    assert torch.allclose(dinv, w_dinv, rtol=2.0 ** -23, atol=0)
    assert torch.equal(vals, dinv[row] * dinv[col])
    if not flags & sg.binding.SYMMETRIZE and n <= 100_000:  # the transposed pattern, through an aggregation of ones
        X = torch.ones((n, 4), device="cuda")
        Y = torch.empty_like(X)
        sg.slicegcn_spmm_slice(g, X, Y, transpose=True)
        want = torch.zeros(n, dtype=torch.float64, device="cuda").index_add_(0, col, (dinv[row] * dinv[col]).double())
        assert float((Y[:, 0].double() - want).abs().max()) <= 1e-5 * float(want.max().clamp(min=1))  # sums of n terms of one sign in fp32
    g.destroy()


ALL = sg.binding.SYMMETRIZE | sg.binding.ADD_SELF_LOOPS


@pytest.mark.parametrize("flags", [0, sg.binding.SYMMETRIZE, sg.binding.ADD_SELF_LOOPS, ALL])
@pytest.mark.parametrize("n,m", [(1, 0), (1, 3), (2, 5), (3, 0), (64, 1023), (1000, 513), (1025, 2048), (9000, 3), (70_000, 40_000), (5000, 300_000),
                                 (300_000, 700_000), (700_000, 90)])
def test_random_pairs(n, m, flags):
    rng = np.random.default_rng(n + m)
    check(rng.integers(0, n, m), rng.integers(0, n, m), n, flags)


@pytest.mark.parametrize("flags", [0, sg.binding.SYMMETRIZE, sg.binding.ADD_SELF_LOOPS, ALL])
@pytest.mark.parametrize("n,m", [(100, 300), (2047, 1024), (2048, 1024), (2048, 1025), (2, 3072), (2000, 3072), (2000, 3073), (1_048_576, 3071),
                                 (1_048_576, 3072), (1_048_576, 3073), (1_048_577, 3072)])
def test_one_tile_of_edges(n, m, flags):
    """Up to 3072 edges and diagonal entries, up to 512 buckets: no counting before the distribution; and one more of either."""
    rng = np.random.default_rng(n + m)
    src, dst = rng.integers(0, n, m), rng.integers(0, n, m)
    check(src, dst, n, flags)
    src[m // 2] = n
    with pytest.raises(sg.binding.SliceGCNError, match=r"1 edge\(s\) name a node outside"):
        check(src, dst, n, flags)


@pytest.mark.parametrize("n,m", [(1 << 24, 5000), ((1 << 24) + 1, 5000), ((1 << 24) + 1, 20_000_000)])
def test_few_keys_per_bucket(n, m):
    """From 2^24 nodes on 32-bit keys would take a bucket for every 128 rows: 64 bits for fewer than 150 keys a bucket (the last has 152)."""
    gen = torch.Generator(device="cuda").manual_seed(m)
    src, dst = (torch.randint(0, n, (m,), generator=gen, device="cuda") for _ in range(2))
    dst[:400] = src[:400]                                # self pairs
    src[400:20_400 if m > 10 ** 6 else 2400] = n - 1     # a row beyond a bucket's others
    check(src, dst, n, sg.binding.SYMMETRIZE)
    check(src, dst, n, 0)


@pytest.mark.parametrize("keys", [1, 1023, 1024, 1025, 2047, 2048, 2049, 4095, 4096, 4097, 8191, 8192, 8193, 16383, 16384, 16385, 50_000])
def test_one_row(keys):
    """One row of so many pairs (with the repeats a third more), the others nearly empty: every size of the
    register sort, and the row whose bucket is cut once more."""
    rng = np.random.default_rng(keys)
    n = 600_000 if keys > 8193 else 40_000
    col = rng.choice(n - 1, keys, replace=False) + 1
    src = np.concatenate([np.zeros(keys, np.int64), rng.integers(0, n, 100)])
    dst = np.concatenate([col, rng.integers(0, n, 100)])
    check(src, dst, n, 0)
    again = rng.integers(0, keys, keys // 3)
    check(np.concatenate([src, src[again]]), np.concatenate([dst, dst[again]]), n, ALL)


def test_large_buckets_of_many_rows():
    """Neighbouring rows that fill a bucket many times over, some of them longer than a register sort, with empty rows between."""
    rng = np.random.default_rng(3)
    n = 30_000
    length = [5000, 3000, 9000, 0, 8192, 8193, 1, 0, 0, 20_000, 7000, 1200, 8000, 300, 25_000, 1]
    src = np.concatenate([np.full(c, 128 + r) for r, c in enumerate(length)])
    dst = np.concatenate([rng.choice(n, c, replace=False) for c in length])
    p = rng.permutation(src.size)
    check(src[p], dst[p], n, 0)
    check(np.concatenate([src, src]), np.concatenate([dst, dst]), n, ALL)


def test_all_pairs_alike():
    """Pairs repeated far beyond what a part of a bucket sorts in registers, in both orientations; few keys and many around them."""
    check(np.tile([7, 9], 50_000), np.tile([9, 7], 50_000), 1000, ALL)
    rng = np.random.default_rng(1)
    n = 3_000_000   # wide enough for parts of several bitmaps
    src, dst = np.concatenate([np.full(60_000, 5), rng.integers(0, n, 400_000)]), np.concatenate([rng.integers(100, 104, 60_000), rng.integers(0, n, 400_000)])
    check(src, dst, n, ALL)


@pytest.mark.parametrize("n,low", [(300, 256), (2048, 2048), (2049, 2048), (9000, 2048), (10_000, 2), (200_000, 64), (3_000_000, 1024), (2 ** 24, 1024), (40_000_003, 16)])
def test_parts_cut_again(n, low):
    """Hubs whose parts are cut once, twice and three times before a workgroup sorts them, and parts that hold repeats when no bits are left to
    cut by (`low` values: one of them, or nearly all of them)."""
    rng = np.random.default_rng(n)
    k = min(n - 1, 120_000)
    rows = [(np.full(k, 3), n - 1 - np.arange(k)),                                     # neighbours side by side
            (np.full(k, 4), rng.choice(n, k, replace=False)),                          # and all over
            (np.full(70_000, 6), min(2048, n - low) + rng.integers(0, max(low - 1, 1), 70_000)),     # one part of repeats
            (np.full(40_000, n - 2), np.full(40_000, n - 1)),                          # one pair
            (rng.integers(0, n, 3000), rng.integers(0, n, 3000))]
    src, dst = (np.concatenate([r[i] for r in rows]) for i in (0, 1))
    p = rng.permutation(src.size)
    check(src[p], dst[p], n, 0)
    check(src[p], dst[p], n, ALL)
    check(src, dst, n, ALL)      # wavefronts whose keys are all of one part


def test_most_candidates_in_one_bucket():
    """2^31 - 1 candidate entries, the most that is accepted, nearly all of them in one bucket: its tiles are counted in 32 bits."""
    n, m = 1000, 2 ** 31 - 1
    src, dst = (torch.full((m,), v, dtype=torch.int64, device="cuda") for v in (7, 9))
    src[-3:], dst[-3:] = torch.tensor([999, 7, 0], device="cuda"), torch.tensor([0, 8, 999], device="cuda")
    g = sg.slicegcn_build_norm_csr(src, dst, n, 0)
    del src, dst
    rowptr, colidx, deg, _, _ = arrays(g)
    assert torch.nonzero(deg)[:, 0].tolist() == [0, 7, 999] and deg[[0, 7, 999]].tolist() == [1, 2, 1]
    assert colidx.tolist() == [999, 8, 9, 0] and int(rowptr[-1]) == 4
    X = torch.randn((n, 4), device="cuda")
    Y = torch.empty_like(X)
    sg.slicegcn_spmm_slice(g, X, Y, transpose=True)
    # row 9 of the transposed pattern: 1 / sqrt(2 entries in row 7) times 1 (row 9 is empty)
    assert torch.allclose(Y[9], X[7] / 2 ** 0.5, rtol=1e-6, atol=0) and not bool(Y[1:8].any())
    g.destroy()
    torch.cuda.empty_cache()


def test_star():
    n = 300_001
    check(np.zeros(n - 1, np.int64), np.arange(1, n), n, ALL)
    check(np.arange(1, n), np.full(n - 1, n - 1), n, 0)


@pytest.mark.parametrize("n,m", [(2 ** 22, 3_000_000), (2 ** 24, 9_000_000), (40_000_003, 2_000_000)])
def test_two_passes_and_wide_keys(n, m):
    """Keys that fill 32 bits exactly (2^24 nodes), and 64-bit keys (40 M nodes); a hub among them."""
    g = torch.Generator(device="cuda").manual_seed(m)
    src = torch.randint(0, n, (m,), generator=g, device="cuda")
    dst = torch.randint(0, n, (m,), generator=g, device="cuda")
    src[:20_000] = n - 1
    dst[0], dst[1] = n - 2, 0
    check(src, dst, n, ALL)
    check(src[:100_000], dst[:100_000], n, 0)


def test_bad_ids_are_counted():
    src, dst = torch.tensor([0, 5, -1, 3]).cuda(), torch.tensor([1, 2, 2, 10]).cuda()
    with pytest.raises(sg.binding.SliceGCNError, match="2 edge"):
        sg.slicegcn_build_norm_csr(src, dst, 10, ALL)
