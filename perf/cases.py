"""The work a user of this package has it do, as cases that can be timed: graph construction, single
aggregations, whole slice models forward and backward, inference and complete training epochs.

The listed sizes are the benchmark workloads of ``synth.configs`` (cfg1 to cfg5 and ``comm``) and sizes the
tests use; ``draw`` spreads over the ranges between them.  Everything is fp32, the one data type the library has.
A case names its kind of work and its sizes:

  aggregate  one ``slicegcn_spmm_slice`` call on one feature slice
  build      one ``slicegcn_build_norm_csr`` call, edge list to handle
  slices     ``SliceStack`` forward and backward for a given upstream gradient (k = 1: one slice model on a GPU
             of its own)
  infer      ``SliceStack`` forward and the classifier's logits
  train      ``SliceGCNTrainer.epoch``: forward, loss, backward, update
"""
from __future__ import annotations

import math

import torch

from paper_2408_11500_amd import binding as B
from paper_2408_11500_amd.stack import Classifier, Optimizer, SliceStack
from paper_2408_11500_amd.train import SliceGCNTrainer
from synth import graphs

# planted communities of the ``comm`` workload: block size, neighbours drawn inside and outside of it
COMM, COMM_IN, COMM_OUT = 512, 24, 2


def listed():
    return [
        # One aggregation on a small graph (cfg1's), as a call of its own: latency and launches are all there is.
        dict(name="aggregate_small", kind="aggregate", graph="er", n=2048, m=4096, width=64, padded=True, directed=False,
             prescaled=False),
        # A directed graph aggregated along its reversed edges, on a slice kept as a plain contiguous 25-wide matrix
        # (no padding, rows not on 16-byte boundaries): what a user has who slices with torch.
        dict(name="aggregate_directed_ragged", kind="aggregate", graph="rmat", n=100_003, m=1_500_007, width=25, padded=False,
             directed=True, prescaled=False),
        # The headline aggregation (cfg5): one 32-wide slice over 10 M nodes and 310 M stored entries.
        dict(name="aggregate_large", kind="aggregate", graph="rmat", n=10_000_000, m=150_000_000, width=32, padded=True,
             directed=False, prescaled=False),
        # A new graph arrives: edge list of a co-purchase graph (cfg4) to the handle every other call takes.
        dict(name="build_copurchase", kind="build", graph="rmat", n=2_449_029, m=62_000_000, directed=False, order="natural"),
        # Training on a small graph (cfg1), call by call.
        dict(name="train_small", kind="train", graph="er", n=2048, m=4096, feat=128, k=2, hidden=64, layers=2, classes=8,
             fusion=False, replay=False),
        # The same for a slightly larger graph with the epoch captured into a HIP graph; widths that fill no tile.
        dict(name="train_small_replay", kind="train", graph="er", n=5000, m=20_000, feat=100, k=3, hidden=96, layers=3, classes=7,
             fusion=False, replay=True),
        # The citation graph (cfg2), the ordinary training run.
        dict(name="train_citation", kind="train", graph="rmat", n=169_343, m=1_185_401, feat=128, k=4, hidden=256, layers=3,
             classes=40, fusion=False, replay=False),
        # The feature-fusion variant of it: a learned projection feeds every slice model and takes their input gradients.
        dict(name="train_fusion", kind="train", graph="rmat", n=169_343, m=1_185_401, feat=128, k=4, hidden=256, layers=3,
             classes=40, fusion=True, replay=False),
        # A dense social graph with wide slices (cfg3): 301 feature columns per slice, about 490 neighbours per node.
        dict(name="train_social", kind="train", graph="rmat", n=232_965, m=57_000_000, feat=602, k=2, hidden=256, layers=2,
             classes=41, fusion=False, replay=False),
        # A co-purchase graph (cfg4): narrow first layer, 64-wide hidden layers, 2.4 M nodes.
        dict(name="train_copurchase", kind="train", graph="rmat", n=2_449_029, m=62_000_000, feat=100, k=4, hidden=256, layers=3,
             classes=47, fusion=False, replay=False),
        # One of the eight slice models of the largest workload (cfg5), as one GPU of the paper's setup runs it.
        dict(name="slice_large", kind="slices", graph="rmat", n=10_000_000, m=150_000_000, feat=32, k=1, hidden=32, layers=3,
             order="natural", product="aggregate"),
        # Inference on a graph with communities (comm) whose handle carries the breadth-first row order.
        dict(name="infer_communities", kind="infer", graph="comm", n=2_000_000, m=2_000_000 * (COMM_IN + COMM_OUT), feat=128, k=4,
             hidden=128, layers=2, classes=16, order="bfs", product="aggregate"),
    ]


# ---- drawn cases ------------------------------------------------------------------------------------------------------

def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _draw_graph(rng, n_max, m_max):
    n = _log(rng, 1000, n_max)
    graph = rng.choice(["rmat", "rmat", "er"])
    m = int(n * math.exp(rng.uniform(math.log(2.0), math.log(60.0))))
    return dict(graph=graph, n=n, m=max(n, min(m, m_max, n * n // 400)))  # R-MAT needs room for distinct pairs


def _draw(rng):
    kind = rng.choice(["aggregate", "aggregate", "build", "slices", "infer", "train", "train", "train"])
    if kind == "aggregate":
        return dict(kind=kind, **_draw_graph(rng, 10_000_000, 150_000_000), width=_log(rng, 8, 320), padded=rng.random() < 0.75,
                    directed=rng.random() < 0.25, prescaled=rng.random() < 0.3)
    if kind == "build":
        return dict(kind=kind, **_draw_graph(rng, 2_500_000, 62_000_000), directed=rng.random() < 0.25,
                    order=rng.choice(["natural", "natural", "natural", "degree", "bfs"]))
    g = _draw_graph(rng, 2_500_000, 62_000_000)
    k = rng.choice([1, 2, 2, 3, 4, 4, 5, 8])
    feat = _log(rng, 16 * k, 602)
    hidden = k * _log(rng, 16, 512 // k if k > 2 else 128)
    model = dict(feat=feat, k=k, hidden=hidden, layers=rng.choice([1, 2, 2, 3, 3]))
    if kind == "slices":
        return dict(kind=kind, **g, **model, order="natural", product=rng.choice(["aggregate", "aggregate", "auto"]))
    if kind == "infer":
        return dict(kind=kind, **g, **model, classes=_log(rng, 2, 64), order=rng.choice(["natural", "natural", "bfs"]),
                    product=rng.choice(["aggregate", "aggregate", "auto"]))
    return dict(kind=kind, **g, **model, classes=_log(rng, 2, 64), fusion=rng.random() < 0.25,
                replay=g["n"] < 50_000 and rng.random() < 0.5)


def _state_bytes(case):
    """About what prepare() holds on the GPU."""
    n, nnz = case["n"], _nnz(case)
    if case["kind"] == "aggregate":
        return 24 * nnz + 8 * n * case["width"]
    if case["kind"] == "build":
        return 40 * nnz
    w, h, k = _slice_width(case), case["hidden"] // case["k"], case["k"]
    per_slice = 2 * (w + 32) + 2 * case["layers"] * (h + 32)
    return 24 * nnz + 4 * n * (k * per_slice + 2 * case["hidden"] + 4 * (w + h + 64) +
                               (4 * case["hidden"] + 3 * case["feat"] if case["kind"] == "train" else 0))


def draw(rng):
    """One more case of the same ranges: sizes log-uniform, at most as costly as the largest listed one."""
    flops = max(work(c)["flops"] for c in listed() if c["kind"] == "train")
    while True:
        case = _draw(rng)
        if work(case)["flops"] <= flops and _state_bytes(case) <= 40e9:
            return case


# ---- inputs -----------------------------------------------------------------------------------------------------------

def _nnz(case):
    """Stored entries of the normalised adjacency (for ``comm`` an upper bound: a few drawn pairs repeat)."""
    return (1 if case.get("directed") else 2) * case["m"] + case["n"]


def _slice_width(case):
    return -(-case["feat"] // case["k"])


def _edges(case, seed):
    if case["graph"] == "er":
        return graphs.erdos_renyi(case["n"], case["m"], seed, device="cuda")
    if case["graph"] == "comm":
        return graphs.planted_communities(case["n"], COMM, COMM_IN, COMM_OUT, seed, device="cuda")
    return graphs.rmat(case["n"], case["m"], seed, device="cuda")


def _flags(case):
    order = {"natural": 0, "degree": B.REORDER_DEGREE, "bfs": B.REORDER_BFS}[case.get("order", "natural")]
    return B.ADD_SELF_LOOPS | (0 if case.get("directed") else B.SYMMETRIZE) | order


def _glorot(gen, rows, cols):
    return (torch.rand((rows, cols), generator=gen, device="cuda") * 2 - 1) * math.sqrt(6.0 / (rows + cols))


def _bias(gen, width):
    return torch.randn(width, generator=gen, device="cuda") * 0.05


def _set_slice_params(stack, gen):
    for i in range(stack.k):
        for layer, (wi, wo) in enumerate(stack.widths):
            stack.set_params(i, layer, _glorot(gen, wi, wo), _bias(gen, wo), _glorot(gen, wi, wo), _bias(gen, wo))
    stack.E.copy_(torch.randn(stack.E.shape, generator=gen, device="cuda") * 0.1)


def _set_dense_params(mlp, gen):
    mlp.set_params(_glorot(gen, *mlp.W1.shape), _bias(gen, mlp.b1.numel()), _glorot(gen, *mlp.W2.shape), _bias(gen, mlp.b2.numel()))


def prepare(case, seed):
    gen = torch.Generator(device="cuda").manual_seed(seed)
    src, dst = _edges(case, seed)
    n, kind = case["n"], case["kind"]
    if kind == "build":
        return dict(case=case, src=src, dst=dst, flags=_flags(case))
    g = B.slicegcn_build_norm_csr(src, dst, n, _flags(case))
    del src, dst
    if kind == "aggregate":
        w = case["width"]
        ld = (w + 31) // 32 * 32 if case["padded"] else w
        X = torch.randn((n, ld), generator=gen, device="cuda")
        if case["prescaled"]:  # a constant operand is scaled once, ahead of the calls
            B.slicegcn_scale_rows(g, X, X, width=w)
        ws = torch.empty(B.slicegcn_spmm_workspace_bytes(g, w, case["directed"]), dtype=torch.uint8, device="cuda")
        return dict(case=case, g=g, X=X[:, :w], Y=torch.empty((n, ld), device="cuda")[:, :w], ws=ws)
    X = torch.randn((n, case["feat"]), generator=gen, device="cuda")
    k, hs = case["k"], case["hidden"] // case["k"]
    if kind == "train":
        y = X[:, :case["classes"]].argmax(dim=1)  # something to learn: the largest of the first features
        tr = SliceGCNTrainer(g, X, y, k, hs, case["layers"], case["hidden"], case["classes"], use_ff=case["fusion"],
                             graph_replay=case["replay"])
        _set_slice_params(tr.stack, gen)
        _set_dense_params(tr.cls, gen)
        if tr.ff is not None:
            _set_dense_params(tr.ff, gen)
        tr.start(1e-3, 1e-5, 1000)
        # a run under way, as after loading a checkpoint: Adam's moments have a history, so an update is a smooth
        # function of the gradient (a first step is its sign, which rounding decides wherever a gradient is near zero)
        tr.opt.V.fill_(1e-6)
        tr.opt.t = 100
        return dict(case=case, g=g, trainer=tr, epoch=100)
    slices, _ = B.slicegcn_slice_strategy(case["feat"], k)
    order = B.LAYER_ORDER_AUTO if case["product"] == "auto" else 0
    stack = SliceStack(g, n, k, slices[0][1] - slices[0][0], hs, case["layers"], order=order)
    for i, (a, b) in enumerate(slices):
        B.slicegcn_slice_feature(X, a, b, stack.X[i])
    _set_slice_params(stack, gen)
    stack.prepare_inputs()
    if kind == "slices":
        opt = Optimizer([stack], lr_max=1e-3)  # keeps the gradients of all layers in one buffer
        return dict(case=case, g=g, stack=stack, opt=opt, dH=torch.randn((n, k * hs), generator=gen, device="cuda"))
    cls = Classifier(n, k * hs, case["hidden"], case["classes"])
    _set_dense_params(cls, gen)
    return dict(case=case, g=g, stack=stack, cls=cls)


# ---- one pass ---------------------------------------------------------------------------------------------------------

class _DeviceArray:
    """A handle's borrowed device array, readable as a tensor; keeps the handle alive."""

    def __init__(self, g, ptr, count, typestr):
        self.g = g
        self.__cuda_array_interface__ = dict(data=(ptr, False), shape=(count,), typestr=typestr, strides=None, version=2)


def _handle_arrays(g):
    v = g.view()
    arrays = dict(rowptr=(v.rowptr, v.n_nodes + 1, "<i4"), colidx=(v.colidx, v.nnz, "<i4"), deg=(v.deg, v.n_nodes, "<i4"),
                  dinv=(v.dinv, v.n_nodes, "<f4"), vals=(v.vals, v.nnz, "<f4"))
    if v.order:
        arrays["order"] = (v.order, v.n_nodes, "<i4")
    out = {}
    for name, where in arrays.items():
        out[name] = torch.as_tensor(_DeviceArray(g, *where), device="cuda")
        out[name].handle = g  # the arrays belong to the handle: whoever holds one of these tensors holds it too
    return out


def run(state):
    case, kind = state["case"], state["case"]["kind"]
    if kind == "aggregate":
        return B.slicegcn_spmm_slice(state["g"], state["X"], state["Y"], transpose=case["directed"], ws=state["ws"],
                                     prescaled=case["prescaled"])
    if kind == "build":
        return _handle_arrays(B.slicegcn_build_norm_csr(state["src"], state["dst"], case["n"], state["flags"]))
    if kind == "train":
        tr = state["trainer"]
        loss = tr.epoch(state["epoch"])
        state["epoch"] = (state["epoch"] + 1) % 1000
        opt = tr.opt
        return dict(loss=loss, H=tr.stack.Hcat, dH=tr.dH, gradients=opt.G, parameters=opt.P, m=opt.M, v=opt.V)
    stack = state["stack"]
    if kind == "slices":
        H = stack.forward()
        stack.backward(state["dH"])
        return dict(H=H, gradients=state["opt"].G)
    cls = state["cls"]
    H = stack.forward()
    B.slicegcn_linear_fwd(H, cls.W1, cls.b1, cls.A, cls.mask, act=B.ACT_RELU)
    B.slicegcn_linear_fwd(cls.A, cls.W2, cls.b2, cls.logits, None, act=B.ACT_NONE)
    return dict(H=H, logits=cls.logits)


# ---- what a pass cannot do without ------------------------------------------------------------------------------------

def work(case):
    n, nnz, kind = case["n"], _nnz(case), case["kind"]
    if kind == "aggregate":
        w = case["width"]
        values = 0 if case["prescaled"] else 4
        return {"bytes": (4 + values) * nnz + 4 * (n + 1) + 8 * n * w, "flops": 2 * nnz * w}
    if kind == "build":
        return {"bytes": 16 * case["m"] + 8 * nnz + 4 * (n + 1) + 8 * n, "flops": nnz}
    k, hs, layers = case["k"], case["hidden"] // case["k"], case["layers"]
    width, back = _slice_width(case), kind in ("slices", "train")
    fusion = bool(case.get("fusion"))
    flops = 0
    for layer in range(layers):
        wi = width if layer == 0 else hs
        wa = min(wi, hs) if case.get("product") == "auto" else wi
        input_gradient = back and (layer > 0 or fusion)
        flops += 2 * nnz * wa * (2 if input_gradient else 1)
        flops += 4 * n * wi * hs * (1 + (1 if back else 0) + (1 if input_gradient else 0))
    flops *= k
    # the graph, the features and the representation; the gradient of the representation where there is one
    nbytes = 8 * nnz + 4 * (n + 1) + 4 * n * case["feat"] + 4 * n * k * hs * (2 if back else 1)
    if kind in ("infer", "train"):
        dense = 2 * n * (k * hs * case["hidden"] + case["hidden"] * case["classes"])
        flops += dense * (3 if kind == "train" else 1)
        nbytes += 4 * n * case["classes"] if kind == "infer" else 4 * n
    if fusion:
        flops += 2 * n * case["feat"] * (2 * case["feat"] + 3 * width)
    return {"bytes": nbytes, "flops": flops}


def tolerance(case):
    if case["kind"] == "build":
        return {"rel": 1e-6, "max": 1e-6}  # whole numbers exactly; 1/sqrt and its products to a unit in the last place
    if case["kind"] == "aggregate":
        return {"rel": 2e-6, "max": 2e-5}  # fp32 sums of a row's entries, in another order
    if case["kind"] == "infer":
        return {"rel": 1e-5, "max": 2e-4}
    # An activation within rounding of zero (a few in 10^8) may pass in one implementation and not in another; each such
    # node moves a weight gradient, itself a sum of mostly cancelling terms, by far more than rounding does.
    return {"rel": 1e-3, "max": 0.02}
