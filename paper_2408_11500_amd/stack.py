"""Call sequence of one full-batch pass over k feature slices (the inner loops of the paper's
training algorithm): for every slice, L layer evaluations, then slice encoding + CONCAT, and
the same chain backwards.  This module only owns buffers (torch device tensors) and orders the
library calls; every arithmetic step is a kernel of ``libslicegcn.so``.
"""
from __future__ import annotations

from typing import NamedTuple

import torch

from . import binding as B

# Slices run in groups whose layers share their launches while the rows one launch works on stay within this many bytes
# (see SliceStack.group).  Training epochs at 64 MB / 1 GB / 4 GB, 3 layers of 64-wide slices: 60 k nodes, 5 slices 2.31 / 1.86 / 1.86
# ms; 169 k nodes, 4 slices 3.62 / 3.42 / 3.42; 1 M nodes, 4 slices 20.8 / 20.8 / 19.9.  At 16 GB 2.4 M nodes, 4 slices run as a group
# too: 74.1 -> 73.1 ms for 6.5 GB more.
GROUP_BYTES = 4 << 30


def padded_ld(width: int) -> int:
    """Leading dimension for a slice operand: every row starts on a 128-byte boundary, so a gathered
    row (or a column pass over it) touches the fewest cache lines (a 301-wide slice at ld 304 has
    every other row straddle one line more: 8.7 vs 7.8 ms per aggregation)."""
    return (width + 31) // 32 * 32


try:  # torch's own comparison of many tensors' type, device, shape and strides in one call
    from torch._C._dynamo.guards import TensorGuards
except ImportError:
    TensorGuards = None


class TensorLayouts:
    """Whether a list of tensors (or None) still is the memory, types, devices, shapes and strides of the list it was made
    from.  51 tensors: 11 us; with tuples of these attributes (TensorGuards = None) 30, a quarter of a pass over 2048 nodes."""

    NONE = torch.empty(0)  # stands where there is none

    def __init__(self, tensors=()):
        self.gaps = type(None) in map(type, tensors)
        if self.gaps:
            tensors = self._filled(tensors)
        self.ptrs = list(map(torch.Tensor.data_ptr, tensors))
        self.twins = ()
        if len(set(map(id, tensors))) < len(tensors):  # TensorGuards takes no tensor twice (slices may share inputs or weights)
            first = {}
            self.twins = [(i, first[id(t)]) for i, t in enumerate(tensors) if first.setdefault(id(t), i) != i]
            self.unique = sorted(first.values())
            tensors = [tensors[i] for i in self.unique]
        self.guards = TensorGuards and tensors and TensorGuards(*tensors, dynamic_dims_sizes=None, dynamic_dims_strides=None)
        self.layouts = None if self.guards else self._layouts(tensors)

    @classmethod
    def _filled(cls, tensors):
        return [cls.NONE if t is None else t for t in tensors]

    @staticmethod
    def _layouts(tensors):
        return [(t.dtype, t.device, t.shape, t.stride()) for t in tensors]

    def same(self, tensors) -> bool:
        if self.gaps:
            tensors = self._filled(tensors)
        try:
            if list(map(torch.Tensor.data_ptr, tensors)) != self.ptrs:
                return False
        except TypeError:  # None, where there was none
            return False
        if self.twins:
            if any(tensors[i] is not tensors[j] for i, j in self.twins):
                return False
            tensors = [tensors[i] for i in self.unique]
        return self.guards.check(*tensors) if self.guards else self._layouts(tensors) == self.layouts


class LayerPlan(NamedTuple):
    """Argument blocks of one direction of a pass, and what they were laid out for."""
    ios: list      # per layer: LayerIo of every slice
    shapes: list   # per layer: LayerGroup of every slice
    alike: bool    # all slices fit one group
    fused: bool    # the encoding rides on the last layer
    layouts: TensorLayouts


class SliceStack:
    def __init__(self, graph: B.Graph, n_nodes: int, k: int, first_width: int, slice_hidden: int, layers: int,
                 device="cuda", slice_encoding: bool = True, act_last: int = B.ACT_RELU,
                 shared_input: torch.Tensor | None = None, cache_first_aggregation: bool = False,
                 fuse_encoding: bool = True, order: int = 0, scaled: bool | None = None, streams: int = 1):
        """``shared_input``: with feature fusion every slice model reads the same fused n x first_width
        matrix; the stack then also returns the gradient with respect to it (``dXin``).
        ``order``: 0 (aggregate first), LAYER_TRANSFORM_FIRST or LAYER_ORDER_AUTO, applied to every layer.
        ``scaled``: keep the activations between aggregate-first layers as D~^-1/2 H (the layer flags IN_SCALED /
        OUT_SCALED), so that no aggregation reads the stored values; the raw slices are then scaled once by
        ``prepare_inputs`` (call it after filling ``X``).  None = by graph size: the layout pays where the
        aggregation streams the stored entries from memory (measured: -3 % per step at 126 M and 310 M entries) and
        costs a little where the whole graph sits in cache and the dense kernels' extra row factors show
        (+3 % at 2.5 M entries), so it is used from 16 M stored entries on.
        ``streams``: how many slice models run at a time, each on a HIP stream of its own (the slice models are
        independent between the raw features and the concatenation, and a graph handle is read-only, so they only
        need workspaces of their own).  1 = on the caller's stream: in groups whose layers share
        their launches (see ``group``), or one after the other on large graphs.  More gains nothing where slices form groups
        (169 k nodes, 4 slices: 2.39 ms a pass on one stream, 2.37 on two) and loses elsewhere; every slice computes exactly
        what it computes alone, so results are bitwise the same."""
        self.g, self.n, self.k, self.L = graph, n_nodes, k, layers
        self.w0, self.hs = first_width, slice_hidden
        self.dev = torch.device(device)
        self.act_last = act_last
        f32 = dict(dtype=torch.float32, device=self.dev)
        self.widths = [(first_width if l == 0 else slice_hidden, slice_hidden) for l in range(layers)]
        self.order = order
        if scaled is None:
            scaled = graph.view().nnz >= (1 << 24)
        self.scaled = scaled
        # layers that run in the transform-first order keep no aggregation of their input
        self.tf = [order == B.LAYER_TRANSFORM_FIRST or (order == B.LAYER_ORDER_AUTO and wo < wi) for wi, wo in self.widths]
        # layout flags per layer: a layer reads a scaled input when its producer could write one (the previous layer if
        # both run aggregate-first; the raw slice, scaled in place by prepare_inputs, for the first layer)
        shared = shared_input is not None
        self.in_scaled = [scaled and not self.tf[l] and (not shared if l == 0 else not self.tf[l - 1]) for l in range(layers)]
        self.layout = [(B.LAYER_IN_SCALED if self.in_scaled[l] else 0) |
                       (B.LAYER_OUT_SCALED if l + 1 < layers and self.in_scaled[l + 1] else 0) for l in range(layers)]
        self.inputs_prepared = False
        # inputs
        # with direct slicing the first layer aggregates constant features: A^ X_s can be kept across passes
        # (the paper's implementation recomputes it; off by default so that a pass measures every kernel)
        self.cache_first = cache_first_aggregation and shared_input is None and not self.tf[0]
        self.first_valid = [False] * k
        self.shared = shared_input is not None
        self.X = ([shared_input] * k if self.shared
                  else [torch.zeros((n_nodes, padded_ld(first_width)), **f32) for _ in range(k)])
        self.dXin = torch.empty((n_nodes, padded_ld(first_width)), **f32) if self.shared else None
        # parameters and their gradients: [slice][layer] -> dict
        self.params = [[None] * layers for _ in range(k)]
        self.grads = [[None] * layers for _ in range(k)]
        self.E = torch.zeros((k, slice_hidden), **f32) if slice_encoding else None
        self.dE = torch.zeros((k, slice_hidden), **f32) if slice_encoding else None
        # activations kept for the backward pass
        self.H = [[torch.empty((n_nodes, padded_ld(slice_hidden)), **f32) for _ in range(layers - 1)] for _ in range(k)]
        self.Z = [[None if self.tf[l] else torch.empty((n_nodes, padded_ld(wi)), **f32) for l, (wi, _) in enumerate(self.widths)]
                  for _ in range(k)]
        mw = (slice_hidden + 31) // 32
        self.mask = [[torch.zeros((n_nodes, mw), dtype=torch.int32, device=self.dev) for _ in range(layers)] for _ in range(k)]
        self.Hcat = torch.empty((n_nodes, k * slice_hidden), **f32)
        # Slice encoding adds the row vector E[i] to every node row of slice i; the last layer's self-term bias does
        # the same, so E[i] can ride on it: the last layer then stores the encoded output straight into its column
        # block (no encoding pass) and dE[i] is that layer's db_self (no column-sum pass over dH).
        self.fuse_encoding = fuse_encoding and slice_encoding
        # slice i runs on lane i mod lanes; a lane has its own stream, workspace and backward scratch
        self.lanes = max(1, min(k, int(streams)))
        self.streams = [torch.cuda.Stream(device=self.dev) for _ in range(self.lanes)] if self.lanes > 1 else []
        # On one lane the slices run in groups of `group`: a layer of all of them is one set of launches, which is what a
        # small graph needs (its kernels last microseconds and leave most of the chip idle) and where the last, partly filled
        # round of a launch's workgroups still shows.  A large graph gains nothing and would need every buffer of the backward
        # pass per slice, so a group ends where one launch touches GROUP_BYTES.
        row_bytes = 4 * 4 * max(padded_ld(first_width), padded_ld(slice_hidden))  # Z, input and output, twice the widest
        if self.shared:
            row_bytes += 4 * padded_ld(first_width)  # the slice's input gradient
        self.group = 1 if self.lanes > 1 else max(1, min(k, B.MAX_GROUP, GROUP_BYTES // (n_nodes * row_bytes)))
        slots = max(self.lanes, self.group)
        self.dbuf = [[torch.empty((n_nodes, padded_ld(slice_hidden)), **f32) for _ in range(2)] if layers > 1 else []
                     for _ in range(slots)]
        # with a shared (learned) input the first slice's gradient is formed where the sum is wanted; the other slices that run
        # together keep theirs until all of them are there, and they are added in slice order
        self.together = k if self.lanes > 1 else self.group
        self.dXs = [torch.empty((n_nodes, padded_ld(first_width)), **f32)
                    for _ in range(k - 1 if k <= self.together else self.together)] if self.shared else []
        ws = 0
        for l, (wi, wo) in enumerate(self.widths):
            ws = max(ws, B.slicegcn_layers_fwd_workspace_bytes(graph, wi, wo, self.group, order),
                     B.slicegcn_layers_bwd_workspace_bytes(graph, wi, wo, l > 0 or self.shared, self.group, order))
        ws = max(ws, B.slicegcn_concat_bwd_workspace_bytes(n_nodes, [slice_hidden] * k))
        self.ws_lane = [torch.empty(ws, dtype=torch.uint8, device=self.dev) for _ in range(self.lanes)]
        self.ws = self.ws_lane[0]
        self._plans = [None, None]  # forward, backward

    # ---------------------------------------------------------------------------------
    def set_params(self, i: int, l: int, W_agg, b, W_self, b_self):
        wi, wo = self.widths[l]
        f32 = dict(dtype=torch.float32, device=self.dev)
        self.params[i][l] = dict(W_agg=W_agg.to(**f32).contiguous(), b=b.to(**f32).contiguous(),
                                 W_self=None if W_self is None else W_self.to(**f32).contiguous(),
                                 b_self=None if b_self is None else b_self.to(**f32).contiguous())
        self.grads[i][l] = dict(dW_agg=torch.empty((wi, wo), **f32), db=torch.empty(wo, **f32),
                                dW_self=torch.empty((wi, wo), **f32) if W_self is not None else None,
                                db_self=torch.empty(wo, **f32) if W_self is not None else None)

    def parameter_slots(self):
        """(holder of the parameter, key, holder of its gradient, key) for every learnable tensor."""
        out = []
        for i in range(self.k):
            for l in range(self.L):
                for pn, gn in (("W_agg", "dW_agg"), ("b", "db"), ("W_self", "dW_self"), ("b_self", "db_self")):
                    if self.params[i][l][pn] is not None:
                        out.append((self.params[i][l], pn, self.grads[i][l], gn))
        if self.E is not None:
            out.append((self, "E", self, "dE"))
        return out

    def inputs_changed(self):
        """Call after writing new features into ``X``: cached first-layer aggregations are dropped."""
        self.first_valid = [False] * self.k
        self.inputs_prepared = False

    def prepare_inputs(self):
        """Once per set of raw features: with the scaled layout the slices in ``X`` become D~^-1/2 X_s, in place."""
        if self.in_scaled[0] and not self.shared and not self.inputs_prepared:
            for x in self.X:
                B.slicegcn_scale_rows(self.g, x[:, :self.w0], x, width=self.w0)
        self.inputs_prepared = True

    def hin(self, i: int, l: int) -> torch.Tensor:
        wi = self.widths[l][0]
        return (self.X[i] if l == 0 else self.H[i][l - 1])[:, :wi]

    def hout(self, i: int, l: int) -> torch.Tensor:
        if l == self.L - 1:
            return self.Hcat[:, i * self.hs:(i + 1) * self.hs]
        return self.H[i][l][:, :self.hs]

    def input_gradient(self, i: int) -> torch.Tensor:
        """Where slice i's gradient of a shared input goes."""
        return self.dXin if i == 0 else self.dXs[i % self.together - (i < self.together)]

    def act(self, l: int) -> int:
        return self.act_last if l == self.L - 1 else B.ACT_RELU

    # ---------------------------------------------------------------------------------
    def encoding_fused(self) -> bool:
        last = self.L - 1
        return self.fuse_encoding and all(self.params[i][last]["W_self"] is not None and
                                          self.params[i][last]["b_self"] is not None for i in range(self.k))

    # ---- call arguments of every layer, laid out once ---------------------------------
    def _tensors(self, back: bool):
        """The tensors one direction of a pass hands to the layers, in a fixed order."""
        out = [*self.X]
        if back:
            out.append(self.dE)
            if self.shared:
                out += (self.dXin, *self.dXs)
            for pair in self.dbuf:
                out += pair
        else:
            out += (self.Hcat, self.E)
        for i in range(self.k):
            out += self.H[i]
            out += self.Z[i]
            out += self.mask[i]
            for l, p in enumerate(self.params[i]):
                if p is None:  # not set yet
                    out.append(None)
                elif back:
                    gr = self.grads[i][l]
                    out += (p["W_agg"], p["W_self"], gr["dW_agg"], gr["db"], gr["dW_self"], gr["db_self"])
                else:
                    out += (p["W_agg"], p["b"], p["W_self"], p["b_self"])
        return out

    def _plan(self, back: bool, fused: bool) -> LayerPlan:
        """The argument blocks of one direction.  They are laid out again, with every check, when a tensor they are made from
        is no longer what it was (parameters are rebound when an optimiser takes them over) or the encoding changed its place;
        the activation and the flags of a layer are put in by each call."""
        tensors, plan = self._tensors(back), self._plans[back]
        if plan is not None and fused == plan.fused and plan.layouts.same(tensors):
            return plan
        self._plans[back] = None
        ios, shapes, alike = [], [], True
        for l, (wi, wo) in enumerate(self.widths):
            last = l == self.L - 1
            io, of_layer, kinds = (B.LayerIo * self.k)(), [], set()
            for i in range(self.k):
                p, x = self.params[i][l], io[i]
                if p is None:  # the call refuses it
                    of_layer.append(B.LayerGroup(B._LayerDesc(wi, wo, 0, 0), 1, 0, 0, 0, 0, 0, 0))
                    kinds.add(None)
                    continue
                for name, W in (("W_agg", p["W_agg"]), ("W_self", p["W_self"])):
                    if W is not None and tuple(W.shape) != (wi, wo):
                        raise ValueError(f"{name} must be w_in x w_out")
                x.Hin, ldi = B._mat(self.hin(i, 0) if l == 0 else self.H[i][l - 1], "Hin")
                x.Z, ldz = B._mat(self.Z[i][l], "Z") if self.Z[i][l] is not None else (None, 0)
                x.mask, mask_words = B._mat(self.mask[i][l], "mask", torch.int32)
                ldo = ldgo = ldgi = 0
                if not back:
                    x.params = B._LayerParams(*(B._vec(p[n], n) for n in ("W_agg", "b", "W_self", "b_self")))
                    x.Hout, ldo = B._mat(self.hout(i, l) if last else self.H[i][l], "Hout")
                    if fused and last:
                        x.enc = B._vec(self.E[i], "E")
                else:
                    gr, slot = self.grads[i][l], i % len(self.dbuf)
                    x.params = B._LayerParams(B._vec(p["W_agg"], "W_agg"), None, B._vec(p["W_self"], "W_self"), None)
                    x.grads = B._LayerGrads(*(B._vec(gr[n], n) for n in ("dW_agg", "db", "dW_self", "db_self")))
                    if l > 0:
                        x.dHin, ldgi = B._mat(self.dbuf[slot][l % 2], "dHin")
                    elif self.shared:  # raw features need no gradient
                        x.dHin, ldgi = B._mat(self.input_gradient(i), "dHin")
                    if not last:  # the last layer's comes with the call
                        x.dHout, ldgo = B._mat(self.dbuf[slot][(l + 1) % 2], "dHout")
                    if fused and last:
                        x.denc = B._vec(self.dE[i], "dE")
                kind = (p["W_self"] is None, ldi, ldo, ldz, mask_words, ldgo, ldgi)
                of_layer.append(of_layer[-1] if i > 0 and kind == before else B.LayerGroup(B._LayerDesc(wi, wo, 0, 0), 1, *kind[1:]))
                before = kind
                kinds.add(kind)
            ios.append(io)
            shapes.append(of_layer)
            alike = alike and len(kinds) == 1  # slices of other leading dimensions or terms share no launch
        plan = self._plans[back] = LayerPlan(ios, shapes, alike, fused, TensorLayouts(tensors))
        return plan

    def _shape(self, plan: LayerPlan, l: int, first: int, count: int, flags: int = 0) -> B.LayerGroup:
        sh = plan.shapes[l][first]
        sh.count, desc = count, sh.desc
        desc.act, desc.flags = self.act(l), self.order | self.layout[l] | flags
        return sh

    def _forward_group(self, plan: LayerPlan, first: int, count: int, ws):
        cached = self.cache_first and all(self.first_valid[first:first + count])
        for l in range(self.L):
            sh = self._shape(plan, l, first, count, B.LAYER_Z_VALID if cached and l == 0 else 0)
            B.slicegcn_layers_fwd(self.g, sh, plan.ios[l], first, ws)
        self.first_valid[first:first + count] = [True] * count

    def forward_slice(self, i: int):
        if not self.inputs_prepared:
            self.prepare_inputs()
        self._forward_group(self._plan(False, self.encoding_fused()), i, 1, self.ws_lane[i % self.lanes])

    def _on_lanes(self, fn, plan: LayerPlan):
        """fn(plan, first slice, count, workspace) for every group of slices: in turn on the caller's stream, or slice i on lane
        i mod lanes, the lanes starting after what the caller's stream holds so far and the caller's stream going on after
        all of them."""
        if self.lanes == 1:
            group = self.group if plan.alike else 1
            for i in range(0, self.k, group):
                fn(plan, i, min(group, self.k - i), self.ws)
            return
        main = torch.cuda.current_stream()
        for s in self.streams:
            s.wait_stream(main)
        for i in range(self.k):
            with torch.cuda.stream(self.streams[i % self.lanes]):
                fn(plan, i, 1, self.ws_lane[i % self.lanes])
        for s in self.streams:
            main.wait_stream(s)

    def forward(self) -> torch.Tensor:
        if not self.inputs_prepared:
            self.prepare_inputs()
        fused = self.encoding_fused()
        self._on_lanes(self._forward_group, self._plan(False, fused))
        # the last layer of every slice already stored into its column block: encode in place, unless that is done
        if not fused:
            B.slicegcn_concat([self.hout(i, self.L - 1) for i in range(self.k)], self.E, self.Hcat)
        return self.Hcat

    def backward(self, dH: torch.Tensor):
        fused = self.encoding_fused()
        plan = self._plan(True, fused)
        if self.E is not None and not fused:
            B.slicegcn_concat_bwd(dH, [self.hs] * self.k, dE=self.dE, ws=self.ws)
        ptr, ld = B._mat(dH, "dH")
        for i in range(self.k):  # CONCAT backward is a column view
            plan.ios[-1][i].dHout = ptr + 4 * i * self.hs
            plan.shapes[-1][i].ldgo = ld

        def backward_group(plan: LayerPlan, first: int, count: int, ws):
            for l in reversed(range(self.L)):
                B.slicegcn_layers_bwd(self.g, self._shape(plan, l, first, count), plan.ios[l], first, ws)
            if self.lanes == 1:
                self._add_input_gradients(first, count)

        self._on_lanes(backward_group, plan)
        if self.lanes > 1:
            for i in range(0, self.k, B.MAX_GROUP):
                self._add_input_gradients(i, min(B.MAX_GROUP, self.k - i))

    def _add_input_gradients(self, first: int, count: int):
        others = [self.input_gradient(i)[:, :self.w0] for i in range(max(first, 1), first + count)] if self.shared else []
        if others:
            B.slicegcn_accumulate_many(self.dXin[:, :self.w0], others)


class Classifier:
    """The paper's MLP_CLS on the concatenated representation followed by the mean softmax
    cross-entropy of its loss equation: logits = relu(H W1 + b1) W2 + b2.  Owns buffers and orders
    the library calls; every arithmetic step is a kernel of ``libslicegcn.so``."""

    def __init__(self, n_nodes: int, width: int, hidden: int, classes: int, device="cuda"):
        self.n, self.w, self.h, self.c = n_nodes, width, hidden, classes
        self.dev = torch.device(device)
        f32 = dict(dtype=torch.float32, device=self.dev)
        self.W1 = torch.zeros((width, hidden), **f32); self.b1 = torch.zeros(hidden, **f32)
        self.W2 = torch.zeros((hidden, classes), **f32); self.b2 = torch.zeros(classes, **f32)
        self.dW1 = torch.empty_like(self.W1); self.db1 = torch.empty_like(self.b1)
        self.dW2 = torch.empty_like(self.W2); self.db2 = torch.empty_like(self.b2)
        self.A = torch.empty((n_nodes, hidden), **f32)
        self.dA = torch.empty((n_nodes, hidden), **f32)
        self.mask = torch.zeros((n_nodes, (hidden + 31) // 32), dtype=torch.int32, device=self.dev)
        self.logits = torch.empty((n_nodes, classes), **f32)  # overwritten by its own gradient in backward
        self.loss = torch.zeros(1, **f32)
        ws = max(B.slicegcn_softmax_ce_workspace_bytes(n_nodes), B.slicegcn_linear_bwd_full_workspace_bytes(n_nodes, width, hidden),
                 B.slicegcn_linear_bwd_full_workspace_bytes(n_nodes, hidden, classes))
        self.ws = torch.empty(ws, dtype=torch.uint8, device=self.dev)

    def set_params(self, W1, b1, W2, b2):
        for dst, src in ((self.W1, W1), (self.b1, b1), (self.W2, W2), (self.b2, b2)):
            dst.copy_(src)

    def forward(self, H: torch.Tensor, labels: torch.Tensor) -> torch.Tensor:
        """Loss of the batch (device scalar).  Leaves the gradient of the loss with respect to the
        logits in ``self.logits`` for ``backward``."""
        B.slicegcn_linear_fwd(H, self.W1, self.b1, self.A, self.mask, act=B.ACT_RELU)
        B.slicegcn_linear_fwd(self.A, self.W2, self.b2, self.logits, None, act=B.ACT_NONE)
        B.slicegcn_softmax_ce(self.logits, labels, self.loss, self.logits, self.ws)  # gradient in place
        return self.loss

    def backward(self, H: torch.Tensor, dH: torch.Tensor):
        """dH receives the gradient of the loss with respect to H; the parameter gradients go to
        dW1, db1, dW2, db2."""
        B.slicegcn_linear_bwd(self.A, self.W2, None, self.logits, self.dA, self.dW2, self.db2, self.ws, act=B.ACT_NONE)
        B.slicegcn_linear_bwd(H, self.W1, self.mask, self.dA, dH, self.dW1, self.db1, self.ws, act=B.ACT_RELU)

    def forward_backward(self, H: torch.Tensor, labels: torch.Tensor, dH: torch.Tensor) -> torch.Tensor:
        self.forward(H, labels)
        self.backward(H, dH)
        return self.loss


class FeatureFusion:
    """The paper's MLP_FF (feature-fusion equation; two dense layers d' -> d' -> slice_size with a ReLU
    between them, shared by all slices): Xff = relu(X W1 + b1) W2 + b2.  Owns buffers and orders the
    library calls; every arithmetic step is a kernel of ``libslicegcn.so``."""

    def __init__(self, n_nodes: int, feat: int, out_width: int, device="cuda"):
        self.n, self.f, self.s = n_nodes, feat, out_width
        self.dev = torch.device(device)
        f32 = dict(dtype=torch.float32, device=self.dev)
        self.W1 = torch.zeros((feat, feat), **f32); self.b1 = torch.zeros(feat, **f32)
        self.W2 = torch.zeros((feat, out_width), **f32); self.b2 = torch.zeros(out_width, **f32)
        self.dW1 = torch.empty_like(self.W1); self.db1 = torch.empty_like(self.b1)
        self.dW2 = torch.empty_like(self.W2); self.db2 = torch.empty_like(self.b2)
        self.A = torch.empty((n_nodes, feat), **f32)
        self.dA = torch.empty((n_nodes, feat), **f32)
        self.mask = torch.zeros((n_nodes, (feat + 31) // 32), dtype=torch.int32, device=self.dev)
        self.Xff = torch.zeros((n_nodes, padded_ld(out_width)), **f32)  # padding columns stay zero
        ws = max(B.slicegcn_linear_bwd_full_workspace_bytes(n_nodes, feat, feat),
                 B.slicegcn_linear_bwd_full_workspace_bytes(n_nodes, feat, out_width))
        self.ws = torch.empty(ws, dtype=torch.uint8, device=self.dev)

    def set_params(self, W1, b1, W2, b2):
        for dst, src in ((self.W1, W1), (self.b1, b1), (self.W2, W2), (self.b2, b2)):
            dst.copy_(src)

    def forward(self, X: torch.Tensor) -> torch.Tensor:
        B.slicegcn_linear_fwd(X, self.W1, self.b1, self.A, self.mask, act=B.ACT_RELU)
        B.slicegcn_linear_fwd(self.A, self.W2, self.b2, self.Xff[:, :self.s], None, act=B.ACT_NONE)
        return self.Xff

    def backward(self, X: torch.Tensor, dXff: torch.Tensor):
        """dXff: n x out_width gradient of the fused features (the sum over the slice models)."""
        B.slicegcn_linear_bwd(self.A, self.W2, None, dXff, self.dA, self.dW2, self.db2, self.ws, act=B.ACT_NONE)
        B.slicegcn_linear_bwd(X, self.W1, self.mask, self.dA, None, self.dW1, self.db1, self.ws, act=B.ACT_RELU)


def _dense_slots(obj):
    return [(obj, "W1", obj, "dW1"), (obj, "b1", obj, "db1"), (obj, "W2", obj, "dW2"), (obj, "b2", obj, "db2")]


Classifier.parameter_slots = _dense_slots
FeatureFusion.parameter_slots = _dense_slots


class Optimizer:
    """Adam with a cosine-annealed learning rate (the paper's experimental settings) over all learnable
    tensors of the given models.  The tensors are moved into one flat buffer (gradients into another) and
    the models' attributes rebound to views of it, so one library call updates every parameter."""

    ALIGN = 64  # floats: every tensor starts on a 256-byte boundary, so vector paths stay usable

    def __init__(self, models, lr_max: float, lr_min: float = 0.0, t_max: int = 1, beta1: float = 0.9,
                 beta2: float = 0.999, eps: float = 1e-8, weight_decay: float = 0.0):
        slots = [s for m in models for s in m.parameter_slots()]
        get = lambda o, k: o[k] if isinstance(o, dict) else getattr(o, k)
        offs, total = [], 0
        for po, pk, _, _ in slots:
            offs.append(total)
            total += (get(po, pk).numel() + self.ALIGN - 1) // self.ALIGN * self.ALIGN
        dev = get(slots[0][0], slots[0][1]).device
        self.P, self.G, self.M, self.V = (torch.zeros(total, dtype=torch.float32, device=dev) for _ in range(4))
        for (po, pk, go, gk), o in zip(slots, offs):
            old = get(po, pk)
            pv = self.P[o:o + old.numel()].view(old.shape)
            pv.copy_(old)
            gv = self.G[o:o + old.numel()].view(old.shape)
            for holder, key, view in ((po, pk, pv), (go, gk, gv)):
                if isinstance(holder, dict):
                    holder[key] = view
                else:
                    setattr(holder, key, view)
        self.hyper = (beta1, beta2, eps, weight_decay)
        self.lr_max, self.lr_min, self.t_max = lr_max, lr_min, t_max
        self.t = 0

    def step(self, epoch: int) -> float:
        """One update with the learning rate of ``epoch`` (0-based); returns that rate."""
        self.t += 1
        lr = B.slicegcn_cosine_lr(self.lr_max, self.lr_min, epoch, self.t_max)
        b1, b2, eps, wd = self.hyper
        B.slicegcn_adam_step(self.P, self.G, self.M, self.V, lr, self.t, b1, b2, eps, wd)
        return lr


class GraphedStep:
    """A sequence of library calls captured once into a HIP graph and replayed with one launch.

    For the small workloads a pass is a few hundred kernels of microseconds each and the time goes
    into launching them; a replayed graph removes that.  ``fn`` must only issue library calls on the
    current stream and touch preallocated buffers (every entry point except graph construction
    qualifies: none allocates, synchronises or clears memory with a memset node).  The buffers are
    read through their addresses, so new inputs written into the same tensors are picked up by the
    next replay."""

    def __init__(self, fn, warmup: int = 1):
        self.stream = torch.cuda.Stream()
        self.stream.wait_stream(torch.cuda.current_stream())
        with torch.cuda.stream(self.stream):
            for _ in range(warmup):
                fn()
        torch.cuda.current_stream().wait_stream(self.stream)
        torch.cuda.synchronize()
        self.graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(self.graph, stream=self.stream):
            fn()

    def replay(self):
        self.graph.replay()
