"""The work that a training program has this library do, as cases that can be timed and checked.

Four kinds of call, all through the Python binding:

  epoch  one training epoch of a whole model (Model.epoch), as the bench runs it;
  layer  one layer forward (layer_fwd), backward (layer_bwd) or both, as a program with its own
         loop calls them: dense or sparse input features, every aggregator, hidden layers (ReLU)
         and the loss layer (softmax cross-entropy, with its logits);
  graph  the edge list to A + I in CSR form (build_csr), paid once per graph;
  probe  the density probe of the input features and their CSR and CSC views (feature_stats),
         paid once per feature matrix.

Graphs are Chung-Lu power laws (degree exponent 2.5) and Graph500-style RMAT samples with randomly
permuted node ids, the two families of gcn_synth, drawn here on the device.
"""
import math

import torch

import paper_2512_01678_amd.gcn as G

AGGS = {"gcn": G.AGG_NORM, "sum": G.AGG_SUM, "mean": G.AGG_MEAN, "max": G.AGG_MAX}
ACTS = {"relu": G.ACT_RELU, "softmax": G.ACT_SOFTMAX_CE}


def listed():
    return [
        # a citation graph of a few thousand nodes with bag-of-words features: the smallest model,
        # where launches and their latency count
        dict(name="epoch_cora", kind="epoch", graph="chung_lu", n=2708, e=5278, f=1433, hidden=16, layers=2,
             classes=7, density=0.013, agg="gcn"),
        # the bench's default: the largest graph that is trained whole, 2.45 M nodes, 126 M entries
        dict(name="epoch_products", kind="epoch", graph="chung_lu", n=2449029, e=61859140, f=100, hidden=256,
             layers=3, classes=47, density=1.0, agg="gcn"),
        # hidden layer of a mid-sized citation graph (about 15 entries per row), each direction
        dict(name="hidden_fwd_arxiv", kind="layer", graph="chung_lu", n=169343, e=1166243, f_in=256, f_out=256,
             act="relu", index=1, agg="gcn", density=1.0, run="fwd"),
        dict(name="hidden_bwd_arxiv", kind="layer", graph="chung_lu", n=169343, e=1166243, f_in=256, f_out=256,
             act="relu", index=1, agg="gcn", density=1.0, run="bwd"),
        # the loss layer of the same model: a narrow aggregation with the softmax epilogue
        dict(name="loss_arxiv", kind="layer", graph="chung_lu", n=169343, e=1166243, f_in=256, f_out=40,
             act="softmax", index=2, agg="gcn", density=1.0, run="both"),
        # a widening first layer aggregates its input before the transform (mean aggregator)
        dict(name="widening_arxiv_mean", kind="layer", graph="chung_lu", n=169343, e=1166243, f_in=128, f_out=256,
             act="relu", index=0, agg="mean", density=1.0, run="both"),
        # the max aggregator of the same graph
        dict(name="hidden_arxiv_max", kind="layer", graph="chung_lu", n=169343, e=1166243, f_in=128, f_out=128,
             act="relu", index=1, agg="max", density=1.0, run="both"),
        # a dense social graph (about 490 entries per row), first layer with wide dense features
        dict(name="first_fwd_reddit", kind="layer", graph="chung_lu", n=232965, e=57307946, f_in=602, f_out=256,
             act="relu", index=0, agg="gcn", density=1.0, run="fwd"),
        # its loss layer backward: 41 classes, input gradient for the hidden layer
        dict(name="loss_bwd_reddit", kind="layer", graph="chung_lu", n=232965, e=57307946, f_in=256, f_out=41,
             act="softmax", index=1, agg="gcn", density=1.0, run="bwd"),
        # sparse input features (1 % of 4096 columns) on an RMAT graph of 2^21 nodes
        dict(name="sparse_rmat", kind="layer", graph="rmat", n=1 << 21, e=1 << 25, f_in=4096, f_out=128, act="relu",
             index=0, agg="gcn", density=0.01, run="both"),
        # set-up: the largest graph from its edge list, and features from their dense form
        dict(name="graph_products", kind="graph", graph="chung_lu", n=2449029, e=61859140),
        dict(name="probe_sparse", kind="probe", n=1 << 20, f=1024, density=0.01),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _draw_graph(rng, most_entries):
    """A graph of at most most_entries entries of A + I."""
    if rng.random() < 0.25:
        scale = rng.randint(12, 21)
        while (1 << scale) * 33 > most_entries and scale > 12:
            scale -= 1
        return dict(graph="rmat", n=1 << scale, e=16 << scale)
    n = _log(rng, 2000, 2449029)
    deg = math.exp(rng.uniform(math.log(4.0), math.log(490.0)))
    deg = min(deg, n / 8.0, max(2.0, most_entries / n - 1.0))
    n = min(n, int(most_entries / 3))
    return dict(graph="chung_lu", n=n, e=max(1, int(n * deg / 2)))


def draw(rng):
    kind = rng.choices(["epoch", "layer", "sparse", "graph", "probe"], [2, 8, 2, 1, 1])[0]
    if kind == "epoch":
        sparse = rng.random() < 0.3
        hidden = rng.choice([_log(rng, 8, 256), 64, 128, 256])
        classes, layers = _log(rng, 2, 60), rng.randint(2, 3)
        f = _log(rng, 300, 2000) if sparse else _log(rng, 16, 602)
        # no more gathered values than the largest listed epoch
        c = _draw_graph(rng, min(120_000_000, int(1.0e11 / (2 * layers * max(hidden, 32)))))
        if sparse:
            c["n"] = min(c["n"], 1 << 20) if c["graph"] == "chung_lu" else c["n"]
            c["e"] = min(c["e"], c["n"] * 200)
        return dict(kind="epoch", **c, f=f, hidden=hidden, layers=layers, classes=classes,
                    density=math.exp(rng.uniform(math.log(0.002), math.log(0.05))) if sparse else 1.0,
                    agg=rng.choice(["gcn", "gcn", "gcn", "sum", "mean"]))
    if kind == "layer":
        act = rng.choice(["relu", "relu", "softmax"])
        agg = rng.choice(["gcn", "gcn", "gcn", "mean", "sum", "max"])
        index = rng.randint(0, 1) if act == "relu" else 1
        f_in = _log(rng, 16, 602 if index == 0 and agg != "max" else 256)
        f_out = _log(rng, 2, 60) if act == "softmax" else rng.choice([_log(rng, 8, 256), 64, 128, 256])
        c = _draw_graph(rng, min(126_000_000, int(2.5e10 / max(f_out, 32 if agg != "max" else 4 * f_in))))
        return dict(kind="layer", **c, f_in=f_in, f_out=f_out, act=act, index=index, agg=agg, density=1.0,
                    run=rng.choice(["fwd", "bwd", "both"]))
    if kind == "sparse":
        c = _draw_graph(rng, 60_000_000)
        f = _log(rng, 300, 4096)
        density = math.exp(rng.uniform(math.log(0.001), math.log(0.05)))
        c["n"] = c["n"] if c["graph"] == "rmat" else min(c["n"], int(4.0e8 / (f * density)), int(8e9 / f))
        c["e"] = min(c["e"], c["n"] * 200)
        return dict(kind="layer", **c, f_in=f, f_out=rng.choice([_log(rng, 8, 256), 16, 64, 128]), act="relu",
                    index=0, agg=rng.choice(["gcn", "gcn", "sum", "mean"]), density=min(density, 4.0e8 / (f * c["n"])),
                    run=rng.choice(["fwd", "bwd", "both"]))
    if kind == "graph":
        c = _draw_graph(rng, 126_000_000)
        return dict(c, kind="graph", e=c["e"] // (2 if c["graph"] == "rmat" else 1))
    n = _log(rng, 2708, 1 << 20)
    return dict(kind="probe", n=n, f=min(_log(rng, 64, 4096), (1 << 30) // n),
                density=math.exp(rng.uniform(math.log(0.001), math.log(0.06))))


# ---------------------------------------------------------------------------
# inputs, from the seed alone
# ---------------------------------------------------------------------------


def _gen(seed, stream):
    return torch.Generator(device="cuda").manual_seed((seed * 1000003 + stream * 7919 + 12345) & 0x7FFFFFFFFFFF)


def _pairs(c, e, g):
    """e sampled endpoint pairs (int32), node ids not yet permuted."""
    n = c["n"]
    if c["graph"] == "rmat":
        src = torch.zeros(e, dtype=torch.int32, device="cuda")
        dst = torch.zeros(e, dtype=torch.int32, device="cuda")
        for lvl in range(n.bit_length() - 1):
            r = torch.rand(e, device="cuda", generator=g)
            src.add_((r >= 0.76).int(), alpha=1 << lvl)
            dst.add_((((r >= 0.57) & (r < 0.76)) | (r >= 0.95)).int(), alpha=1 << lvl)
        return src, dst
    # Chung-Lu: weight (i + i0)^(-2/3), i0 such that the largest expected degree is
    # min(n / 8, 100 means); endpoints by the inverse of the continuous distribution
    mean = 2.0 * c["e"] / n
    dmax = max(min(n / 8.0, 100.0 * mean), 1.5 * mean)
    lo, hi = 1e-6, 1e12
    for _ in range(200):
        i0 = math.sqrt(lo * hi)
        top = n * mean * i0 ** (-2.0 / 3.0) / (3.0 * ((n + i0) ** (1.0 / 3.0) - i0 ** (1.0 / 3.0)))
        lo, hi = (i0, hi) if top > dmax else (lo, i0)
    a, b = i0 ** (1.0 / 3.0), (n + i0) ** (1.0 / 3.0)

    def ends():
        u = torch.rand(e, device="cuda", generator=g, dtype=torch.float64)
        u = u.mul_(b - a).add_(a).pow_(3).sub_(i0)
        return u.to(torch.int32).clamp_(0, n - 1)

    return ends(), ends()


def _edges(c, seed):
    """Sampled endpoint pairs (int32).  Repeated pairs and self pairs stay in: build_csr drops them."""
    g = _gen(seed, 1)
    perm = torch.randperm(c["n"], device="cuda", generator=g, dtype=torch.int32)
    src, dst = _pairs(c, c["e"], g)
    return perm[src], perm[dst]


def _edges_counted(c, seed):
    """e pairs of which one in sixteen repeats another the other way round or joins a node to itself: as
    many entries of A + I for every seed."""
    n, e, g = c["n"], c["e"], _gen(seed, 1)
    perm = torch.randperm(n, device="cuda", generator=g, dtype=torch.int32)
    need = e - e // 16
    keys = torch.zeros(0, dtype=torch.long, device="cuda")
    while keys.numel() < need:
        s, d = _pairs(c, int(need * 1.1) + 256, g)
        k = (torch.minimum(s, d).long() * n + torch.maximum(s, d))[s != d]
        keys = torch.unique(torch.cat([keys, k]))
    keys = keys[torch.randperm(keys.numel(), device="cuda", generator=g)[:need]]
    s, d = perm[keys // n], perm[keys % n]
    twice, self_ = (e // 16) - (e // 64), e // 64
    mix = torch.randperm(e, device="cuda", generator=g)
    src, dst = torch.cat([s, d[:twice], s[:self_]]), torch.cat([d, s[:twice], s[:self_]])
    return src[mix], dst[mix]


def _normal(rows, w, seed, stream, pitch=None):
    buf = torch.zeros((rows, pitch or G.pitch(w)), dtype=torch.float32, device="cuda")
    buf[:, :w] = torch.randn((rows, w), device="cuda", generator=_gen(seed, stream))
    return buf[:, :w]


def _features(c, n, f, seed):
    """Input features: N(0, 1), or (0, 1] with probability `density` and zero elsewhere."""
    ld = (f + 3) // 4 * 4
    if c["density"] >= 1.0:
        return _normal(n, f, seed, 3, ld)
    X = torch.zeros((n, ld), dtype=torch.float32, device="cuda")[:, :f]
    for r in range(0, n, 1 << 18):  # by rows: the comparison's result is not held for all of X
        b = X[r:r + (1 << 18)]
        b.uniform_(0.0, 1.0 / c["density"], generator=_gen(seed, 3000 + (r >> 18)))
        b.masked_fill_(b > 1.0, 0.0)
    return X


def _features_counted(c, seed):
    """Sparse features with as many nonzeros for every seed."""
    n, f = c["n"], c["f"]
    count = int(n * f * c["density"])
    X = _features(dict(density=c["density"] * (1.0 + 8.0 / math.sqrt(count)) + 1e-6), n, f, seed)
    at = X.nonzero()
    at = at[torch.randperm(at.shape[0], device="cuda", generator=_gen(seed, 8))[:at.shape[0] - count]]
    X[at[:, 0], at[:, 1]] = 0.0
    return X


def _glorot(fi, fo, seed, stream):
    a = math.sqrt(6.0 / (fi + fo))
    return (torch.rand((fi, fo), device="cuda", generator=_gen(seed, stream)) * 2 - 1) * a


def _labels(n, classes, seed):
    return torch.randint(0, classes, (n,), device="cuda", generator=_gen(seed, 4), dtype=torch.int32)


def _widths(c):
    return (c["f"],) + (c["hidden"],) * (c["layers"] - 1) + (c["classes"],)


def _graph(c, seed, width):
    src, dst = _edges(c, seed)
    g = G.build_csr(c["n"], src, dst)
    G.tune_row_order(g, width)
    return g


def _layer_inputs(c, seed):
    """(H_in or None when sparse, W, b, labels, G): what a layer call of this case is given."""
    n, fi, fo = c["n"], c["f_in"], c["f_out"]
    Hin = None
    if c["index"] > 0:
        Hin = _normal(n, fi, seed, 5).clamp_(min=0.0)  # a hidden layer's ReLU output
    elif c["density"] >= 1.0:
        Hin = _features(c, n, fi, seed)
    W = _glorot(fi, fo, seed, 10)
    b = torch.randn(fo, device="cuda", generator=_gen(seed, 11)) * 0.05
    y = _labels(n, fo, seed)
    grad = None
    if c["run"] == "bwd":
        grad = _normal(n, fo, seed, 6)
        if c["act"] == "softmax":  # (softmax - onehot) / n
            p = torch.softmax(grad, 1)
            p[torch.arange(n, device="cuda"), y.long()] -= 1.0
            grad.copy_(p / n)
        else:  # half of it cut by the ReLU
            grad.mul_((torch.rand(n, fo, device="cuda", generator=_gen(seed, 7)) < 0.5) * (1.0 / n))
    return Hin, W, b, y, grad


def _sparse(X):
    return G.feature_stats(X, force_mode=G.SPARSE)[1]


# Adam state of a run under way: moments of the size that the gradients have after some epochs
_MOMENT, _STEP = 1e-3, 20


def _epoch_params(c, seed):
    w = _widths(c)
    Ws = [_glorot(w[l], w[l + 1], seed, 10 + l) for l in range(len(w) - 1)]
    bs = [torch.randn(w[l + 1], device="cuda", generator=_gen(seed, 30 + l)) * 0.05 for l in range(len(w) - 1)]
    mom = []
    for k, p in enumerate(Ws + bs):
        g = _gen(seed, 50 + k)
        mom.append((torch.randn(p.shape, device="cuda", generator=g) * (0.3 * _MOMENT),
                    (torch.rand(p.shape, device="cuda", generator=g) + 0.5) * _MOMENT ** 2))
    return Ws, bs, mom


def prepare(case, seed):
    c = case
    if c["kind"] == "graph":
        src, dst = _edges_counted(c, seed)
        return dict(c=c, src=src, dst=dst)
    if c["kind"] == "probe":
        return dict(c=c, X=_features_counted(c, seed))
    if c["kind"] == "epoch":
        w = _widths(c)
        g = _graph(c, seed, w[1])
        X = _features(c, c["n"], c["f"], seed)
        x = _sparse(X) if c["density"] < 1.0 else None
        Ws, bs, mom = _epoch_params(c, seed)
        m = G.Model(c["n"], w, [t.cpu() for t in Ws], [t.cpu() for t in bs], x_sparse=x is not None,
                    ld_x=X.stride(0), aggs=[AGGS[c["agg"]]] * c["layers"])
        for l in range(m.L):
            m.mW[l].copy_(mom[l][0])
            m.vW[l].copy_(mom[l][1])
            m.mb[l].copy_(mom[m.L + l][0])
            m.vb[l].copy_(mom[m.L + l][1])
        m.c.step = _STEP
        return dict(c=c, m=m, g=g, X=None if x is not None else X, x=x, y=_labels(c["n"], c["classes"], seed))
    n, fi, fo = c["n"], c["f_in"], c["f_out"]
    agg = AGGS[c["agg"]]
    g = _graph(c, seed, fo)
    Hin, W, b, y, grad = _layer_inputs(c, seed)
    x = _sparse(_features(c, n, fi, seed)) if Hin is None else None
    ld_in = Hin.stride(0) if Hin is not None else (fi + 3) // 4 * 4
    L = G.make_layer(fi, fo, ld_in, G.pitch(fo), ACTS[c["act"]], c["index"], agg=agg)
    s = dict(c=c, g=g, L=L, Hin=Hin, x=x, W=W, b=b, y=y, saved=None, arg=None, ws=None, wsb=None,
             Hout=G.padded(n, fo), loss=torch.zeros(1, device="cuda"), logits=None, grad=grad,
             dW=torch.empty_like(W), db=torch.empty_like(b), Gprev=None)
    if G.layer_order(fi, fo, c["index"], ACTS[c["act"]], x_sparse=x is not None, agg=agg) == G.AGGREGATE_FIRST:
        s["saved"], s["arg"] = G.saved_buffer(n, fi, ld_in, agg)
    if c["act"] == "softmax":
        s["logits"] = G.padded(n, fo)
    if c["index"] > 0 and c["run"] != "fwd":
        s["Gprev"] = G.padded(n, fi)
    if c["run"] == "bwd" and s["saved"] is not None:
        _fwd(s)  # the backward of an aggregate-first layer reads what its forward saved
    return s


def _fwd(s):
    s["ws"] = G.layer_fwd(s["g"], s["L"], s["Hin"], s["x"], s["W"], s["b"], s["Hout"], saved=s["saved"],
                          labels=s["y"] if s["logits"] is not None else None,
                          loss=s["loss"] if s["logits"] is not None else None, logits=s["logits"], ws=s["ws"])


def run(state):
    s, kind = state, state["c"]["kind"]
    if kind == "graph":
        g = G.build_csr(s["c"]["n"], s["src"], s["dst"])
        return dict(row_ptr=g.row_ptr, col=g.col_idx[:g.nnz], deg=g.deg, dinv=g.dinv, val=g.val[:g.nnz],
                    order=g.order)
    if kind == "probe":
        info, x = G.feature_stats(s["X"], force_mode=G.SPARSE)
        return dict(nnz=info["nnz"], row_ptr=x.row_ptr, col=x.col, val=x.val, col_ptr=x.col_ptr, row=x.row,
                    cval=x.cval)
    if kind == "epoch":
        m = s["m"]
        loss = m.epoch(s["g"], X=s["X"], x=s["x"], labels=s["y"])
        return dict(loss=loss, H=m.act, dW=m.dW, db=m.db, W=m.W, b=m.b, mW=m.mW, vW=m.vW)
    out = {}
    which = s["c"]["run"]
    if which != "bwd":
        _fwd(s)
        out = dict(H=s["Hout"], saved=s["saved"], arg=s["arg"])
        if s["logits"] is not None:
            out.update(loss=s["loss"], logits=s["logits"])
    if which != "fwd":
        # after a softmax layer's forward, Hout holds its loss gradient
        grad = s["grad"] if which == "bwd" else s["Hout"]
        s["wsb"] = G.layer_bwd(s["g"], s["L"], grad, s["Hin"], s["x"], s["saved"], s["W"], s["dW"], s["db"],
                               Gprev=s["Gprev"], ws=s["wsb"])
        out.update(dW=s["dW"], db=s["db"], Gprev=s["Gprev"])
    return out


# ---------------------------------------------------------------------------
# what a pass cannot do without
# ---------------------------------------------------------------------------


def work(case):
    c = case
    n = c["n"]
    if c["kind"] == "probe":  # X read once, both views written
        nnz = c["density"] * n * c["f"]
        return dict(bytes=4.0 * n * c["f"] + 16.0 * nnz + 8.0 * (n + c["f"]), flops=0.0)
    E = 2.0 * c["e"] + n  # about: repeated pairs collapse
    if c["kind"] == "graph":  # the pairs read; columns, values, offsets, degrees written
        return dict(bytes=8.0 * c["e"] + 8.0 * E + 20.0 * n, flops=0.0)
    graph = 4.0 * E + 12.0 * n  # columns, offsets, one factor per row

    def layer(fi, fo, index, density, fwd, bwd, sparse):
        xb = 4.0 * n * fi if not sparse else 8.0 * density * n * fi
        xf = 2.0 * n * fi * fo * (density if sparse else 1.0)
        by = fl = 0.0
        if fwd:
            by += graph + xb + 4.0 * fi * fo + 4.0 * n * fo
            fl += xf + 2.0 * E * min(fi, fo)
        if bwd:
            by += graph + xb + 4.0 * n * fo + 8.0 * fi * fo
            fl += xf + 2.0 * E * min(fi, fo)
            if index > 0:
                by += 4.0 * n * fi
                fl += 2.0 * n * fi * fo
        return by, fl

    if c["kind"] == "epoch":  # every layer's input and output once in each direction
        w, by, fl = _widths(c), 0.0, 0.0
        for l in range(len(w) - 1):
            b, f = layer(w[l], w[l + 1], l, c["density"], True, True, l == 0 and c["density"] < 1.0)
            by, fl = by + b + 24.0 * w[l] * w[l + 1], fl + f
        return dict(bytes=by, flops=fl)
    by, fl = layer(c["f_in"], c["f_out"], c["index"], c["density"], c["run"] != "bwd", c["run"] != "fwd",
                   c["density"] < 1.0)
    return dict(bytes=by, flops=fl)


def tolerance(case):
    if case["kind"] in ("graph", "probe"):
        return "exact"  # integers, and values defined to the last bit
    if case["kind"] == "epoch":
        # sums of 32-bit terms through all layers; a pre-activation within rounding of zero may fall
        # on the other side of the ReLU, which moves single elements of the gradients (other summation
        # orders and native fp32 products: 2e-5 and 2e-4 seen on dW of the first of three layers)
        return dict(rel=1e-4, max=1e-3)
    # the same for single layers: 7e-7 and 9.5e-6 seen (490 entries per row)
    return dict(rel=3e-6, max=4e-5)


# ---------------------------------------------------------------------------
# the same in 64 bits, from the inputs alone
# ---------------------------------------------------------------------------


class _Adj:
    """A + I from the pairs, with the weights of each aggregator."""

    def __init__(self, c, seed):
        n = self.n = c["n"]
        src, dst = (_edges_counted if c["kind"] == "graph" else _edges)(c, seed)
        s, d = src.long(), dst.long()
        me = torch.arange(n, device="cuda")
        keys = torch.unique(torch.cat([s * n + d, d * n + s, me * (n + 1)]))
        del s, d, src, dst
        self.row, self.col = keys // n, keys % n
        self.deg = torch.bincount(self.row, minlength=n)
        self.ptr = torch.cat([torch.zeros(1, dtype=torch.long, device="cuda"), torch.cumsum(self.deg, 0)])
        self.dinv = 1.0 / torch.sqrt(self.deg.double())

    def times(self, agg, M, transpose=False):
        if agg == "gcn":
            val = self.dinv[self.row] * self.dinv[self.col]
        elif agg == "sum":
            val = torch.ones(self.col.numel(), dtype=torch.float64, device="cuda")
        else:
            val = (1.0 / self.deg.double())[self.col if transpose else self.row]
        A = torch.sparse_csr_tensor(self.ptr, self.col, val, (self.n, self.n))
        out = torch.empty_like(M)
        for k in range(0, M.shape[1], 64):
            out[:, k:k + 64] = A @ M[:, k:k + 64].contiguous()
        return out

    def maximum(self, M):
        """The largest neighbour value of each column, and the first neighbour that has it."""
        P, arg = torch.empty_like(M), torch.empty(M.shape, dtype=torch.long, device="cuda")
        step = max(1, int(1.5e9 / self.col.numel()))
        for k in range(0, M.shape[1], step):
            part = M[:, k:k + step].contiguous()
            v = part[self.col]
            P[:, k:k + step] = torch.segment_reduce(v, "max", offsets=self.ptr, axis=0)
            cand = torch.where(v == P[:, k:k + step][self.row], self.col[:, None].double(), float(self.n))
            arg[:, k:k + step] = torch.segment_reduce(cand, "min", offsets=self.ptr, axis=0).long()
        return P, arg


def _cols(X, rows=1 << 17):
    for r in range(0, X.shape[0], rows):
        yield r, X[r:r + rows].double()


def _times_w(X, W):
    """X W by blocks of rows, in 64 bits."""
    out = torch.empty((X.shape[0], W.shape[1]), dtype=torch.float64, device="cuda")
    for r, x in _cols(X):
        out[r:r + x.shape[0]] = x @ W
    return out


def _t_times(X, Q):
    """X^T Q by blocks of rows, in 64 bits."""
    out = torch.zeros((X.shape[1], Q.shape[1]), dtype=torch.float64, device="cuda")
    for r, x in _cols(X):
        out += x.t().contiguous() @ Q[r:r + x.shape[0]]
    return out


def _layer64_fwd(A, agg, first, H, W, b, act, y):
    """(output, saved aggregate, maximisers, loss, logits, Z) of one layer."""
    P = arg = None
    if first:
        P, arg = A.maximum(H.double()) if agg == "max" else (A.times(agg, H.double()), None)
        Z = P @ W + b
    else:
        Z = A.times(agg, _times_w(H, W)) + b
    if act == "relu":
        return Z.clamp(min=0.0), P, arg, None, None, Z
    lp = torch.log_softmax(Z, 1)
    at = torch.arange(A.n, device="cuda")
    loss = -lp[at, y.long()].mean().reshape(1)
    g = lp.exp()
    g[at, y.long()] -= 1.0
    return g / A.n, P, arg, loss, Z, Z


def _layer64_bwd(A, agg, first, grad, H, P, arg, W, below):
    db = grad.sum(0)
    if first:
        dW = P.t() @ grad
        if not below:
            return dW, db, None
        T = grad @ W.t()
        if agg == "max":
            D = torch.zeros_like(T).scatter_add_(0, arg, T)
        else:
            D = A.times(agg, T, transpose=True)
        return dW, db, D * (H > 0)
    Q = A.times(agg, grad, transpose=True)
    return _t_times(H, Q), db, (Q @ W.t()) * (H > 0) if below else None


def exact(case, seed):
    c = case
    if c["kind"] == "probe":
        return None  # counts, offsets and copies of the values
    A = _Adj(c, seed)
    if c["kind"] == "graph":
        return dict(row_ptr=None, col=None, deg=None, dinv=A.dinv, val=A.dinv[A.row] * A.dinv[A.col], order=None)
    if c["kind"] == "layer":
        agg, sparse = c["agg"], c["density"] < 1.0
        H, W, b, y, grad = _layer_inputs(c, seed)
        H = _features(c, c["n"], c["f_in"], seed) if H is None else H
        W, b = W.double(), b.double()
        first = G.layer_order(c["f_in"], c["f_out"], c["index"], ACTS[c["act"]], x_sparse=sparse,
                              agg=AGGS[agg]) == G.AGGREGATE_FIRST
        out, P, arg = {}, None, None
        if c["run"] != "bwd" or first:
            h, P, arg, loss, logits, _ = _layer64_fwd(A, agg, first, H, W, b, c["act"], y)
        if c["run"] != "bwd":
            out = dict(H=h, saved=P, arg=None)
            if logits is not None:
                out.update(loss=loss, logits=logits)
        if c["run"] != "fwd":
            grad = grad.double() if c["run"] == "bwd" else h
            dW, db, Gp = _layer64_bwd(A, agg, first, grad, H, P, arg, W, c["index"] > 0)
            out.update(dW=dW, db=db, Gprev=Gp)
        return out
    w, agg, sparse = _widths(c), c["agg"], c["density"] < 1.0
    n, L = c["n"], c["layers"]
    Ws, bs, mom = _epoch_params(c, seed)
    Ws, bs = [t.double() for t in Ws], [t.double() for t in bs]
    H, kept, hidden = _features(c, n, c["f"], seed), [], []
    y = _labels(n, c["classes"], seed)
    for l in range(L):
        act = "softmax" if l == L - 1 else "relu"
        first = G.layer_order(w[l], w[l + 1], l, ACTS[act], x_sparse=sparse and l == 0) == G.AGGREGATE_FIRST
        h, P, arg, loss, _, _ = _layer64_fwd(A, agg, first, H, Ws[l], bs[l], act, y)
        kept.append((first, H, P, arg))
        if act == "relu":
            hidden.append(h)
        H = h
    dWs, dbs, grad = [None] * L, [None] * L, H
    for l in range(L - 1, -1, -1):
        first, Hl, P, arg = kept[l]
        dWs[l], dbs[l], grad = _layer64_bwd(A, agg, first, grad, Hl, P, arg, Ws[l], l > 0)
    t = _STEP + 1
    out = dict(loss=loss, H=hidden, dW=dWs, db=dbs, W=[], b=[], mW=[], vW=[])
    for k, (p, g) in enumerate(zip(Ws + bs, dWs + dbs)):
        m = 0.9 * mom[k][0].double() + 0.1 * g
        v = 0.999 * mom[k][1].double() + 0.001 * g * g
        new = p - 0.01 * (m / (1.0 - 0.9 ** t)) / ((v / (1.0 - 0.999 ** t)).sqrt() + 1e-8)
        if k < L:
            out["W"].append(new)
            out["mW"].append(m)
            out["vW"].append(v)
        else:
            out["b"].append(new)
    return out
