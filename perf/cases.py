"""The work a user of this library has it do, as measurable cases: full-batch training steps, single
layers, the neighbour aggregation alone, the dense combination, edge-weighted aggregation, serving,
sampled batches and plan building, through the public entry points (`LayerStack`, `feed`, `binding`).

Sizes are those of this repository's own workloads (`gt_inputs/configs.py`, `bench.py`), or generic ones
of the same ranges.  `padded` says how the program holds its tensors: rows padded to 16 bytes (what the
header recommends and `LayerStack` does for its own buffers) or plain contiguous torch tensors, whose
row stride is the width itself (what a program has that loads features of 602 or 47 columns).

A graph is an in-edge CSR of exactly `edges` distinct (destination, source) pairs, rows sorted by
source: "rmat" is the power-law generator of `gt_inputs/graphs.py` (0.57, 0.19, 0.19, 0.05), "er" draws
uniform pairs; symmetric-norm graphs have every self-loop.
"""
import numpy as np
import torch

DEV = "cuda:0"


# ------------------------------------------------------------------------------------------------
# the cases
# ------------------------------------------------------------------------------------------------
def _case(kind, name=None, **kw):
    c = dict(kind=kind, **kw)
    if name:
        c["name"] = name
    return c


def listed():
    return [
        # smallest full-graph training step (a citation-graph-sized GCN): launches and latency
        _case("step", "tiny_step", graph="rmat", n=4096, edges=61440, dims="64-64-16", dtype="f32", reduce="symnorm",
              padded=True),
        # the flagship: full-batch training step of a three-layer bf16 GCN on a products-sized power-law graph
        _case("step", "products_step", graph="rmat", n=2097152, edges=52142592, dims="100-256-256-47", dtype="bf16",
              reduce="symnorm", padded=True),
        # first layer of a reddit-sized fp32 GCN (602 features): forward and parameter gradients, rows padded
        _case("layer", "reddit_first_layer", graph="rmat", n=262144, edges=11814051, fin=602, fout=128, dtype="f32",
              reduce="symnorm", relu=True, first=True, padded=True),
        # its last layer (41 classes) on plain contiguous tensors, with the gradient of its input
        _case("layer", "reddit_last_layer", graph="rmat", n=262144, edges=11814051, fin=128, fout=41, dtype="f32",
              reduce="mean", relu=False, first=False, padded=False),
        # aggregation and its derivative alone, on plain contiguous bf16 rows of 47 columns, uniform graph,
        # a vertex count that is no multiple of anything
        _case("pull", "pull_ragged", graph="er", n=1000003, edges=16000048, width=47, dtype="bf16", reduce="mean",
              padded=False),
        # the dense transformation of a 602-feature bf16 layer: forward, input gradient, weight gradient
        _case("apply", "apply_bf16", rows=524288, fin=602, fout=256, dtype="bf16", padded=True),
        # NGCF message passing, width 64: element-wise product, add, mean; forward and both derivatives
        _case("edge", "ngcf", graph="rmat", n=131072, edges=4194304, width=64, dtype="f32", g="mul", h="add",
              reduce="mean", padded=True),
        # dot-product edge scores and scaled aggregation (attention without the softmax), bf16
        _case("edge", "dot_attention", graph="rmat", n=262144, edges=8388608, width=128, dtype="bf16", g="dot", h="scale",
              reduce="sum", padded=True),
        # serving: one aggregation-first layer whose intermediate is never stored (fused entry point)
        _case("infer", "serve_fused", graph="rmat", n=1048576, edges=16777216, fin=128, fout=64, dtype="bf16",
              reduce="mean", fused=True, padded=True),
        # a sampled training batch of 300 seeds from start to end: sample, renumber, look up, plan, step
        _case("batch", "batch_300", n=1048576, edges=25165824, seeds=300, fan1=25, fan2=10, feat=100, hidden=64,
              classes=47, dtype="f32"),
        # the same with 16,384 seeds and 256 features: throughput of batch preparation
        _case("batch", "batch_16k", n=1048576, edges=25165824, seeds=16384, fan1=25, fan2=10, feat=256, hidden=256,
              classes=47, dtype="f32"),
        # the plan of a full graph (degrees, transposed structure, work lists): paid once per graph
        _case("plan", "plan_full", graph="rmat", n=1000003, edges=25000000),
    ]


def _log(rng, lo, hi):
    """A whole number spread over the logarithm of lo..hi; odd ones as likely as even ones."""
    return max(lo, min(hi, int(round(lo * (hi / lo) ** rng.random()))))


def draw(rng):
    kind = rng.choice(["step", "layer", "layer", "pull", "pull", "apply", "edge", "infer", "batch", "plan"])
    dtype = rng.choice(["f32", "bf16"])
    graph = rng.choice(["rmat", "er"])
    reduce = rng.choice(["sum", "mean", "symnorm"])
    padded = rng.random() < 0.5
    n = _log(rng, 4096, 1200000)
    deg = _log(rng, 6, 40)
    if kind == "step":
        widths = [_log(rng, 32, 320), _log(rng, 32, 256), _log(rng, 2, 64)]
        n = min(n, 700000)
        return _case(kind, graph=graph, n=n, edges=n * min(deg, 25), dims="-".join(map(str, widths)), dtype=dtype,
                     reduce=reduce, padded=padded)
    if kind == "layer":
        fin, fout = _log(rng, 16, 640), _log(rng, 16, 256)
        n = min(n, 60000000 // max(fin, fout), 700000)
        return _case(kind, graph=graph, n=n, edges=n * min(deg, 25), fin=fin, fout=fout, dtype=dtype, reduce=reduce,
                     relu=rng.random() < 0.5, first=rng.random() < 0.5, padded=padded)
    if kind == "pull":
        width = _log(rng, 3, 640)
        n = min(n, 120000000 // width)
        return _case(kind, graph=graph, n=n, edges=n * min(deg, 25), width=width, dtype=dtype, reduce=reduce, padded=padded)
    if kind == "apply":
        fin, fout = _log(rng, 16, 1024), _log(rng, 2, 320)
        return _case(kind, rows=_log(rng, 1024, 200000000 // max(fin, fout)), fin=fin, fout=fout, dtype=dtype, padded=padded)
    if kind == "edge":
        g = rng.choice(["mul", "dot"])
        h = "scale" if g == "dot" else rng.choice(["add", "mul"])
        width = _log(rng, 8, 160)
        n = min(n, 300000)
        return _case(kind, graph=graph, n=n, edges=min(n * deg, 300000000 // width), width=width, dtype=dtype, g=g, h=h,
                     reduce=rng.choice(["sum", "mean"]), padded=padded)
    if kind == "infer":
        top = 256 if dtype == "bf16" else 128
        return _case(kind, graph=graph, n=n, edges=n * min(deg, 16), fin=_log(rng, 16, top), fout=_log(rng, 8, 96),
                     dtype=dtype, reduce=reduce, fused=rng.random() < 0.5, padded=True)
    if kind == "batch":
        n = max(n, 200000)
        return _case(kind, n=n, edges=n * deg, seeds=_log(rng, 64, 16384), fan1=rng.choice([5, 15, 25]),
                     fan2=rng.choice([5, 10, 15]), feat=_log(rng, 32, 300), hidden=_log(rng, 16, 256),
                     classes=_log(rng, 2, 64), dtype=dtype)
    return _case("plan", graph=graph, n=n, edges=n * min(deg, 25))


# ------------------------------------------------------------------------------------------------
# inputs (torch on the GPU, from the seed alone)
# ------------------------------------------------------------------------------------------------
def _gen(seed, stream):
    return torch.Generator(device=DEV).manual_seed(int(seed) * 1009 + stream)


def _pairs(kind, n, m, g):
    """m (source, destination) draws on n vertices (R-MAT ids at or above n are drawn again by the caller)."""
    if kind == "er":
        return (torch.randint(0, n, (m,), device=DEV, generator=g), torch.randint(0, n, (m,), device=DEV, generator=g))
    src = torch.zeros(m, dtype=torch.int64, device=DEV)
    dst = torch.zeros(m, dtype=torch.int64, device=DEV)
    for _ in range(max(1, (n - 1).bit_length())):
        r = torch.rand(m, device=DEV, generator=g)
        src = src * 2 + (r >= 0.76)
        dst = dst * 2 + (((r >= 0.57) & (r < 0.76)) | (r >= 0.95))
    ok = (src < n) & (dst < n)
    return src[ok], dst[ok]


def _graph(kind, n, edges, seed, loops):
    """rowptr, colidx (int32): exactly `edges` distinct pairs, rows by destination, sorted by source."""
    g = _gen(seed, 1)
    want = edges - (n if loops else 0)
    keys = torch.empty(0, dtype=torch.int64, device=DEV)
    m = int(want * 1.2) + 1024
    while keys.numel() < want:
        s, d = _pairs(kind, n, m, g)
        k = d * n + s
        if loops:
            k = k[s != d]
        keys = torch.unique(torch.cat([keys, k]))
        m = max(want // 2, 1024)
    if keys.numel() > want:   # leave out what was drawn too many, at random
        r = torch.rand(keys.numel(), device=DEV, generator=g)
        keys = keys[torch.sort(torch.argsort(r)[:want]).values]
    if loops:
        keys = torch.sort(torch.cat([keys, torch.arange(n, device=DEV) * (n + 1)])).values
    dst = torch.div(keys, n, rounding_mode="floor")
    rowptr = torch.zeros(n + 1, dtype=torch.int64, device=DEV)
    rowptr[1:] = torch.cumsum(torch.bincount(dst, minlength=n), 0)
    return rowptr.int(), (keys - dst * n).int()


def _tdt(dtype):
    return torch.bfloat16 if dtype == "bf16" else torch.float32


def _rows(n, F, dtype, padded, g, scale=1.0):
    """A [n, F] tensor of N(0, scale) values, rows padded to 16 bytes or contiguous."""
    v = 8 if dtype == "bf16" else 4
    ld = (F + v - 1) // v * v if padded else F
    t = torch.zeros((n, ld), dtype=_tdt(dtype), device=DEV)
    t[:, :F] = torch.randn((n, F), device=DEV, generator=g) * scale
    return t[:, :F]


def _weight(fin, fout, dtype, g):
    lim = (6.0 / (fin + fout)) ** 0.5
    return ((torch.rand((fin, fout), device=DEV, generator=g) * 2 - 1) * lim).to(_tdt(dtype))


def _inputs(c, seed):
    """Everything the case reads, as plain tensors."""
    kind, g = c["kind"], _gen(seed, 2)
    s = {}
    if kind in ("step", "layer", "pull", "edge", "infer", "plan"):
        s["rowptr"], s["colidx"] = _graph(c["graph"], c["n"], c["edges"], seed, c.get("reduce") == "symnorm")
    if kind == "step":
        dims = [int(d) for d in c["dims"].split("-")]
        s["dims"] = dims
        s["X"] = _rows(c["n"], dims[0], c["dtype"], c["padded"], g)
        s["W"] = [_weight(a, b, c["dtype"], g) for a, b in zip(dims, dims[1:])]
        s["b"] = [torch.randn(b, device=DEV, generator=g) * 0.1 for b in dims[1:]]
        s["G"] = _rows(c["n"], dims[-1], c["dtype"], c["padded"], g)
    elif kind in ("layer", "infer"):
        s["X"] = _rows(c["n"], c["fin"], c["dtype"], c["padded"], g)
        s["W"] = _weight(c["fin"], c["fout"], c["dtype"], g)
        s["b"] = torch.randn(c["fout"], device=DEV, generator=g) * 0.1
        if kind == "layer":
            s["dY"] = _rows(c["n"], c["fout"], c["dtype"], c["padded"], g)
    elif kind == "pull":
        s["X"] = _rows(c["n"], c["width"], c["dtype"], c["padded"], g)
        s["dY"] = _rows(c["n"], c["width"], c["dtype"], c["padded"], g)
    elif kind == "apply":
        s["X"] = _rows(c["rows"], c["fin"], c["dtype"], c["padded"], g)
        s["dZ"] = _rows(c["rows"], c["fout"], c["dtype"], c["padded"], g)
        s["W"] = _weight(c["fin"], c["fout"], c["dtype"], g)
        s["b"] = torch.randn(c["fout"], device=DEV, generator=g) * 0.1
    elif kind == "edge":
        sc = c["width"] ** -0.25 if c["g"] == "dot" else 1.0
        s["Xs"] = _rows(c["n"], c["width"], c["dtype"], c["padded"], g, sc)
        s["Xd"] = _rows(c["n"], c["width"], c["dtype"], c["padded"], g, sc)
        s["dY"] = _rows(c["n"], c["width"], c["dtype"], c["padded"], g)
    elif kind == "batch":
        s["rowptr"], s["colidx"] = _graph("rmat", c["n"], c["edges"], seed, False)
        s["dims"] = [c["feat"], c["hidden"], c["classes"]]
        s["table"] = _rows(c["n"], c["feat"], c["dtype"], True, g)
        s["W"] = [_weight(a, b, c["dtype"], g) for a, b in zip(s["dims"], s["dims"][1:])]
        s["b"] = [torch.randn(b, device=DEV, generator=g) * 0.1 for b in s["dims"][1:]]
        s["seeds"] = torch.randperm(c["n"], device=DEV, generator=g)[:c["seeds"]].int()
        s["G"] = _rows(c["seeds"], c["classes"], c["dtype"], False, g)
        s["key"] = int(seed) % 100003 + 5
    return s


def prepare(case, seed):
    """The tensors, and what a program keeps for them: the graph's plan, the layer's buffers, the model."""
    from paper_2305_17469_amd import binding as B
    from paper_2305_17469_amd.stack import LayerStack
    c, s = case, _inputs(case, seed)
    s["case"] = c
    if c["kind"] in ("layer", "pull", "edge", "infer"):
        s["graph"] = B.Graph(s["rowptr"], s["colidx"], c["n"])
    if c["kind"] == "step":
        blk = dict(rowptr=s["rowptr"], colidx=s["colidx"], n_dst=c["n"], n_src=c["n"])
        s["model"] = LayerStack([blk] * len(s["W"]), s["dims"], c["dtype"], c["reduce"], s["W"], s["b"])
    if c["kind"] in ("layer", "infer"):
        # as in LayerStack: the layer above hands down a gradient that carries this layer's ReLU derivative
        s["desc"] = B.make_desc(c["reduce"], c["dtype"], c.get("relu", True), c["fin"], c["fout"],
                                need_dx=c["kind"] == "layer" and not c["first"], dy_is_dz=True)
        s["bufs"] = B.LayerBuffers(s["graph"], s["desc"])
        if c["kind"] == "infer" and c["fused"]:
            s["fused"] = B.gt_aggregate_combine_supported(c["dtype"], c["fin"], c["fout"])
    return s


# ------------------------------------------------------------------------------------------------
# one pass
# ------------------------------------------------------------------------------------------------
def run(s):
    from paper_2305_17469_amd import binding as B, feed
    from paper_2305_17469_amd.stack import LayerStack
    c = s["case"]
    kind = c["kind"]
    if kind == "step":
        m = s["model"]
        m.step(s["X"], s["G"])
        return dict(out=m.H[-1], dW=list(m.dW), db=list(m.db))
    if kind == "layer":
        Y, used = B.gt_layer_fwd(s["graph"], s["desc"], s["X"], s["W"], s["b"], s["bufs"])
        r = B.gt_layer_bwd(s["graph"], s["desc"], used, s["dY"], s["X"], s["W"], Y, s["bufs"])
        out = dict(Y=Y, dW=r["dW"], db=r["db"])
        if not c["first"]:
            out["dX"] = r["dX"]
        return out
    if kind == "infer":
        if s.get("fused"):
            return dict(Y=B.gt_aggregate_combine_fwd(s["graph"], c["reduce"], s["X"], s["W"], s["b"], relu=True))
        return dict(Y=B.gt_layer_fwd(s["graph"], s["desc"], s["X"], s["W"], s["b"], s["bufs"], inference=True)[0])
    if kind == "pull":
        return dict(Y=B.gt_aggregate_fwd(s["graph"], c["reduce"], s["X"]), dX=B.gt_aggregate_bwd(s["graph"], c["reduce"], s["dY"]))
    if kind == "apply":
        return dict(Y=B.gt_combine(s["X"], s["W"], s["b"], relu=True), dX=B.gt_combine(s["dZ"], s["W"], transB=True),
                    dW=B.gt_combine(s["X"], s["dZ"], transA=True, out_dtype=torch.float32))
    if kind == "edge":
        gr = s["graph"]
        w = B.gt_neighbor_apply_fwd(gr, c["g"], s["Xs"], s["Xd"])
        y = B.gt_pull_fwd(gr, c["reduce"], c["h"], s["Xs"], w)
        dxs, dw = B.gt_pull_bwd(gr, c["reduce"], c["h"], s["dY"], s["Xs"], w)
        dxs2, dxd = B.gt_neighbor_apply_bwd(gr, c["g"], dw, s["Xs"], s["Xd"])
        return dict(w=w, y=y, dxs=dxs, dw=dw, dxs2=dxs2, dxd=dxd)
    if kind == "batch":
        blocks, X = feed.prepare_batch(s["rowptr"], s["colidx"], s["table"], s["seeds"], (c["fan1"], c["fan2"]), s["key"])
        m = LayerStack(blocks, s["dims"], c["dtype"], "mean", s["W"], s["b"])
        m.step(X, s["G"])
        # the sizes of the blocks depend on what was sampled; the rows nearest the seeds always have one shape
        return dict(out=m.H[-1], dW=list(m.dW), db=list(m.db), rows=blocks[-1]["rowptr"],
                    sizes=[n for b in blocks for n in (b["n_dst"], b["n_src"], b["colidx"].numel())])
    g = B.Graph(s["rowptr"], s["colidx"], c["n"])
    s["last"] = g   # a program keeps the plan it built
    return dict(zip(("in_deg", "out_deg", "rowptr_t", "colidx_t", "perm"), g.outputs()))


# ------------------------------------------------------------------------------------------------
# what the path cannot do without
# ------------------------------------------------------------------------------------------------
def work(case):
    """Every input read once, every output written once (gathered tables once, not once per edge); the
    multiply-adds of the cheaper of the two placements."""
    c, kind = case, case["kind"]
    es = 2 if c.get("dtype") == "bf16" else 4

    def layer(n_src, n_dst, E, fi, fo, first, bwd=True):
        b = (n_src * fi + n_dst * fo + fi * fo) * es + 4 * (E + n_dst)
        f = 2 * n_dst * fi * fo + 2 * E * min(fi, fo)
        if bwd:
            b += (n_dst * fo + n_src * fi) * es + 4 * fi * fo
            f += 2 * n_dst * fi * fo
            if not first:
                b += n_src * fi * es + 4 * (E + n_src)
                f += 2 * n_dst * fi * fo + 2 * E * min(fi, fo)
        return b, f

    if kind == "step":
        d = [int(x) for x in c["dims"].split("-")]
        parts = [layer(c["n"], c["n"], c["edges"], a, b, l == 0) for l, (a, b) in enumerate(zip(d, d[1:]))]
        return dict(bytes=sum(p[0] for p in parts), flops=sum(p[1] for p in parts))
    if kind in ("layer", "infer"):
        b, f = layer(c["n"], c["n"], c["edges"], c["fin"], c["fout"], c.get("first", True), kind == "layer")
        return dict(bytes=b, flops=f)
    if kind == "pull":
        return dict(bytes=2 * (2 * c["n"] * c["width"] * es + 4 * (c["edges"] + c["n"])), flops=4 * c["edges"] * c["width"])
    if kind == "apply":
        r, a, b = c["rows"], c["fin"], c["fout"]
        return dict(bytes=(3 * r * (a + b) + 3 * a * b) * es, flops=6 * r * a * b)
    if kind == "edge":
        n, E, F = c["n"], c["edges"], c["width"]
        ew = 4 * E if c["g"] == "dot" else E * F * es   # one edge tensor: written, read, its gradient written and read
        return dict(bytes=4 * ew + 8 * n * F * es + 16 * E, flops=12 * E * F)
    if kind == "batch":
        # most vertices of a power-law graph have few in-edges, and samples meet the same hubs again: about a fifth
        # and four fifths of what the fanouts allow, out of about a quarter of the vertices (from sampled sizes)
        met = lambda x: c["n"] / 4 * (1 - np.exp(-x / (c["n"] / 4)))   # noqa: E731
        d1 = 0.2 * c["fan1"] * c["seeds"]
        n1 = met(c["seeds"] + d1)
        d2 = 0.8 * c["fan2"] * n1
        n2 = met(n1 + d2)
        b1, f1 = layer(n2, n1, d2, c["feat"], c["hidden"], True)
        b2, f2 = layer(n1, c["seeds"], d1, c["hidden"], c["classes"], False)
        return dict(bytes=int(b1 + b2 + 2 * n2 * c["feat"] * es + 24 * (d1 + d2)), flops=int(f1 + f2))
    return dict(bytes=4 * (3 * c["edges"] + 4 * c["n"]), flops=c["edges"])


def tolerance(case):
    """Single layers: fp32 sums, or results and a layer's intermediate rounded to bf16 (measured against 64 bits: up
    to 3e-6 and 2e-3).  Whole models: a value next to zero may come out on the other side of the ReLU, and its
    gradient with it: one such decision in a small fp32 model, about one in 500 in a bf16 one (measured against 64
    bits: 2.8e-4 and 3.2e-2 of a weight gradient)."""
    if case["kind"] == "plan":
        return "exact"
    if case["kind"] in ("step", "batch"):
        return {"rel": 3e-2, "max": 0.9} if case["dtype"] == "bf16" else {"rel": 1e-2, "max": 0.25}
    return {"rel": 1e-2, "max": 5e-2} if case["dtype"] == "bf16" else {"rel": 1e-5, "max": 1e-3}


# ------------------------------------------------------------------------------------------------
# the same in 64 bits, plain torch
# ------------------------------------------------------------------------------------------------
def _rep(rowptr):
    deg = (rowptr[1:] - rowptr[:-1]).long()
    return torch.repeat_interleave(torch.arange(deg.numel(), device=DEV), deg), deg


def _coef(rows, cols, deg, reduce):
    if reduce == "sum":
        return None
    d = deg.double()
    if reduce == "mean":
        return 1.0 / d[rows]
    inv = torch.where(d > 0, d.clamp(min=1).rsqrt(), torch.zeros_like(d))
    return inv[rows] * inv[cols]


def _scatter(X, src, dst, coef, n_out, w=None):
    """out[dst] += coef * X[src] (* w), a few million terms at a time."""
    out = torch.zeros((n_out, X.shape[1]), dtype=torch.float64, device=DEV)
    step = max(1, 200000000 // max(1, X.shape[1]))
    for i in range(0, src.numel(), step):
        t = X[src[i:i + step]]
        if coef is not None:
            t = t * coef[i:i + step, None]
        if w is not None:
            t = t * w[i:i + step]
        out.index_add_(0, dst[i:i + step], t)
    return out


def _model64(blocks, X, W, b, G, reduce):
    """Layers act(A X W + b), ReLU on all but the last; returns the output and the parameter gradients.
    The cheaper order of A and W (same function).  Gradients that pass through a ReLU are left out: they jump where a
    pre-activation is at rounding level, so no computation in another precision has their value."""
    L, hs, es = len(W), [X], []
    for rowptr, colidx in blocks:
        rows, deg = _rep(rowptr)
        cols = colidx.long()
        es.append((rows, cols, _coef(rows, cols, deg, reduce), deg.numel()))
    for l in range(L):
        rows, cols, cf, nd = es[l]
        h = hs[-1]
        if W[l].shape[1] < W[l].shape[0]:
            z = _scatter(h @ W[l], cols, rows, cf, nd) + b[l]
        else:
            z = _scatter(h, cols, rows, cf, nd) @ W[l] + b[l]
        hs.append(z.clamp(min=0) if l < L - 1 else z)
    dW, db = [None] * L, [None] * L
    rows, cols, cf, nd = es[-1]
    db[-1] = G.sum(0)
    dW[-1] = hs[-2].t() @ _scatter(G, rows, cols, cf, hs[-2].shape[0])
    return hs[-1], dW, db


def _mix32(x):
    x = x ^ (x >> np.uint32(16))
    x = x * np.uint32(0x7FEB352D)
    x = x ^ (x >> np.uint32(15))
    x = x * np.uint32(0x846CA68B)
    return x ^ (x >> np.uint32(16))


def _sample64(rowptr, colidx, dst, fanout, key, hop):
    """Rows and global ids of the keyed sample: lists of at most `fanout` whole, of at most 64 in the order of
    their positions' keys, longer ones through the six-round Feistel permutation."""
    u = np.uint32
    gold = 0x9E3779B9
    rk = _mix32(_mix32(np.array([(key + gold * hop) & 0xFFFFFFFF], dtype=u)) ^ dst.astype(u))
    e0, d = rowptr[dst].astype(np.int64), (rowptr[dst + 1] - rowptr[dst]).astype(np.int64)
    cnt = np.minimum(d, fanout)
    out = np.zeros(dst.size + 1, dtype=np.int64)
    np.cumsum(cnt, out=out[1:])
    row = np.repeat(np.arange(dst.size), cnt)
    t = np.arange(out[-1]) - out[:-1][row]
    pos = t.copy()
    mid = (d > fanout) & (d <= 64)
    if mid.any():
        j = np.arange(64, dtype=u)
        k = _mix32(rk[mid][:, None] + (j[None, :] + u(1)) * u(gold)).astype(np.int64)
        k[j[None, :].astype(np.int64) >= d[mid][:, None]] = 1 << 40
        order = np.argsort(k, axis=1, kind="stable")
        where = np.cumsum(mid) - 1
        m = mid[row]
        pos[m] = order[where[row[m]], t[m]]
    big = ((d > fanout) & (d > 64))[row]
    if big.any():
        r, x, dd = rk[row[big]], t[big].astype(u), d[row[big]]
        bits = np.ceil(np.log2(dd.astype(np.float64))).astype(np.int64)
        h = ((bits + 1) // 2).astype(u)
        mask = (u(1) << h) - u(1)
        keys = [_mix32(r + u((gold * (i + 1)) & 0xFFFFFFFF)) for i in range(6)]
        todo = np.ones(x.size, dtype=bool)
        while todo.any():
            L, R, hh, mm = x[todo] >> h[todo], x[todo] & mask[todo], h[todo], mask[todo]
            for i in range(6):
                L, R = R, L ^ (_mix32(R ^ keys[i][todo]) & mm)
            x[todo] = (L << hh) | R
            todo &= x >= dd
        pos[big] = x
    return out, colidx[e0[row] + pos]


def _batch64(c, s):
    rowptr, colidx = s["rowptr"].cpu().numpy(), s["colidx"].cpu().numpy()
    dst, blocks = s["seeds"].cpu().numpy().astype(np.int64), []
    for hop, fanout in enumerate((c["fan1"], c["fan2"])):
        ptr, picked = _sample64(rowptr, colidx, dst, fanout, s["key"], hop)
        seen = np.concatenate([dst, picked.astype(np.int64)])
        ids, first = np.unique(seen, return_index=True)
        order = np.argsort(first, kind="stable")
        local = np.empty(ids.size, dtype=np.int64)
        local[order] = np.arange(ids.size)
        loc = local[np.searchsorted(ids, picked)]
        blocks.append((torch.from_numpy(ptr).to(DEV), torch.from_numpy(loc).to(DEV)))
        dst = ids[order]
    blocks.reverse()
    return blocks, s["table"][torch.from_numpy(dst).to(DEV)].double()


def exact(case, seed):
    c, kind = case, case["kind"]
    if kind == "plan":
        return None
    s = _inputs(case, seed)
    D = lambda t: t.double()   # noqa: E731
    if kind == "step":
        out, dW, db = _model64([(s["rowptr"], s["colidx"])] * len(s["W"]), D(s["X"]), [D(w) for w in s["W"]],
                               [D(b) for b in s["b"]], D(s["G"]), c["reduce"])
        return dict(out=out, dW=dW, db=db)
    if kind == "batch":
        blocks, X = _batch64(c, s)
        out, dW, db = _model64(blocks, X, [D(w) for w in s["W"]], [D(b) for b in s["b"]], D(s["G"]), "mean")
        return dict(out=out, dW=dW, db=db, rows=None, sizes=None)
    if kind == "apply":
        X, W, dZ = D(s["X"]), D(s["W"]), D(s["dZ"])
        return dict(Y=(X @ W + D(s["b"])).clamp(min=0), dX=dZ @ W.t(), dW=X.t() @ dZ)
    rows, deg = _rep(s["rowptr"])
    cols, n = s["colidx"].long(), c["n"]
    cf = _coef(rows, cols, deg, c["reduce"])
    if kind == "pull":
        return dict(Y=_scatter(D(s["X"]), cols, rows, cf, n), dX=_scatter(D(s["dY"]), rows, cols, cf, n))
    if kind in ("layer", "infer"):
        X, W = D(s["X"]), D(s["W"])
        z = (_scatter(X @ W, cols, rows, cf, n) if c["fout"] < c["fin"] else _scatter(X, cols, rows, cf, n) @ W) + D(s["b"])
        Y = z.clamp(min=0) if kind == "infer" or c["relu"] else z
        if kind == "infer":
            return dict(Y=Y)
        dZ = D(s["dY"])
        S = _scatter(dZ, rows, cols, cf, n)
        out = dict(Y=Y, dW=X.t() @ S, db=dZ.sum(0))
        if not c["first"]:
            out["dX"] = S @ W.t()
        return out
    # edge weighting, one primitive after the other
    xs, xd, dY = D(s["Xs"]), D(s["Xd"]), D(s["dY"])
    inv = torch.ones(n, dtype=torch.float64, device=DEV) if c["reduce"] == "sum" else 1.0 / deg.clamp(min=1).double()
    gy = (dY * inv[:, None])[rows]
    w = (xs[cols] * xd[rows]).sum(1) if c["g"] == "dot" else xs[cols] * xd[rows]
    wv = w[:, None] if c["g"] == "dot" else w
    if c["h"] == "add":
        y = _scatter(xs, cols, rows, None, n) + torch.zeros_like(dY).index_add_(0, rows, w)
        dw = gy
        dxs = torch.zeros_like(xs).index_add_(0, cols, gy)
    else:
        y = _scatter(xs, cols, rows, None, n, wv)
        dw = (gy * xs[cols]).sum(1) if c["h"] == "scale" else gy * xs[cols]
        dxs = torch.zeros_like(xs).index_add_(0, cols, gy * wv)
    y = y * inv[:, None]
    dv = dw[:, None] if c["g"] == "dot" else dw
    return dict(w=w, y=y, dxs=dxs, dw=dw, dxs2=torch.zeros_like(xs).index_add_(0, cols, dv * xd[rows]),
                dxd=torch.zeros_like(xd).index_add_(0, rows, dv * xs[cols]))
