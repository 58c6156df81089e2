"""The calls that a program using this library makes, at the sizes it makes them: pooling over
sorted segments, fused gather-weight-reduce over a graph's edges, their gradients through the
autograd functions, and a graph-convolution layer.

A case is a dict of plain values. ``prepare`` makes its inputs on the GPU from a seed, ``run`` is
one pass through the public entry points, ``exact`` the same results in 64 bits from plain torch.

Keys: call (below), nnz (rows or edges), segments (output rows), F (columns), lengths (how the
rows spread over the segments), empty (share of segments without rows), reduce, dtype (of src or
X), index (type of the ids); for the fused calls also x_rows (rows of X), cols (how the edges'
sources spread) and weighted; for the layer F_out; for segment_reduce stats (the caller kept the
index's length statistics).
"""
import math

import torch

import paper_2404_03019_amd as geot
from paper_2404_03019_amd import autograd as ga

DTYPES = {"f32": torch.float32, "bf16": torch.bfloat16, "f16": torch.float16}
INDEX = {"i64": torch.int64, "i32": torch.int32}
DEVICE = "cuda"


def listed():
    return [
        # a small pooling (a batch of molecules, a small mesh): latency and launches
        dict(name="pool_small", call="segment_reduce", nnz=65_536, segments=4_096, F=32, lengths="zipf", empty=0.05,
             reduce="sum", dtype="f32", index="i64", stats=False),
        # per-edge scores of a few attention heads, their maximum per node (the softmax's first step)
        dict(name="scores_max", call="segment_reduce", nnz=2_000_000, segments=100_000, F=4, lengths="poisson",
             empty=0.0, reduce="max", dtype="f32", index="i64", stats=False),
        # messages of one narrow hidden layer averaged per node
        dict(name="hidden_mean", call="segment_reduce", nnz=2_000_000, segments=100_000, F=16, lengths="poisson",
             empty=0.0, reduce="mean", dtype="f32", index="i64", stats=False),
        # the benchmark's power-law graph: the largest pooling
        dict(name="powerlaw_sum", call="segment_reduce", nnz=114_615_892, segments=232_965, F=32, lengths="lognormal",
             empty=0.0, reduce="sum", dtype="f32", index="i64", stats=False),
        # a point cloud's k = 16 neighbour features in 16-bit storage, maximum per point
        dict(name="points_max", call="segment_reduce", nnz=16_777_216, segments=1_048_576, F=64, lengths="fixed",
             empty=0.0, reduce="max", dtype="bf16", index="i32", stats=False),
        # class scores (47 columns: no vector width divides a row) pooled in half precision
        dict(name="classes_mean", call="segment_reduce", nnz=1_500_007, segments=170_003, F=47, lengths="lognormal",
             empty=0.1, reduce="mean", dtype="f16", index="i32", stats=False),
        # the benchmark's SpMM graph: the largest fused call (full-graph inference)
        dict(name="spmm_sum", call="gather_scatter", nnz=61_859_140, segments=2_449_029, F=128, lengths="zipf",
             empty=0.0, reduce="sum", dtype="f32", index="i64", x_rows=2_449_029, cols="uniform", weighted=True),
        # inference over a mid-size citation-like graph in 16-bit storage
        dict(name="citation_sum", call="gather_scatter", nnz=1_200_007, segments=170_003, F=128, lengths="lognormal",
             empty=0.05, reduce="sum", dtype="bf16", index="i32", x_rows=170_003, cols="skewed", weighted=True),
        # training on a sampled mini-batch (a new edge list each step): output and both gradients
        dict(name="minibatch_grad", call="gather_grad", nnz=160_007, segments=11_003, F=100, lengths="poisson",
             empty=0.0, reduce="sum", dtype="f32", index="i64", x_rows=90_001, cols="skewed", weighted=True),
        # max aggregation trained on a whole graph: output and the gradient of the features
        dict(name="maxpool_grad", call="gather_grad", nnz=8_000_000, segments=400_000, F=64, lengths="lognormal",
             empty=0.02, reduce="max", dtype="f32", index="i32", x_rows=400_000, cols="skewed", weighted=False),
        # mean pooling trained: output and the gradient of the pooled rows
        dict(name="pool_grad", call="segment_grad", nnz=4_000_000, segments=200_003, F=48, lengths="poisson",
             empty=0.0, reduce="mean", dtype="f32", index="i64"),
        # one graph-convolution layer, forward and backward, on a graph that the program keeps
        dict(name="graph_conv", call="graph_conv", nnz=10_000_000, segments=500_000, F=128, lengths="lognormal",
             empty=0.0, reduce="sum", dtype="f32", index="i64", x_rows=500_000, cols="skewed", weighted=True,
             F_out=64),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case: any of the calls, from about 20,000 rows up to the largest listed work."""
    call = rng.choice(["segment_reduce", "segment_reduce", "gather_scatter", "gather_scatter", "segment_grad",
                       "gather_grad", "graph_conv"])
    F = rng.choice([1, 2, 3, 4, 7, 8, 15, 16, 32, 40, 47, 64, 64, 100, 128, 128, 200, 256])
    # the most elements (rows x columns) and rows of one pass
    cells, rows = {"segment_reduce": (3.6e9, 1.1e8), "gather_scatter": (7.9e9, 6.0e7), "segment_grad": (1.0e9, 3.0e7),
                   "gather_grad": (5.0e8, 8.0e6), "graph_conv": (1.0e9, 1.0e7)}[call]
    if call == "graph_conv":
        F = max(F, 16)
    nnz = _log_int(rng, 2e4, min(rows, cells / F))
    mean = math.exp(rng.uniform(math.log(2.0), math.log(300.0)))
    segments = max(64, min(int(nnz / mean), int(6e8 / F)))
    c = dict(call=call, nnz=nnz, segments=segments, F=F, lengths=rng.choice(["poisson", "lognormal", "zipf", "fixed"]),
             empty=rng.choice([0.0, 0.0, 0.05, 0.3]), reduce=rng.choice(["sum", "mean", "max"]),
             dtype=rng.choice(["f32", "f32", "bf16", "f16"]), index=rng.choice(["i64", "i64", "i32"]))
    if call == "segment_reduce":
        c["stats"] = rng.random() < 0.3
    elif call != "segment_grad":
        c.update(x_rows=segments if call == "graph_conv" else max(64, int(segments * rng.uniform(0.5, 4.0))),
                 cols=rng.choice(["uniform", "skewed"]), weighted=rng.random() < 0.6)
        c["x_rows"] = min(c["x_rows"], int(6e8 / F))
    if call == "graph_conv":
        c.update(dtype="f32", F_out=rng.choice([16, 32, 47, 64, 128]), reduce=rng.choice(["sum", "mean"]))
    return c


# ---------------------------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------------------------
def _lengths(case, g):
    """Segment lengths that add up to nnz, in the case's spread."""
    S, n = case["segments"], case["nnz"]
    u = torch.rand(S, generator=g, device=DEVICE, dtype=torch.float64).clamp_(1e-9, 1.0)
    kind = case["lengths"]
    if kind == "poisson":
        w = torch.poisson(torch.full((S,), n / S, device=DEVICE, dtype=torch.float64), generator=g)
    elif kind == "lognormal":
        w = torch.exp(1.2 * torch.randn(S, generator=g, device=DEVICE, dtype=torch.float64))
    elif kind == "zipf":          # a power law with exponent 2, cut where one segment would hold everything
        w = torch.floor(1.0 / u).clamp_(max=float(S))
    else:
        w = torch.ones_like(u)
    if case["empty"]:
        w = w * (torch.rand(S, generator=g, device=DEVICE) >= case["empty"])
    if float(w.sum()) <= 0:
        w = torch.ones_like(u)
    ends = torch.cumsum(w, 0)
    ends = torch.round(ends * (n / ends[-1])).to(torch.int64)
    ends[-1] = n
    return torch.diff(ends, prepend=ends.new_zeros(1))


def _inputs(case, seed):
    """(values, ids, weight or None, columns or None): everything the pass reads, in its types."""
    g = torch.Generator(device=DEVICE).manual_seed(seed)
    ids = torch.repeat_interleave(torch.arange(case["segments"], device=DEVICE), _lengths(case, g),
                                  output_size=case["nnz"]).to(INDEX[case["index"]])
    fused = "x_rows" in case
    rows = case["x_rows"] if fused else case["nnz"]
    x = torch.randn(rows, case["F"], generator=g, device=DEVICE).to(DTYPES[case["dtype"]])
    col = weight = None
    if fused:
        if case["cols"] == "uniform":
            col = torch.randint(0, rows, (case["nnz"],), generator=g, device=DEVICE)
        else:                     # popular sources: half of the edges come from a quarter of the rows
            u = torch.rand(case["nnz"], generator=g, device=DEVICE, dtype=torch.float64)
            col = torch.randperm(rows, generator=g, device=DEVICE)[(u * u * rows).to(torch.int64).clamp_(max=rows - 1)]
        col = col.to(INDEX[case["index"]])
        if case["weighted"]:
            weight = torch.rand(case["nnz"], generator=g, device=DEVICE)
    return x, ids, weight, col, g


def prepare(case, seed):
    x, ids, weight, col, g = _inputs(case, seed)
    s = dict(case=case, x=x, ids=ids, weight=weight, col=col)
    S, F = case["segments"], case["F"]
    if case["call"] == "segment_reduce":
        s["stats"] = geot.index_stats(ids.long(), S) if case["stats"] else None
    if case["call"] in ("segment_grad", "gather_grad"):
        s["grad"] = torch.randn(S, F, generator=g, device=DEVICE)
        s["x"].requires_grad_()
        if weight is not None:
            s["weight"].requires_grad_()
    if case["call"] == "graph_conv":
        s["grad"] = torch.randn(S, case["F_out"], generator=g, device=DEVICE)
        s["x"].requires_grad_()
        layer = ga.GraphConv(F, case["F_out"], reduce=case["reduce"]).to(DEVICE)
        with torch.no_grad():
            layer.lin.weight.copy_(torch.randn(case["F_out"], F, generator=g, device=DEVICE) / math.sqrt(F))
            layer.bias.copy_(torch.randn(case["F_out"], generator=g, device=DEVICE))
        s["layer"] = layer
        s["graph"] = ga.Graph(col, ids, S, weight, case["x_rows"])
    return s


# ---------------------------------------------------------------------------------------------
# one pass
# ---------------------------------------------------------------------------------------------
def run(s):
    c = s["case"]
    call, S = c["call"], c["segments"]
    if call == "segment_reduce":
        return geot.segment_reduce(s["x"], s["ids"], S, c["reduce"], stats=s["stats"])
    if call == "gather_scatter":
        return geot.gather_scatter(s["x"], s["col"], s["weight"], s["ids"], S, c["reduce"])
    if call == "segment_grad":
        out = ga.segment_reduce(s["x"], s["ids"], S, c["reduce"])
        (gx,) = torch.autograd.grad(out, (s["x"],), s["grad"])
        return {"out": out, "grad_src": gx}
    if call == "gather_grad":
        out = ga.gather_scatter(s["x"], s["col"], s["weight"], s["ids"], S, c["reduce"])
        wrt = (s["x"],) if s["weight"] is None else (s["x"], s["weight"])
        return {"out": out, "grads": torch.autograd.grad(out, wrt, s["grad"])}
    out = s["layer"](s["x"], s["graph"])
    grads = torch.autograd.grad(out, (s["x"], s["layer"].lin.weight, s["layer"].bias), s["grad"])
    return {"out": out, "grads": grads}


# ---------------------------------------------------------------------------------------------
# what a pass cannot do without
# ---------------------------------------------------------------------------------------------
def work(case):
    """Every input read once and every output written once."""
    n, S, F = case["nnz"], case["segments"], case["F"]
    es, ib = (4 if case["dtype"] == "f32" else 2), (4 if case["index"] == "i32" else 8)
    if case["call"] in ("segment_reduce", "segment_grad"):
        bytes_, flops = n * (F * es + ib) + S * F * 4, n * F
        if case["call"] == "segment_grad":     # grad_out read, grad_src written
            bytes_, flops = bytes_ + S * F * 4 + n * F * es, 2 * flops
        return {"bytes": bytes_, "flops": flops}
    weighted = case["weighted"]
    x_bytes = min(case["x_rows"], n) * F * es
    edges = n * (2 * ib + (4 if weighted else 0))
    flops = n * F * (2 if weighted else 1)
    if case["call"] == "gather_scatter":
        return {"bytes": edges + x_bytes + S * F * 4, "flops": flops}
    if case["call"] == "gather_grad":          # out, grad_out, X's gradient and the weights'
        bytes_ = edges + x_bytes + 2 * S * F * 4 + case["x_rows"] * F * es + (n * 4 if weighted else 0)
        return {"bytes": bytes_, "flops": flops * (3 if weighted else 2)}
    # the layer gathers the narrower of its two widths, forward and backward
    Fo, Fm = case["F_out"], min(F, case["F_out"])
    bytes_ = 2 * edges + 2 * case["x_rows"] * F * 4 + 2 * S * Fo * 4 + 2 * F * Fo * 4
    return {"bytes": bytes_, "flops": 2 * n * Fm * (2 if weighted else 1) + 6 * case["x_rows"] * F * Fo}


def tolerance(case):
    """Max is a selection, exact. Sums in fp32 in another order: 1e-7 off 64 bits at every listed
    size and 1e-7 between two orders (the transposed lists' order is free); the layer's weight
    gradient, a product over all nodes, 1.2e-6. Gradients of 16-bit values are rounded to their
    type once, 2e-3 (bf16) and 3e-4 (f16) off."""
    if case["call"] in ("segment_reduce", "gather_scatter") and case["reduce"] == "max":
        return "exact"
    if case["call"] in ("segment_grad", "gather_grad") and case["dtype"] != "f32":
        return {"rel": 8e-3 if case["dtype"] == "bf16" else 1e-3, "max": 2e-2}
    if case["call"] == "graph_conv":
        return {"rel": 5e-6, "max": 1e-4}
    return {"rel": 1e-6, "max": 5e-5}


# ---------------------------------------------------------------------------------------------
# the same results in 64 bits
# ---------------------------------------------------------------------------------------------
_CELLS = 1 << 28                   # elements of 64-bit messages held at a time


def _messages(x, weight, col, lo, hi):
    """Rows [lo, hi) of the messages in 64 bits. A weighted maximum compares products that were
    rounded to fp32 once, as the definition has it; sums take the product unrounded."""
    m = x[lo:hi] if col is None else x[col[lo:hi]]
    m = m.double()
    return m if weight is None else m * weight[lo:hi, None].double()


def _reduce(x, weight, col, ids, S, how):
    """out in 64 bits and, for max, the lowest row attaining each maximum (rows of none: len(ids))."""
    n, F = ids.numel(), x.shape[1]
    step = max(1, _CELLS // F)
    out = torch.full((S, F), -math.inf if how == "max" else 0.0, device=x.device, dtype=torch.float64)
    if how != "max":
        for lo in range(0, n, step):
            hi = min(n, lo + step)
            out.index_add_(0, ids[lo:hi], _messages(x, weight, col, lo, hi))
        if how == "mean":
            out /= torch.bincount(ids, minlength=S).clamp_(min=1)[:, None]
        return out, None

    def message(lo, hi):
        return _messages(x, weight, col, lo, hi).float().double()

    first = torch.full((S, F), n, device=x.device, dtype=torch.int64)
    for lo in range(0, n, step):
        hi = min(n, lo + step)
        out.index_reduce_(0, ids[lo:hi], message(lo, hi), "amax")
    for lo in range(0, n, step):
        hi = min(n, lo + step)
        rows = torch.arange(lo, hi, device=x.device)[:, None].expand(hi - lo, F)
        first.index_reduce_(0, ids[lo:hi], torch.where(message(lo, hi) == out[ids[lo:hi]], rows, n), "amin")
    return torch.where(torch.isinf(out), 0.0, out), first


def _gradients(x, weight, col, ids, grad, how, first):
    """The gradients of x's rows (through col where given) and of the weights, in 64 bits."""
    n, F = ids.numel(), x.shape[1]
    grad = grad.double()
    gx = torch.zeros(x.shape, device=x.device, dtype=torch.float64)
    gw = torch.zeros(n, device=x.device, dtype=torch.float64)
    if how == "max":
        seg, f = torch.nonzero(first < n, as_tuple=True)
        e = first[seg, f]
        src = e if col is None else col[e]
        g = grad[seg, f]
        gx.view(-1).index_add_(0, src * F + f, g if weight is None else g * weight[e].double())
        gw.index_add_(0, e, g * x[src, f].double())
    else:
        if how == "mean":
            grad = grad / torch.bincount(ids, minlength=grad.shape[0]).clamp_(min=1)[:, None]
        step = max(1, _CELLS // F)
        for lo in range(0, n, step):
            hi = min(n, lo + step)
            g = grad[ids[lo:hi]]
            if col is None:
                gx[lo:hi] = g
                continue
            gw[lo:hi] = (g * x[col[lo:hi]].double()).sum(1)
            gx.index_add_(0, col[lo:hi], g if weight is None else g * weight[lo:hi, None].double())
    return gx, gw


def exact(case, seed):
    s = prepare(dict(case, stats=False), seed)
    x, ids, weight = s["x"].detach(), s["ids"].long(), s["weight"]
    weight = weight.detach() if weight is not None else None
    col = s["col"].long() if s["col"] is not None else None
    S, how = case["segments"], case["reduce"]
    if case["call"] == "graph_conv":
        W, h = s["layer"].lin.weight.detach().double(), x.double()
        z = h @ W.t()
        out, first = _reduce(z, weight, col, ids, S, how)
        gz, _ = _gradients(z, weight, col, ids, s["grad"], how, first)
        return {"out": out + s["layer"].bias.detach().double(),
                "grads": (gz @ W, gz.t() @ h, s["grad"].double().sum(0))}
    out, first = _reduce(x, weight, col, ids, S, how)
    if case["call"] in ("segment_reduce", "gather_scatter"):
        return out
    gx, gw = _gradients(x, weight, col, ids, s["grad"], how, first)
    if case["call"] == "segment_grad":
        return {"out": out, "grad_src": gx}
    return {"out": out, "grads": (gx,) if weight is None else (gx, gw)}
