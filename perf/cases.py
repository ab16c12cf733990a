"""What this library is timed on: the work a program that trains or serves graph neural networks has it do.

A case is a dict of plain values.  ``kind`` names the calls:

    gcn      a GCN layer's aggregation, forward (bias and activation in its epilogue) and backward
    step     the same on a graph that changes from pass to pass: both plans rebuilt and the CSC formed
             each time (sampled or rewired graphs)
    sage     a GraphSAGE layer's mean and max aggregation, the max with the edges attaining it
    gat      a GAT layer's attention on given scores, forward and backward, through the forward's row softmax states
             (``keep`` "states") or its attention weights (``keep`` "alpha", every per-edge gradient out)
    scores   the two SDDMM forms on their own: additive scores with the edge softmax, and dot products
    dense    a layer's feature transform and the attention scores of its heads
    infer    2-layer GCN and GAT inference, whole calls
    codec    activation compression and its decoder

Sizes are those of this repository's workloads (graphs shaped like citation, ogbn and Reddit graphs), of
its tests, and generic ones.  Graphs are random with a power-law degree (R-MAT with permuted ids, or
Chung-Lu where the mean degree is in the hundreds), columns sorted in each row, one self-loop per node.
"""
from __future__ import annotations

import math

import torch

import paper_2103_00959_amd as cg

DTYPES = {"f32": torch.float32, "bf16": torch.bfloat16, "f16": torch.float16}
SLOPE = 0.2


def listed():
    return [
        # citation graph (2.7k nodes), hidden width 64 in fp32: the smallest training call, launch latency
        {"name": "gcn_small", "kind": "gcn", "graph": "rmat", "n": 2708, "nnz": 13264, "F": 64,
         "dtype": "f32", "plan": "plain", "bias": False},
        # ogbn-arxiv-sized training in fp32 on a graph that changes every step: setup and both directions
        {"name": "step_medium", "kind": "step", "graph": "rmat", "n": 169343, "nnz": 2501829, "F": 128,
         "dtype": "f32", "plan": "sliced"},
        # full-batch training on a skewed 122M-edge graph, bf16 features: the benchmark's aggregation
        {"name": "gcn_large", "kind": "gcn", "graph": "rmat", "n": 2400000, "nnz": 122400000, "F": 256,
         "dtype": "bf16", "plan": "sliced", "bias": False},
        # GraphSAGE mean and max over 300-wide input features (word vectors) in bf16
        {"name": "sage_medium", "kind": "sage", "graph": "rmat", "n": 169343, "nnz": 2501829, "F": 300,
         "dtype": "bf16", "plan": "plain"},
        # a GCN's output layer: 41 classes (an odd width), with its bias, on an ogbn-products-sized graph
        {"name": "gcn_classes", "kind": "gcn", "graph": "rmat", "n": 2449029, "nnz": 64308169, "F": 41,
         "dtype": "bf16", "plan": "sliced", "bias": True},
        # a hidden GAT layer's training pass on the 122M-edge graph, 4 heads of 64 in bf16
        {"name": "gat_large", "kind": "gat", "graph": "rmat", "n": 2400000, "nnz": 122400000, "H": 4, "D": 64,
         "dtype": "bf16", "plan": "sliced", "keep": "states"},
        # 8 heads of 16 in fp32 on the ogbn-products-sized graph, attention weights and their gradients kept
        {"name": "gat_heads", "kind": "gat", "graph": "rmat", "n": 2449029, "nnz": 64308169, "H": 8, "D": 16,
         "dtype": "f32", "plan": "sliced", "keep": "alpha"},
        # a GAT's output layer: one head of 41 classes, medium graph
        {"name": "gat_classes", "kind": "gat", "graph": "rmat", "n": 169343, "nnz": 2501829, "H": 1, "D": 41,
         "dtype": "bf16", "plan": "plain", "keep": "states"},
        # attention scores on their own (link scoring, attention analysis)
        {"name": "scores_medium", "kind": "scores", "graph": "rmat", "n": 400000, "nnz": 12000000, "H": 4, "D": 32,
         "dtype": "bf16", "plan": "plain"},
        # the input layer of a Reddit-sized graph: 602 features to 4 heads of 32
        {"name": "dense_input", "kind": "dense", "n": 232965, "k": 602, "H": 4, "D": 32, "dtype": "bf16"},
        # serving: both 2-layer models on a Reddit-sized graph (114.6M edges)
        {"name": "infer_reddit", "kind": "infer", "graph": "power", "n": 232965, "nnz": 114615892, "k": 602,
         "hidden": 128, "heads": 4, "classes": 41, "dtype": "bf16", "plan": "sliced"},
        # activation-compressed training: 256-wide activations of 2.4M nodes at 2 bits and back
        {"name": "codec_large", "kind": "codec", "n": 2400000, "F": 256, "dtype": "bf16", "bits": 2, "group": 256},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _width(rng, lo, hi):
    """A layer width: half of them multiples of 8, the others any number (classes, raw features)."""
    w = _log(rng, lo, hi)
    return max(8, w // 8 * 8) if rng.random() < 0.5 else w


def _heads(rng):
    H = rng.choice([1, 2, 3, 4, 8])
    D = rng.choice([8, 16, 32, 64]) if rng.random() < 0.6 else rng.randint(5, 80)
    return H, D


def _draw_graph(rng, c, width, most_edges=60_000_000, most_gather=8.0e9, lo=2000, hi=2_400_000):
    """Nodes and edges over the whole range, the gathered elements (edges x width) bounded."""
    n = _log(rng, lo, hi)
    nnz = int(n * math.exp(rng.uniform(math.log(4), math.log(100))))
    nnz = min(nnz, most_edges, int(most_gather / width), n * max(2, n // 8))
    n = min(n, nnz // 3)
    c.update(graph=rng.choice(["rmat", "rmat", "power"]), n=n, nnz=nnz)
    c["plan"] = rng.choice(["plain", "sliced", "none"] if nnz <= 3_000_000 else ["plain", "sliced"])
    return c


def draw(rng):
    kind = rng.choice(["gcn", "gcn", "step", "sage", "gat", "gat", "scores", "dense", "infer", "codec"])
    dt = rng.choice(["f32", "bf16", "f16"])
    c = {"kind": kind, "dtype": dt}
    if kind in ("gcn", "step", "sage"):
        c["F"] = _width(rng, 8, 512)
        _draw_graph(rng, c, c["F"], most_edges=40_000_000 if kind == "step" else 60_000_000,
                    most_gather=2.0e9 if kind == "sage" else 8.0e9)
        if kind == "gcn":
            c["bias"] = rng.random() < 0.5
        if kind == "step" and c["plan"] == "none":
            c["plan"] = "plain"
    elif kind in ("gat", "scores"):
        c["H"], c["D"] = _heads(rng)
        _draw_graph(rng, c, c["H"] * c["D"], most_edges=30_000_000, most_gather=1.0e9)
        if kind == "gat":
            c["keep"] = rng.choice(["states", "alpha"])
    elif kind == "dense":
        c["dtype"] = rng.choice(["bf16", "f16"])
        c["k"] = _width(rng, 16, 1500)
        c["H"], c["D"] = _heads(rng)
        c["n"] = min(_log(rng, 2000, 2_400_000), 600_000_000 // c["k"])
    elif kind == "infer":
        c.update(dtype=rng.choice(["bf16", "f16"]), k=_width(rng, 32, 1000), hidden=rng.choice([64, 128, 256]),
                 heads=rng.choice([1, 4, 8]), classes=rng.randint(2, 64))
        _draw_graph(rng, c, c["hidden"], most_edges=50_000_000, most_gather=6.0e9, hi=500_000)
    else:
        F = rng.choice([64, 128, 256, 512]) if rng.random() < 0.6 else _log(rng, 32, 600)
        c.update(F=F, n=min(_log(rng, 2000, 2_400_000), 600_000_000 // F), bits=rng.choice([2, 3, 4, 8]),
                 group=rng.choice([64, 128, 256]))
    return c


# --------------------------------------------------------------- inputs

def _gen(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed) * 7919 + 17)
    return g


def _rmat_keys(n, m, g):
    """m draws of an R-MAT edge (a, b, c = .57, .19, .19) as row * n + column, node ids permuted."""
    levels = max(1, (n - 1).bit_length())
    r = torch.zeros(m, dtype=torch.int64, device="cuda")
    c = torch.zeros(m, dtype=torch.int64, device="cuda")
    for _ in range(levels):
        u = torch.rand(m, device="cuda", generator=g)
        r.mul_(2).add_(u >= 0.76)
        c.mul_(2).add_(((u >= 0.57) & (u < 0.76)) | (u >= 0.95))
    perm = torch.randperm(n, device="cuda", generator=g)
    r = perm[(r * n) >> levels]
    return r.mul_(n).add_(perm[(c * n) >> levels])


def _power_keys(n, m, g):
    """m draws of a Chung-Lu edge: both ends by weights from a power law on [1, 20000] (mean about 490)."""
    k, top = 0.29, 20000.0
    w = (1.0 - torch.rand(n, device="cuda", generator=g, dtype=torch.float64) * (1.0 - top ** -k)).pow_(-1.0 / k)
    at = torch.cumsum(w, 0)
    at /= at[-1].clone()

    def ends():
        u = torch.rand(m, device="cuda", generator=g, dtype=torch.float64)
        return torch.searchsorted(at, u).clamp_(max=n - 1)

    return ends().mul_(n).add_(ends())


def _graph(case, g):
    """(rowptr, col) int32 of exactly nnz edges, one self-loop per node, columns sorted in each row."""
    n, nnz = case["n"], case["nnz"]
    want = nnz - n
    keys = (_rmat_keys if case["graph"] == "rmat" else _power_keys)(n, int(want * 1.2), g)
    keys = torch.unique(keys)
    # exactly the wanted number, spread evenly (a few repeated edges where a small graph ran out)
    at = torch.arange(want, device="cuda", dtype=torch.int64).mul_(keys.numel()).div_(want, rounding_mode="floor")
    loops = torch.arange(n, device="cuda", dtype=torch.int64).mul_(n + 1)
    keys = torch.sort(torch.cat([keys[at], loops])).values
    row = torch.div(keys, n, rounding_mode="floor")
    col = (keys - row * n).to(torch.int32)
    rowptr = torch.zeros(n + 1, dtype=torch.int32, device="cuda")
    rowptr[1:] = torch.cumsum(torch.bincount(row, minlength=n), 0)
    return rowptr, col


def _normal(shape, g, dtype=torch.float32, scale=1.0):
    x = torch.randn(shape, device="cuda", generator=g)
    return (x if scale == 1.0 else x.mul_(scale)).to(dtype)


def _rows(rowptr):
    n = rowptr.numel() - 1
    return torch.repeat_interleave(torch.arange(n, device="cuda"), rowptr.diff().long())


def _inputs(case, seed):
    """The tensors a call gets, from the seed alone."""
    g, kind, dt = _gen(seed), case["kind"], DTYPES[case["dtype"]]
    s = {}
    if "graph" in case:
        n, nnz = case["n"], case["nnz"]
        rowptr, col = s["rowptr"], s["col"] = _graph(case, g)
        if kind in ("gcn", "step", "sage", "infer"):
            # symmetric normalization, as a GCN's program computes it once
            deg = rowptr.diff().float().rsqrt_()
            indeg = torch.bincount(col, minlength=n).float().clamp_(min=1).rsqrt_()
            s["val"] = deg[_rows(rowptr)] * indeg[col.long()]
    n = case["n"]
    if kind in ("gcn", "step", "sage"):
        s["X"] = _normal((n, case["F"]), g, dt)
        if kind != "sage":
            s["G"] = _normal((n, case["F"]), g, dt)
        if case.get("bias"):
            s["bias"] = _normal((case["F"],), g)
    elif kind in ("gat", "scores"):
        H, D = case["H"], case["D"]
        s["X"] = _normal((n, H, D), g, dt)
        s["P"] = _normal((n, H, D), g, dt)
        s["s_src"], s["s_dst"] = (
            (s["X"].float() * _normal((H, D), g, scale=D ** -0.5)).sum(-1) for _ in range(2))
    elif kind == "dense":
        H, D, k = case["H"], case["D"], case["k"]
        s["X"] = _normal((n, k), g, dt)
        s["W"] = _normal((H * D, k), g, dt, k ** -0.5)
        s["b"] = _normal((H * D,), g)
        s["a_src"] = _normal((H, D), g, scale=D ** -0.5)
        s["a_dst"] = _normal((H, D), g, scale=D ** -0.5)
    elif kind == "infer":
        k, hid, H, C = case["k"], case["hidden"], case["heads"], case["classes"]
        s["X"] = _normal((n, k), g, dt)
        both = {"W1": _normal((hid, k), g, dt, k ** -0.5), "b1": _normal((hid,), g, scale=0.1),
                "W2": _normal((C, hid), g, dt, hid ** -0.5), "b2": _normal((C,), g, scale=0.1)}
        s["gcn"] = dict(both)
        s["gat"] = dict(both, a_src1=_normal((H, hid // H), g, scale=(hid // H) ** -0.5),
                        a_dst1=_normal((H, hid // H), g, scale=(hid // H) ** -0.5),
                        a_src2=_normal((1, C), g, scale=C ** -0.5), a_dst2=_normal((1, C), g, scale=C ** -0.5))
    else:
        s["X"] = _normal((n, case["F"]), g, dt)
        s["seed"] = int(seed) * 1000003 + 12345
    return s


def _plan(case, rowptr, col, width, heads):
    if case["plan"] == "none":
        return None
    sliced = {"col": col, "n_cols": case["n"]} if case["plan"] == "sliced" else {}
    return cg.Plan(rowptr, case["nnz"], max_feat=width, max_heads=heads, **sliced)


def prepare(case, seed):
    s = _inputs(case, seed)
    kind = s["kind"] = case["kind"]
    s["case"] = case
    if "graph" not in case:
        return s
    if kind == "infer":
        C8 = (case["classes"] + 7) // 8 * 8
        s["plan"] = _plan(case, s["rowptr"], s["col"], max(case["hidden"], C8), case["heads"])
        return s
    width, heads = (case["F"], 0) if "F" in case else (case["H"] * case["D"], case["H"])
    s["plan"] = _plan(case, s["rowptr"], s["col"], width, heads)
    if kind in ("gcn", "step", "gat"):
        csc = cg.csr_to_csc(s["rowptr"], s["col"], s.get("val"), case["n"])
        s["colptr"], s["row_t"], s["val_t"], s["perm"] = csc
        s["plan_t"] = _plan(case, s["colptr"], s["row_t"], width, heads)
    if kind == "step":
        s["workspace"] = torch.empty(cg.csr_to_csc_workspace(case["n"], case["n"], case["nnz"]),
                                     dtype=torch.uint8, device="cuda")
    return s


# --------------------------------------------------------------- one pass

def run(s):
    return _RUN[s["kind"]](s)


def _run_gcn(s):
    if "bias" in s:
        Y = cg.gspmm(s["rowptr"], s["col"], s["val"], s["X"], "sum", plan=s["plan"], bias=s["bias"])
    else:
        Y = cg.spmm(s["rowptr"], s["col"], s["val"], s["X"], plan=s["plan"])
    dX = cg.spmm_t(s["colptr"], s["row_t"], s["val_t"], s["G"], plan_t=s["plan_t"])
    return {"Y": Y, "dX": dX}


def _run_step(s):
    s["plan"].rebuild(s["rowptr"], s["col"] if s["plan"].sliced else None)
    Y = cg.spmm(s["rowptr"], s["col"], s["val"], s["X"], plan=s["plan"])
    colptr, row_t, val_t, perm = cg.csr_to_csc(s["rowptr"], s["col"], s["val"], s["case"]["n"],
                                               workspace=s["workspace"])
    s["plan_t"].rebuild(colptr, row_t if s["plan_t"].sliced else None)
    dX = cg.spmm_t(colptr, row_t, val_t, s["G"], plan_t=s["plan_t"])
    return {"Y": Y, "dX": dX, "colptr": colptr, "row_t": row_t, "val_t": val_t, "perm": perm}


def _run_sage(s):
    mean = cg.gspmm(s["rowptr"], s["col"], None, s["X"], "mean", plan=s["plan"])
    top, arg = cg.gspmm(s["rowptr"], s["col"], s["val"], s["X"], "max", plan=s["plan"], return_arg=True)
    return {"mean": mean, "max": top, "arg": arg}


def _run_gat(s):
    s_src, s_dst = s["s_src"], s["s_dst"]
    args = (s["rowptr"], s["col"], s["colptr"], s["row_t"], s["perm"], s_dst, s_src)
    if s["case"]["keep"] == "states":
        Y, st = cg.gat_aggregate_stats(s["rowptr"], s["col"], s_dst, s["X"], s_src=s_src, negative_slope=SLOPE,
                                       plan=s["plan"])
        o = cg.gat_backward(*args, None, s["X"], s["P"], SLOPE, plan=s["plan"], plan_t=s["plan_t"], row_stats=st,
                            out={"dalpha": None, "dscore": None})
        return {"Y": Y, "states": st, "dX": o["dX"], "ds_dst": o["ds_dst"], "ds_src": o["ds_src"]}
    Y, alpha = cg.gat_aggregate(s["rowptr"], s["col"], s_dst, s_src, s["X"], SLOPE, return_alpha=True, plan=s["plan"])
    o = cg.gat_backward(*args, alpha, s["X"], s["P"], SLOPE, plan=s["plan"], plan_t=s["plan_t"])
    return {"Y": Y, "alpha": alpha, "dX": o["dX"], "ds_dst": o["ds_dst"], "ds_src": o["ds_src"],
            "dalpha": o["dalpha"], "dscore": o["dscore"]}


def _run_scores(s):
    alpha = cg.sddmm_edge_softmax(s["rowptr"], s["col"], s["s_dst"], s["s_src"], SLOPE, plan=s["plan"])
    dot = cg.sddmm_dot(s["rowptr"], s["col"], s["P"], s["X"], plan=s["plan"])
    return {"alpha": alpha, "dot": dot}


def _run_dense(s):
    H, D = s["a_src"].shape
    Z = cg.linear(s["X"], s["W"], s["b"])
    s_src, s_dst = cg.head_scores(Z.view(-1, H, D), s["a_src"], s["a_dst"])
    return {"Z": Z, "s_src": s_src, "s_dst": s_dst}


def _run_infer(s):
    gcn = cg.gcn_forward(s["rowptr"], s["col"], s["val"], s["X"], s["gcn"], plan=s["plan"])
    gat = cg.gat_forward(s["rowptr"], s["col"], s["X"], s["gat"], SLOPE, plan=s["plan"])
    return {"gcn": gcn, "gat": gat}


def _run_codec(s):
    c = s["case"]
    codes, stats = cg.act_compress(s["X"], c["bits"], c["group"], s["seed"])
    out = cg.act_decompress(codes, stats, c["n"], c["F"], c["bits"], c["group"], out_dtype=s["X"].dtype)
    return {"codes": codes, "stats": stats, "out": out}


_RUN = {"gcn": _run_gcn, "step": _run_step, "sage": _run_sage, "gat": _run_gat, "scores": _run_scores,
        "dense": _run_dense, "infer": _run_infer, "codec": _run_codec}


# --------------------------------------------------------------- what a pass cannot do without

def work(case):
    """Each input read once, each output written once; the arithmetic of the sums themselves."""
    kind, n, b = case["kind"], case["n"], 4 if case["dtype"] == "f32" else 2
    E = case.get("nnz", 0)
    csr = 4 * (n + 1) + 4 * E
    if kind in ("gcn", "step"):
        one = csr + 4 * E + 2 * n * case["F"] * b
        setup = (csr + 4 * E + 4 * (n + 1) + 12 * E) if kind == "step" else 0
        return {"bytes": 2 * one + setup, "flops": 4 * E * case["F"]}
    if kind == "sage":
        F = case["F"]
        return {"bytes": 2 * csr + 4 * E + 2 * n * F * b + 2 * n * F * b + 4 * n * F, "flops": 3 * E * F}
    if kind == "gat":
        H, W = case["H"], case["H"] * case["D"]
        fwd = csr + 8 * n * H + 2 * n * W * b
        # the CSR pass (dY, X, scores), then the CSC pass (row ids, edge ids, dY, dX, score gradients)
        bwd = csr + 2 * n * W * b + 12 * n * H + csr + 4 * E + 2 * n * W * b + 4 * n * H
        kept = 8 * n * H * 2 if case["keep"] == "states" else 8 * E * H + 8 * E * H
        return {"bytes": fwd + bwd + kept, "flops": E * (6 * W + 20 * H)}
    if kind == "scores":
        H, W = case["H"], case["H"] * case["D"]
        return {"bytes": 8 * n * H + 2 * csr + 2 * n * W * b + 8 * E * H, "flops": E * (2 * W + 10 * H)}
    if kind == "dense":
        k, W, H = case["k"], case["H"] * case["D"], case["H"]
        return {"bytes": n * k * b + W * k * b + 2 * n * W * b + 8 * n * H, "flops": 2 * n * k * W + 4 * n * W}
    if kind == "infer":
        k, hid, C, H = case["k"], case["hidden"], case["classes"], case["heads"]
        dense = n * k * b + n * hid * b + n * hid * b + n * C * b
        agg = 2 * csr + 2 * n * (hid + C) * b
        return {"bytes": 2 * (dense + agg) + 8 * E + 16 * n * (H + 1),
                "flops": 4 * n * hid * (k + C) + 4 * E * (hid + C) + 12 * E * (H + 1)}
    F = case["F"]
    groups = n * ((F + case["group"] - 1) // case["group"])
    packed = groups * (case["group"] * case["bits"] // 8 + 8)
    return {"bytes": 2 * (n * F * b + packed), "flops": 30 * n * F}


def tolerance(case):
    """bf16 and fp16 results are rounded once to 8 or 11 bits from fp32 sums, so two correct results differ by
    a last place here and there; fp32 results by the order of their sums."""
    kind, dt = case["kind"], case["dtype"]
    if kind == "codec":
        return "exact"                       # codes, minima and steps are defined bit for bit
    if kind == "infer":
        return {"rel": 1e-2, "max": 0.1}     # three stored 16-bit layers
    if dt == "f32":
        # score gradients are differences of nearly equal sums
        return {"rel": 4e-6, "max": 1e-3} if kind == "gat" else {"rel": 1e-6, "max": 1e-4}
    return {"rel": 4e-3, "max": 3e-2}


# --------------------------------------------------------------- the same in 64 bits

#: Elements of one chunk of gathered rows (float64).
CHUNK = 1 << 28


def _chunks(E, width):
    step = max(1, CHUNK // max(1, width))
    return [(b, min(E, b + step)) for b in range(0, E, step)]


def _sum_rows(n, at, src, w, X):
    """out[at[k]] += w[k] * X[src[k]] in float64; X [m, H, D] or [m, F], w [E, H] or [E] (None: ones)."""
    out = torch.zeros((n,) + tuple(X.shape[1:]), dtype=torch.float64, device="cuda")
    for b, e in _chunks(src.numel(), X[0].numel()):
        x = X[src[b:e]]
        if w is not None:
            x *= w[b:e].unsqueeze(-1)
        out.index_add_(0, at[b:e], x)
    return out


def _softmax(n, row, col, s_dst, s_src):
    t = s_dst[row] + s_src[col]
    e = torch.where(t > 0, t, SLOPE * t)
    m = torch.full((n, e.shape[1]), -math.inf, dtype=torch.float64, device="cuda")
    m.index_reduce_(0, row, e, "amax")
    p = torch.exp(e - m[row])
    z = torch.zeros_like(m).index_add_(0, row, p)
    return t, m, z, p / z[row]


def _dots(row, col, P, Q):
    out = torch.empty((row.numel(), P.shape[1]), dtype=torch.float64, device="cuda")
    for b, e in _chunks(row.numel(), 2 * P[0].numel()):
        out[b:e] = (P[row[b:e]] * Q[col[b:e]]).sum(-1)
    return out


def exact(case, seed):
    s, kind, n = _inputs(case, seed), case["kind"], case["n"]
    d = {k: v.double() for k, v in s.items() if isinstance(v, torch.Tensor) and v.is_floating_point()}
    if kind == "codec":
        F, G = case["F"], case["group"]
        ng = (F + G - 1) // G
        x, stats = d["X"], torch.empty((n, ng, 2), dtype=torch.float64, device="cuda")
        for j in range(ng):
            lo, hi = x[:, j * G:(j + 1) * G].aminmax(dim=1)
            stats[:, j, 0], stats[:, j, 1] = lo, (hi - lo) / (2 ** case["bits"] - 1)
        return {"codes": None, "stats": stats.reshape(-1), "out": None}
    if kind == "dense":
        H, D = s["a_src"].shape
        Z = d["X"] @ d["W"].T + d["b"]
        z = Z.view(n, H, D)
        return {"Z": Z, "s_src": (z * d["a_src"]).sum(-1), "s_dst": (z * d["a_dst"]).sum(-1)}
    row, col = _rows(s["rowptr"]), s["col"].long()
    if kind in ("gcn", "step"):
        Y = _sum_rows(n, row, col, d["val"], d["X"])
        if "bias" in d:
            Y += d["bias"]
        o = {"Y": Y, "dX": _sum_rows(n, col, row, d["val"], d["G"])}
        return dict(o, colptr=None, row_t=None, val_t=None, perm=None) if kind == "step" else o
    if kind == "sage":
        deg = s["rowptr"].diff().double().clamp_(min=1).unsqueeze(1)
        top = torch.full((n, case["F"]), -math.inf, dtype=torch.float64, device="cuda")
        for b, e in _chunks(case["nnz"], case["F"]):
            top.index_reduce_(0, row[b:e], d["X"][col[b:e]] * d["val"][b:e].unsqueeze(1), "amax")
        return {"mean": _sum_rows(n, row, col, None, d["X"]) / deg, "max": top, "arg": None}
    if kind == "infer":
        X = d["X"]
        p = {k: v.double() for k, v in s["gat"].items()}
        H = case["heads"]
        Z = X @ p["W1"].T
        h = torch.relu(_sum_rows(n, row, col, d["val"], Z) + p["b1"])
        gcn = _sum_rows(n, row, col, d["val"], h @ p["W2"].T) + p["b2"]
        z = Z.view(n, H, -1)
        al = _softmax(n, row, col, (z * p["a_dst1"]).sum(-1), (z * p["a_src1"]).sum(-1))[3]
        h = torch.nn.functional.elu(_sum_rows(n, row, col, al, z).reshape(n, -1) + p["b1"])
        z = (h @ p["W2"].T).unsqueeze(1)
        al = _softmax(n, row, col, (z * p["a_dst2"]).sum(-1), (z * p["a_src2"]).sum(-1))[3]
        return {"gcn": gcn, "gat": _sum_rows(n, row, col, al, z).reshape(n, -1) + p["b2"]}
    X, P = d["X"], d["P"]
    t, m, z, al = _softmax(n, row, col, d["s_dst"], d["s_src"])
    if kind == "scores":
        return {"alpha": al, "dot": _dots(row, col, P, X)}
    da = _dots(row, col, P, X)
    c = torch.zeros_like(m).index_add_(0, row, al * da)
    ds = torch.where(t > 0, 1.0, SLOPE) * al * (da - c[row])
    o = {"Y": _sum_rows(n, row, col, al, X), "dX": _sum_rows(n, col, row, al, P),
         "ds_dst": torch.zeros_like(m).index_add_(0, row, ds), "ds_src": torch.zeros_like(m).index_add_(0, col, ds)}
    if case["keep"] == "states":
        return dict(o, states=torch.stack([m, 1.0 / z], 1))
    return dict(o, alpha=al, dalpha=da, dscore=ds)
