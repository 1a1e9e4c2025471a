"""The work that users of this library have it do, as cases that can be timed and checked.

Each case is one pass through the public binding (``paper_2507_16991_amd``) with what a user's
program would have in hand prepared beforehand: graphs drawn on the GPU from the seed, features,
and, where a program keeps them between passes, the CSR, its transpose and the plans.  The sizes
are those of the workloads that ``graphgen`` names (2.7k nodes and 10.6k edges; 169k and 1.17M;
2.45M and 124M; a tenth of 100M and 1.6B; the typed graph of 20.6M edges) or generic ones.

Kinds of case:
  layer       one aggregation over a cached CSR and plan (inference, or the forward of a layer)
  minibatch   a graph seen once: COO->CSR with edge weights, plan, weighted sum
  train       forward and gradients of one aggregation over cached CSR, transpose and plans
  index       the cached formats of a new graph: CSR with edge ids, and its transpose
  hetero      typed graph: combined CSR over all node types, plan, sum over relations
  stacked     several aggregations of one gather (mean, min, max, std)
  readout     a batch of small graphs: segment pointers, plan, stacked global readout
  projection  typed projections on the matrix cores, forward and both gradients
  explain     explanation mode: materialized messages under an edge mask, and its gradients
"""
import math

import torch

import paper_2507_16991_amd as mp

DEV = "cuda:0"
DT = {"f32": torch.float32, "bf16": torch.bfloat16}
REDUCE = {"sum": mp.MP_SUM, "mean": mp.MP_MEAN, "max": mp.MP_MAX, "sum+max": mp.MP_SUM | mp.MP_MAX,
          "mean+max": mp.MP_MEAN | mp.MP_MAX}
STATS = ["mean", "min", "max", "std"]  # the aggregators of principal neighbourhood aggregation
READOUT = ["sum", "mean", "max", "std"]


def listed():
    return [
        # the smallest call: one layer over a graph of a few thousand nodes, where the launches
        # and the host's share count
        dict(name="layer-10k", kind="layer", graph="uniform", n=2708, e=10556, f=64, dtype="f32",
             reduce="sum", weighted=False, idx64=False),
        # neighbour sampling: every step brings a small graph of its own, converted and planned
        dict(name="minibatch-10k", kind="minibatch", graph="uniform", n=2708, e=10556, f=64,
             dtype="f32"),
        # full-batch training with learned edge weights on an ordinary graph: weighted sum and
        # its gradients with respect to features and weights
        dict(name="train-weighted-1.2M", kind="train", graph="powerlaw", n=169343, e=1166243,
             f=128, dtype="f32", reduce="sum", weighted=True),
        # a large graph read in: CSR with edge ids, and the transpose that the backward uses
        dict(name="index-124M", kind="index", graph="chunglu", n=2449029, e=123718280),
        # full-graph inference on it, the headline aggregation
        dict(name="layer-sum-124M", kind="layer", graph="chunglu", n=2449029, e=123718280, f=100,
             dtype="f32", reduce="sum", weighted=False, idx64=False),
        # max pooling in training on it, mixed precision (bf16 features, fp32 gradients)
        dict(name="train-max-124M", kind="train", graph="chunglu", n=2449029, e=123718280, f=100,
             dtype="bf16", reduce="max", weighted=False),
        # low degrees and one huge hub (a web graph), 64-bit rowptr, two aggregations fused
        dict(name="layer-fused-160M", kind="layer", graph="zipf", n=10000000, e=160000000, f=64,
             dtype="bf16", reduce="sum+max", weighted=False, idx64=True),
        # typed nodes and relations, all destination types at once, bf16
        dict(name="hetero-20M", kind="hetero", na=1900000, nb=736000, nc=8700, e0=5400000,
             e1=7100000, e2=7100000, e3=1000000, f=128, dtype="bf16"),
        # stacked aggregators at a width that no vector width divides
        dict(name="stacked-12M", kind="stacked", graph="chunglu", n=244903, e=12371828, f=75,
             dtype="f32"),
        # graph classification: 1,024 graphs in a batch
        dict(name="readout-2.4M", kind="readout", n=2449029, graphs=1024, f=100, dtype="bf16"),
        # typed projections of a training step over the typed graph's node tables
        dict(name="projection-2.6M", kind="projection", na=1900000, nb=736000, nc=8700, f=128,
             fo=128, out="f32"),
        # one step of an explainer that learns an edge mask
        dict(name="explain-1.2M", kind="explain", graph="powerlaw", n=169343, e=1166243, f=128,
             dtype="f32"),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["layer", "layer", "minibatch", "train", "train", "index", "hetero", "stacked",
                       "readout", "projection", "explain"])
    dtype = rng.choice(["f32", "bf16"])
    graph = rng.choice(["uniform", "powerlaw", "chunglu"])
    f = _log(rng, 8, 512)
    n = _log(rng, 2000, 1000000)
    e = n * _log(rng, 2, 64) + rng.randrange(n)
    if kind in ("layer", "train", "stacked"):
        # at most 2^32 gathered elements a pass
        f = max(8, min(f, (1 << 32) // e))
    if kind == "layer":
        return dict(kind=kind, graph=graph, n=n, e=e, f=f, dtype=dtype,
                    reduce=rng.choice(["sum", "mean", "max", "sum+max", "mean+max"]),
                    weighted=rng.random() < 0.3, idx64=rng.random() < 0.3)
    if kind == "minibatch":
        n = _log(rng, 1000, 200000)
        return dict(kind=kind, graph=graph, n=n, e=n * _log(rng, 2, 16) + rng.randrange(n), f=f,
                    dtype=dtype)
    if kind == "train":
        reduce = rng.choice(["sum", "mean", "max"])
        return dict(kind=kind, graph=graph, n=n, e=e, f=f, dtype=dtype, reduce=reduce,
                    weighted=rng.random() < 0.4)
    if kind == "index":
        return dict(kind=kind, graph=graph, n=n, e=e)
    if kind == "hetero":
        return dict(kind=kind, na=n, nb=n // 3 + 1, nc=n // 50 + 1, e0=n * 3, e1=n * 4 + 1,
                    e2=n * 4 + 3, e3=n // 2 + 1, f=min(f, 256), dtype=dtype)
    if kind == "stacked":
        return dict(kind=kind, graph=graph, n=n, e=e, f=f, dtype=dtype)
    if kind == "readout":
        graphs = _log(rng, 32, 8192)
        n = graphs * _log(rng, 10, 2000) + rng.randrange(graphs)
        return dict(kind=kind, n=n, graphs=graphs, f=max(8, min(f, (1 << 29) // n)), dtype=dtype)
    if kind == "projection":
        return dict(kind=kind, na=n, nb=n // 3 + 1, nc=n // 50 + 1, f=8 * _log(rng, 2, 64),
                    fo=8 * _log(rng, 2, 64), out=dtype)
    n = _log(rng, 2000, 200000)
    e = n * _log(rng, 2, 32) + rng.randrange(n)
    return dict(kind=kind, graph=graph, n=n, e=e, f=max(8, min(f, (1 << 29) // e)), dtype="f32")


# ---- inputs ----------------------------------------------------------------------------------

def _gen(seed, stream):
    g = torch.Generator(device=DEV)
    g.manual_seed(1000003 * int(seed) + stream)
    return g


def _ranks(seed, stream, n, e, beta):
    """E draws of a rank in [0, n) with probability proportional to about (rank + 1) ^ -beta, by
    the inverse of the continuous distribution function."""
    u = torch.rand(e, generator=_gen(seed, stream), device=DEV, dtype=torch.float64)
    if beta == 1.0:
        r = torch.exp(u * math.log(n + 1.0))
    else:
        a = 1.0 - beta
        r = (u * ((n + 1.0) ** a - 1.0) + 1.0) ** (1.0 / a)
    return (r.to(torch.int64) - 1).clamp_(0, n - 1)


def _uniform_ids(seed, stream, n, e):
    return torch.randint(0, n, (e,), generator=_gen(seed, stream), device=DEV, dtype=torch.int32)


def _graph(c, seed):
    """(src, dst) of the case's graph, int32."""
    n, e = c["n"], c["e"]
    if c["graph"] == "uniform":
        return _uniform_ids(seed, 1, n, e), _uniform_ids(seed, 2, n, e)
    ids = torch.randperm(n, generator=_gen(seed, 3), device=DEV).to(torch.int32)
    if c["graph"] == "chunglu":  # both ends by one power law of weights
        return ids[_ranks(seed, 1, n, e, 0.43423)], ids[_ranks(seed, 2, n, e, 0.43423)]
    # destinations by a Zipf-like law, sources uniform
    beta = 1.0 if c["graph"] == "zipf" else 0.909
    return _uniform_ids(seed, 1, n, e), ids[_ranks(seed, 2, n, e, beta)]


def _normal(seed, stream, shape, dtype="f32"):
    return torch.randn(shape, generator=_gen(seed, stream), device=DEV, dtype=torch.float32).to(DT[dtype])


def _gcn_weights(src, dst, n):
    """1 / sqrt(out-degree * in-degree) per edge, fp32."""
    od = torch.bincount(src, minlength=n).to(torch.float64)
    di = torch.bincount(dst, minlength=n).to(torch.float64)
    return (od[src.long()] * di[dst.long()]).rsqrt().to(torch.float32)


def _weights(c, seed, src, dst):
    if not c.get("weighted"):
        return None
    return _gcn_weights(src, dst, c["n"])


def _typed_sizes(c):
    return [c["na"], c["nb"], c["nc"]]


def _relations(c, seed):
    npt = _typed_sizes(c)
    ends = [(0, 0), (0, 1), (1, 0), (1, 2)]
    return [(s, d, _uniform_ids(seed, 10 + r, npt[s], c["e%d" % r]),
             _uniform_ids(seed, 20 + r, npt[d], c["e%d" % r])) for r, (s, d) in enumerate(ends)]


def _segments(c, seed):
    """Sorted graph id of every node: each graph has at least one node."""
    n, k = c["n"], c["graphs"]
    cuts = torch.randperm(n - 1, generator=_gen(seed, 5), device=DEV)[:k - 1] + 1
    first = torch.zeros(n, dtype=torch.int32, device=DEV)
    first[cuts] = 1
    return torch.cumsum(first, 0, dtype=torch.int32)


def _rowptr_dtype(c):
    return torch.int64 if c.get("idx64") else torch.int32


def prepare(c, seed):
    k = c["kind"]
    s = {"c": c}
    if k == "layer" or k == "stacked":
        src, dst = _graph(c, seed)
        w = _weights(c, seed, src, dst)
        s["rowptr"], s["col"], _, s["w"] = mp.coo_to_csr(src, dst, c["n"], val=w,
                                                         rowptr_dtype=_rowptr_dtype(c))
        s["x"] = _normal(seed, 4, (c["n"], c["f"]), c["dtype"])
        s["plan"] = mp.Plan(s["rowptr"], c["e"], c["f"], DT[c["dtype"]])
    elif k == "minibatch":
        s["src"], s["dst"] = _graph(c, seed)
        s["w"] = _gcn_weights(s["src"], s["dst"], c["n"])
        s["x"] = _normal(seed, 4, (c["n"], c["f"]), c["dtype"])
    elif k == "train":
        src, dst = _graph(c, seed)
        w = _weights(c, seed, src, dst)
        s["rowptr"], s["col"], _, s["w"] = mp.coo_to_csr(src, dst, c["n"], val=w)
        s["rowptrT"], s["colT"], s["posT"], s["wT"] = mp.csr_transpose(s["rowptr"], s["col"], c["n"],
                                                                       val=s["w"])
        s["plan"] = mp.Plan(s["rowptr"], c["e"], c["f"], DT[c["dtype"]])
        s["planT"] = mp.Plan(s["rowptrT"], c["e"], c["f"], torch.float32)
        s["x"] = _normal(seed, 4, (c["n"], c["f"]), c["dtype"])
        s["g"] = _normal(seed, 6, (c["n"], c["f"]))
    elif k == "index":
        s["src"], s["dst"] = _graph(c, seed)
    elif k == "hetero":
        s["rels"] = _relations(c, seed)
        s["x"] = [_normal(seed, 30 + t, (n, c["f"]), c["dtype"]) for t, n in enumerate(_typed_sizes(c))]
    elif k == "readout":
        s["batch"] = _segments(c, seed)
        s["ids"] = torch.arange(c["n"], dtype=torch.int32, device=DEV)
        s["x"] = _normal(seed, 4, (c["n"], c["f"]), c["dtype"])
    elif k == "projection":
        n, f, fo = sum(_typed_sizes(c)), c["f"], c["fo"]
        s["seg"] = [0, c["na"], c["na"] + c["nb"], n]
        s["x"] = _normal(seed, 4, (n, f), "bf16")
        s["W"] = (_normal(seed, 7, (3, f, fo)) / math.sqrt(f)).to(torch.bfloat16)
        s["g"] = _normal(seed, 6, (n, fo), "bf16")
    else:  # explain
        src, dst = _graph(c, seed)
        s["rowptr"], s["col"], s["perm"], _ = mp.coo_to_csr(src, dst, c["n"], want_perm=True)
        s["rowptrT"], _, s["posT"], _ = mp.csr_transpose(s["rowptr"], s["col"], c["n"])
        s["plan"] = mp.Plan(s["rowptr"], c["e"], c["f"])
        s["planT"] = mp.Plan(s["rowptrT"], c["e"], c["f"])
        s["x"] = _normal(seed, 4, (c["n"], c["f"]))
        s["g"] = _normal(seed, 6, (c["n"], c["f"]))
        s["mask"] = torch.sigmoid(_normal(seed, 8, (c["e"],)))  # per COO edge, as it is learned
    return s


# ---- one pass --------------------------------------------------------------------------------

def run(s):
    c = s["c"]
    k = c["kind"]
    if k == "layer":
        red = REDUCE[c["reduce"]]
        # the max of unweighted bf16 messages is one of them, kept as it is
        exact_max = red & mp.MP_MAX and c["dtype"] == "bf16" and s["w"] is None
        out, mx, arg = mp.spmm(s["rowptr"], s["col"], s["x"], red, w=s["w"], plan=s["plan"],
                               max_dtype=torch.bfloat16 if exact_max else None)
        return {"out": out, "max": mx, "arg": arg}
    if k == "minibatch":
        rowptr, col, _, w = mp.coo_to_csr(s["src"], s["dst"], c["n"], val=s["w"])
        plan = mp.Plan(rowptr, c["e"], c["f"], DT[c["dtype"]])
        out, _, _ = mp.spmm(rowptr, col, s["x"], mp.MP_SUM, w=w, plan=plan)
        return {"rowptr": rowptr, "col": col, "w": w, "out": out}
    if k == "train":
        red = REDUCE[c["reduce"]]
        out, mx, arg = mp.spmm(s["rowptr"], s["col"], s["x"], red, w=s["w"], plan=s["plan"])
        gx = mp.spmm_backward_x(s["rowptrT"], s["colT"], s["g"], red, posT=s["posT"], wT=s["wT"],
                                rowptr=s["rowptr"], argout=arg, planT=s["planT"])
        gw = None
        if s["w"] is not None:
            gw = mp.spmm_backward_w(s["rowptr"], s["col"], s["x"], s["g"], red, argout=arg)
        return {"out": mx if arg is not None else out, "arg": arg, "gx": gx, "gw": gw}
    if k == "index":
        rowptr, col, perm, _ = mp.coo_to_csr(s["src"], s["dst"], c["n"], want_perm=True)
        rowptrT, colT, posT, _ = mp.csr_transpose(rowptr, col, c["n"])
        return {"rowptr": rowptr, "col": col, "perm": perm, "rowptrT": rowptrT, "colT": colT,
                "posT": posT}
    if k == "hetero":
        npt = _typed_sizes(c)
        rowptr, col = mp.hetero_build(npt, s["rels"], mp.MP_ALL_TYPES)
        plan = mp.Plan(rowptr, int(col.numel()), c["f"], DT[c["dtype"]])
        out = mp.hetero_spmm(npt, s["x"], mp.MP_ALL_TYPES, rowptr, col, plan=plan)
        return {"rowptr": rowptr, "col": col, "out": out}
    if k == "stacked":
        return mp.spmm_multi(s["rowptr"], s["col"], s["x"], STATS, plan=s["plan"])
    if k == "readout":
        ptr, _, _, _ = mp.sorted_coo_to_csr(s["ids"], s["batch"], c["graphs"])
        plan = mp.Plan(ptr, c["n"], c["f"], DT[c["dtype"]])
        return mp.readout(ptr, s["x"], READOUT, plan=plan)
    if k == "projection":
        out = mp.segment_matmul(s["seg"], s["x"], s["W"], out_dtype=DT[c["out"]])
        dx, dW = mp.segment_matmul_backward(s["seg"], s["x"], s["W"], s["g"], dx_dtype=DT[c["out"]])
        return {"out": out, "dx": dx, "dW": dW}
    msg = mp.message_gather(s["col"], s["x"])
    masked = mp.message_scale(msg, s["mask"], idx=s["perm"])
    out, _, _ = mp.message_aggregate(s["rowptr"], masked, mp.MP_SUM, plan=s["plan"])
    dmasked = mp.message_backward(s["rowptr"], s["g"], mp.MP_SUM, E=c["e"])
    gmask = mp.edge_dot(dmasked, msg, oidx=s["perm"])
    dmsg = mp.message_scale(dmasked, s["mask"], idx=s["perm"])
    gx, _, _ = mp.spmm(s["rowptrT"], s["posT"], dmsg, mp.MP_SUM, plan=s["planT"])
    return {"out": out, "gmask": gmask, "gx": gx}


# ---- what a pass cannot do without -----------------------------------------------------------

def work(c):
    k = c["kind"]
    b = 2 if c.get("dtype") == "bf16" else 4
    if k in ("hetero", "projection"):
        n = sum(_typed_sizes(c))
    else:
        n = c["n"]
    f, e = c.get("f", 0), c.get("e", 0)
    if k == "layer":
        red = REDUCE[c["reduce"]]
        out = (4 if red & (mp.MP_SUM | mp.MP_MEAN) else 0)
        if red & mp.MP_MAX:
            out += 4 + (2 if b == 2 and not c["weighted"] else 4)
        rp = 8 if c["idx64"] else 4
        return {"bytes": rp * (n + 1) + 4 * e + (4 * e if c["weighted"] else 0) + n * f * (b + out),
                "flops": e * f * (2 if c["weighted"] else 1)}
    if k == "minibatch":
        return {"bytes": 12 * e + 4 * (n + 1) + 8 * e + n * f * (b + 4), "flops": 2 * e * f}
    if k == "train":
        mx = c["reduce"] == "max"
        w = 1 if c["weighted"] else 0
        # forward: CSR, weights, x, output (and argmax); gradients: the transpose (and positions),
        # weights, g, gx; weights' gradient
        by = 8 * (n + 1) + 8 * e + 12 * w * e + n * f * (b + 4 + 4 + 4)
        if mx:
            by += 4 * n * f + 4 * e
        return {"bytes": by, "flops": (2 + w * 4) * e * f}
    if k == "index":
        return {"bytes": 8 * e + 4 * (n + 1) + 8 * e + 4 * (n + 1) + 8 * e, "flops": 0}
    if k == "hetero":
        e = c["e0"] + c["e1"] + c["e2"] + c["e3"]
        return {"bytes": 8 * e + 4 * e + 4 * (n + 1) + n * f * (b + 4), "flops": e * f}
    if k == "stacked":
        return {"bytes": 4 * (n + 1) + 4 * e + n * f * (b + 4 * 6), "flops": 6 * e * f}
    if k == "readout":
        return {"bytes": 4 * n + n * f * b + c["graphs"] * f * 4 * 5, "flops": 5 * n * f}
    if k == "projection":
        fo, o = c["fo"], 2 if c["out"] == "bf16" else 4
        return {"bytes": n * (f + fo) * (2 + o) + 3 * f * fo * (2 + 4), "flops": 6 * n * f * fo}
    # explain: the tables of messages are what this mode is asked to materialize
    return {"bytes": 4 * (n + 1) + 8 * e + 3 * 4 * n * f + 4 * n * f + 8 * e + 4 * 4 * e * f,
            "flops": 7 * e * f}


def tolerance(c):
    """About four times what fp32 accumulation in the library's order shows against 64 bits: sums
    within 1.9e-7 and gradients of typed weights (over up to 1.9M rows) within 3.3e-7, the standard
    deviation within 2.7e-7, and one rounding to bf16 at 1.7e-3."""
    k = c["kind"]
    if k == "index":
        return "exact"
    if k == "projection":
        return {"rel": 1.4e-6 if c["out"] == "f32" else 7e-3}
    if k == "stacked" or k == "readout":
        return {"rel": 1.2e-6}
    return {"rel": 8e-7}


# ---- the same in 64 bits ---------------------------------------------------------------------

CHUNK = 1 << 28  # gathered elements at a time


def _csr64(dst, n, src):
    """Stable destination-major order by torch alone: (rowptr, col, order)."""
    key, order = torch.sort(dst, stable=True)
    rowptr = torch.searchsorted(key, torch.arange(n + 1, device=DEV, dtype=key.dtype))
    return rowptr, src[order], order, key


def _pieces(row):
    """Pieces of at most 64 positions of one row each (row is sorted): the piece of every position,
    and the row of every piece.  Adding up by pieces first keeps a hub row's additions apart."""
    new = torch.ones(row.numel(), dtype=torch.bool, device=DEV)
    new[1:] = row[1:] != row[:-1]
    new |= torch.arange(row.numel(), device=DEV) % 64 == 0
    return torch.cumsum(new, 0) - 1, row[new].long()


def _add_rows(out, row, m):
    piece, at = _pieces(row)
    part = torch.zeros(at.numel(), m.shape[1], dtype=m.dtype, device=DEV)
    out.index_add_(0, at, part.index_add_(0, piece, m))


def _best_rows(out, row, m, how, least):
    piece, at = _pieces(row)
    f = m.shape[1]
    part = torch.full((at.numel(), f), least, dtype=m.dtype, device=DEV)
    part.scatter_reduce_(0, piece[:, None].expand(-1, f), m, how)
    out.scatter_reduce_(0, at[:, None].expand(-1, f), part, how)


def _sum64(row, col, w, x, n):
    """sum of w * x[col] per row (the message rounded to fp32 where it is weighted)."""
    out = torch.zeros(n, x.shape[1], dtype=torch.float64, device=DEV)
    step = max(1, CHUNK // x.shape[1])
    for p in range(0, row.numel(), step):
        m = x[col[p:p + step].long()]
        m = m.double() if w is None else m.float().mul_(w[p:p + step, None]).double()
        _add_rows(out, row[p:p + step], m)
    return out


def _max64(row, col, w, x, n, sign=1):
    """Largest (sign 1) or smallest (sign -1) message per row and its first position."""
    f = x.shape[1]
    best = torch.full((n, f), -math.inf, dtype=torch.float32, device=DEV)
    arg = torch.full((n, f), 2 ** 31 - 1, dtype=torch.int32, device=DEV)
    step = max(1, CHUNK // (4 * f))
    for what in (0, 1):
        for p in range(0, row.numel(), step):
            r = row[p:p + step].long()
            m = x[col[p:p + step].long()].float() * sign
            if w is not None:
                m *= w[p:p + step, None]
            if what == 0:
                _best_rows(best, row[p:p + step], m, "amax", -math.inf)
            else:
                pos = torch.arange(p, p + r.numel(), dtype=torch.int32, device=DEV)[:, None]
                pos = torch.where(m == best[r], pos, torch.tensor(2 ** 31 - 1, dtype=torch.int32, device=DEV))
                _best_rows(arg, row[p:p + step], pos, "amin", 2 ** 31 - 1)
    empty = torch.isinf(best)
    best = torch.where(empty, 0.0, best.double() * sign)
    return best, torch.where(empty, -1, arg)


def _var64(row, col, x, n, mean):
    out = torch.zeros(n, x.shape[1], dtype=torch.float64, device=DEV)
    step = max(1, CHUNK // x.shape[1])
    for p in range(0, row.numel(), step):
        r = row[p:p + step].long()
        m = x[col[p:p + step].long()].double()
        _add_rows(out, row[p:p + step], (m - mean[r]).square_())
    return out


def _stats64(row, col, x, n, names):
    deg = torch.bincount(row, minlength=n).clamp_(min=1).double()[:, None]
    total = _sum64(row, col, None, x, n)
    res = {}
    for a in names:
        if a == "sum":
            res[a] = total
        elif a == "mean":
            res[a] = total / deg
        elif a == "std":
            res[a] = (_var64(row, col, x, n, total / deg) / deg).sqrt()
        else:
            res[a], res["arg" + a] = _max64(row, col, None, x, n, 1 if a == "max" else -1)
    return res


def exact(c, seed):
    k = c["kind"]
    if c.get("e", 0) * c.get("f", 0) > 1.5e10:
        return None
    if k == "index":
        src, dst = _graph(c, seed)
        rowptr, col, order, key = _csr64(dst, c["n"], src)
        rowptrT, colT, posT, _ = _csr64(col, c["n"], key)
        return {"rowptr": rowptr, "col": col, "perm": order, "rowptrT": rowptrT, "colT": colT,
                "posT": posT}
    if k in ("layer", "minibatch", "train", "stacked", "explain"):
        n = c["n"]
        src, dst = _graph(c, seed)
        w = _gcn_weights(src, dst, n) if k == "minibatch" else _weights(c, seed, src, dst)
        rowptr, col, order, row = _csr64(dst, n, src)
        w = None if w is None else w[order]
        x = _normal(seed, 4, (n, c["f"]), c["dtype"])
        deg = (rowptr[1:] - rowptr[:-1]).clamp(min=1).double()[:, None]
        del src, dst
    if k == "layer":
        red = REDUCE[c["reduce"]]
        res = {"out": None, "max": None, "arg": None}
        if red & (mp.MP_SUM | mp.MP_MEAN):
            res["out"] = _sum64(row, col, w, x, n)
            if red & mp.MP_MEAN:
                res["out"] /= deg
        if red & mp.MP_MAX:
            res["max"], res["arg"] = _max64(row, col, w, x, n)
        return res
    if k == "minibatch":
        return {"rowptr": rowptr, "col": col, "w": w.double(), "out": _sum64(row, col, w, x, n)}
    if k == "train":
        g = _normal(seed, 6, (n, c["f"])).double()
        res = {"out": None, "arg": None, "gx": None, "gw": None}
        if c["reduce"] == "max":
            res["out"], res["arg"] = _max64(row, col, w, x, n)
            hit = res["arg"] >= 0
            arg = res["arg"].clamp(min=0).long()
            v = torch.where(hit, g, 0.0)
            if w is not None:
                res["gw"] = torch.zeros(c["e"], dtype=torch.float64, device=DEV)
                f = torch.arange(c["f"], device=DEV)[None, :].expand_as(arg)
                res["gw"].index_add_(0, arg.reshape(-1),
                                     (v * x[col[arg].long(), f].double()).reshape(-1))
                v = v * w[arg].double()
            res["gx"] = torch.zeros(n, c["f"], dtype=torch.float64, device=DEV)
            res["gx"].scatter_add_(0, col[arg].long(), v)
            return res
        res["out"] = _sum64(row, col, w, x, n)
        if c["reduce"] == "mean":
            res["out"] /= deg
            g = g / deg
        gx = torch.zeros(n, c["f"], dtype=torch.float64, device=DEV)
        gw = None if w is None else torch.zeros(c["e"], dtype=torch.float64, device=DEV)
        step = max(1, CHUNK // c["f"])
        for p in range(0, c["e"], step):
            q = slice(p, p + step)
            m = g[row[q].long()]
            if gw is not None:
                gw[q] = (m * x[col[q].long()].double()).sum(1)
                m = m * w[q, None].double()
            gx.index_add_(0, col[q].long(), m)
        res["gx"], res["gw"] = gx, gw
        return res
    if k == "stacked":
        return _stats64(row, col, x, n, STATS)
    if k == "hetero":
        npt = _typed_sizes(c)
        offs = [0, npt[0], npt[0] + npt[1]]
        rels = _relations(c, seed)
        src = torch.cat([a + offs[s] for s, _, a, _ in rels])
        dst = torch.cat([b + offs[d] for _, d, _, b in rels])
        rowptr, col, _, row = _csr64(dst, sum(npt), src)
        x = torch.cat([_normal(seed, 30 + t, (n, c["f"]), c["dtype"]) for t, n in enumerate(npt)])
        return {"rowptr": rowptr, "col": col, "out": _sum64(row, col, None, x, sum(npt))}
    if k == "readout":
        row = _segments(c, seed)
        col = torch.arange(c["n"], dtype=torch.int32, device=DEV)
        return _stats64(row, col, _normal(seed, 4, (c["n"], c["f"]), c["dtype"]), c["graphs"], READOUT)
    if k == "projection":
        n, f, fo = sum(_typed_sizes(c)), c["f"], c["fo"]
        seg = [0, c["na"], c["na"] + c["nb"], n]
        x = _normal(seed, 4, (n, f), "bf16")
        W = (_normal(seed, 7, (3, f, fo)) / math.sqrt(f)).to(torch.bfloat16).double()
        g = _normal(seed, 6, (n, fo), "bf16")
        out = torch.empty(n, fo, dtype=torch.float64, device=DEV)
        dx = torch.empty(n, f, dtype=torch.float64, device=DEV)
        dW = torch.zeros(3, f, fo, dtype=torch.float64, device=DEV)
        step = max(1, CHUNK // max(f, fo))
        for t in range(3):
            for p in range(seg[t], seg[t + 1], step):
                q = slice(p, min(p + step, seg[t + 1]))
                xd, gd = x[q].double(), g[q].double()
                out[q] = xd @ W[t]
                dx[q] = gd @ W[t].T
                dW[t] += xd.T @ gd
        return {"out": out, "dx": dx, "dW": dW}
    # explain
    g = _normal(seed, 6, (n, c["f"])).double()
    mask = torch.sigmoid(_normal(seed, 8, (c["e"],)))[order].double()
    out = torch.zeros(n, c["f"], dtype=torch.float64, device=DEV)
    gx = torch.zeros_like(out)
    gm = torch.zeros(c["e"], dtype=torch.float64, device=DEV)
    step = max(1, CHUNK // c["f"])
    for p in range(0, c["e"], step):
        q = slice(p, p + step)
        m, d = x[col[q].long()].double(), g[row[q].long()]
        _add_rows(out, row[q], m * mask[q, None])
        gm[order[q]] = (m * d).sum(1)
        gx.index_add_(0, col[q].long(), d * mask[q, None])
    return {"out": out, "gmask": gm, "gx": gx}
