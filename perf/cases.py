"""The work that programs have this library do, as cases to time and compare.

Every case is one pass through the public entry points as a program calls
them. `listed()` holds the standing cases, `draw(rng)` another case of the same
kinds over their whole ranges, `prepare` what a program holds before the call
(inputs, the graph's CSR where a program builds it once), `run` one pass,
`exact` the same outputs in 64 bits by plain torch, `work` the bytes and
operations a pass cannot do without and `tolerance` what two correct
implementations may differ by.

Kinds:
  gcn_sum       pyg_gcn_propagate on a prepared CSR (a GCN operator whose
                normalisation is not kept)
  layer         X Theta on the matrix cores, then the propagate weighted by
                the graph's kept GCN norms (a GCN layer's forward)
  step          a graph seen for the first time: source-blocked CSR, degree,
                GCN propagate, whole-graph mean pool
  minibatch     small graphs batched together, new in every step: CSR, mean
                propagate, max pool per graph
  edgeconv      difference messages under max, forward and backward
  gat           attention coefficients and sum, forward and backward
  weighted      weighted propagate (sum, mean), forward and backward with the
                gradient of the weights
  edge          messages with F-dimensional edge features, forward and backward
  coo           propagate straight from an edge list (a graph used once)
  graph         the preparation of a graph for training: CSR, reversed CSR,
                transpose map
"""
from __future__ import annotations

import math

import torch

import paper_1903_02428_amd as pyg

# large power-law graph of the benchmark: 232,965 nodes, 114,832,965 edges
_BIG_N, _BIG_E = 232_965, 114_600_000 + 232_965


def listed():
    return [
        # latency: a GCN operator on a citation-sized graph (2,708 nodes)
        {"name": "gcn_sum_small_f32", "kind": "gcn_sum", "graph": "uniform", "N": 2708, "E": 10556 + 2708, "F": 16,
         "dtype": "f32"},
        # a citation graph with wide input features (500 -> 64), kept norms
        {"name": "layer_medium_f32", "kind": "layer", "graph": "power", "N": 19717, "E": 88648 + 19717, "Fi": 500,
         "F": 64, "dtype": "f32"},
        # the largest graph in bf16: a GCN layer's forward in inference
        {"name": "layer_large_bf16", "kind": "layer", "graph": "power", "N": _BIG_N, "E": _BIG_E, "Fi": 128, "F": 128,
         "dtype": "bf16"},
        # the benchmark's step: everything a new large graph needs, fp32
        {"name": "step_large_f32", "kind": "step", "graph": "power", "N": _BIG_N, "E": _BIG_E, "F": 128, "B": 2,
         "dtype": "f32"},
        # training on small graphs: every step batches other graphs
        {"name": "minibatch_f32", "kind": "minibatch", "graph": "batch", "graphs": 128, "F": 64, "dtype": "f32"},
        # point clouds: 16 clouds of 1,024 points, 16 neighbours, training
        {"name": "edgeconv_train_f32", "kind": "edgeconv", "graph": "knn", "clouds": 16, "points": 1024, "k": 16,
         "F": 64, "dtype": "f32"},
        # attention layer's training on a citation graph, 8 heads of 8
        {"name": "gat_train_medium_f32", "kind": "gat", "graph": "power", "N": 19717, "E": 88648 + 19717, "H": 8,
         "C": 8, "dtype": "f32"},
        # the same on the largest graph, 8 heads of 16
        {"name": "gat_train_large_f32", "kind": "gat", "graph": "power", "N": _BIG_N, "E": _BIG_E, "H": 8, "C": 16,
         "dtype": "f32"},
        # learned edge weights on a middle-sized graph, rows of 100 features
        # (16-byte rows, no whole number of cache lines)
        {"name": "weighted_train_f32", "kind": "weighted", "graph": "power", "N": 100_000, "E": 2_000_000, "F": 100,
         "aggr": "sum", "dtype": "f32"},
        # bond or relation features in bf16, training
        {"name": "edge_train_bf16", "kind": "edge", "graph": "power", "N": 100_000, "E": 2_000_000, "F": 64,
         "msg": "edge_relu", "aggr": "sum", "dtype": "bf16"},
        # an edge list used once, no CSR kept
        {"name": "coo_sum_f32", "kind": "coo", "graph": "uniform", "N": 16384, "E": 262_144, "F": 64, "aggr": "sum",
         "dtype": "f32"},
        # preparing a million-node weighted graph for training
        {"name": "graph_build_f32", "kind": "graph", "graph": "power", "N": 1_000_000, "E": 16_000_000, "F": 1,
         "dtype": "f32"},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["gcn_sum", "layer", "step", "minibatch", "edgeconv", "gat", "weighted", "edge", "coo", "graph"])
    dtype = rng.choice(["f32", "f32", "bf16"])
    N = _log(rng, 1000, 1_000_000)
    deg = math.exp(rng.uniform(math.log(2.0), math.log(256.0)))
    if kind == "minibatch":
        return {"kind": kind, "graph": "batch", "graphs": _log(rng, 16, 2048), "F": rng.choice([16, 37, 64, 100, 128]),
                "dtype": dtype}
    if kind == "edgeconv":
        return {"kind": kind, "graph": "knn", "clouds": _log(rng, 2, 48), "points": rng.choice([256, 777, 1024, 2048]),
                "k": rng.choice([8, 16, 20, 32]), "F": rng.choice([3, 32, 64, 100, 128]), "dtype": dtype}
    graph = rng.choice(["power", "uniform"])
    F = rng.choice([8, 16, 33, 64, 100, 128, 256])
    # edges times features stay below a fifth of the largest listed case
    E = min(int(N * deg) + N, 40_000_000, 3_000_000_000 // F)
    E = max(E, 2 * N)
    c = {"kind": kind, "graph": graph, "N": N, "E": E, "F": F, "dtype": dtype}
    if kind == "layer":
        c["Fi"] = rng.choice([64, 128, 300, 500, 602])
    elif kind == "step":
        c["F"] = rng.choice([16, 64, 128, 200])
        c["E"] = max(2 * N, min(E, 3_000_000_000 // c["F"]))
        c["B"] = rng.choice([2, 2, 4])
    elif kind == "gat":
        c["H"] = rng.choice([1, 2, 3, 4, 8])
        c["C"] = rng.choice([8, 16, 25, 32])
        c["E"] = max(2 * N, min(E, 1_500_000_000 // (c["H"] * c["C"])))
        del c["F"]
    elif kind == "weighted":
        c["aggr"] = rng.choice(["sum", "mean"])
        c["E"] = max(2 * N, min(E, 1_500_000_000 // F))
    elif kind == "edge":
        c["F"] = rng.choice([16, 33, 64, 128])
        c["E"] = min(E, 800_000_000 // c["F"])
        c["N"] = min(N, c["E"] // 2)
        c["msg"] = rng.choice(["edge_add", "edge_relu", "edge_mul"])
        c["aggr"] = rng.choice(["sum", "mean"])
    elif kind == "coo":
        c["aggr"] = rng.choice(["sum", "mean", "max"])
        c["E"] = min(E, 4_000_000, 256_000_000 // F)
        c["N"] = min(N, c["E"] // 2)
    elif kind == "graph":
        c["F"] = 1
        c["dtype"] = "f32"
    return c


# ------------------------------------------------------------------- inputs

_T = {"f32": torch.float32, "bf16": torch.bfloat16}
_DEV = "cuda"


def _gen(seed):
    g = torch.Generator(device=_DEV)
    g.manual_seed(seed)
    return g


def _power_endpoints(N, M, g):
    """M endpoints drawn by Chung-Lu weights (exponent 2.1, expected degrees
    capped at the square root of their total)."""
    total = 2.0 * M
    base = torch.arange(1, N + 1, dtype=torch.float64) ** (-1.0 / 1.1)
    cap = math.sqrt(total)
    lo, hi = 0.0, total
    for _ in range(60):
        c = 0.5 * (lo + hi)
        if float(torch.clamp(c * base, max=cap).sum()) < total:
            lo = c
        else:
            hi = c
    w = torch.cumsum(torch.clamp(hi * base, max=cap), 0).to(_DEV)
    u = torch.rand(2, M, generator=g, device=_DEV, dtype=torch.float64) * w[-1]
    return torch.searchsorted(w, u).clamp_(max=N - 1)


def _edges(case, g):
    """edge_index [2, E] (int64, edges in random order) of the case's graph:
    undirected pairs in both directions plus self-loops."""
    N, E = _sizes(case)
    if case["graph"] == "knn":
        P, k = case["points"], min(case["k"], case["points"] - 1)
        pts = torch.randn(case["clouds"], P, 3, generator=g, device=_DEV)
        d = torch.cdist(pts, pts)
        d.diagonal(dim1=1, dim2=2).fill_(math.inf)
        near = d.topk(k, dim=2, largest=False).indices
        base = torch.arange(case["clouds"], device=_DEV).view(-1, 1, 1) * P
        src = (near + base).reshape(-1)
        dst = torch.arange(N, device=_DEV).repeat_interleave(k)
        return torch.stack([src, dst]).contiguous(), None
    if case["graph"] == "batch":
        sizes = _batch_sizes(case)[torch.randperm(case["graphs"], generator=torch.Generator().manual_seed(
            int(torch.randint(0, 2 ** 31, (1,), generator=g, device=_DEV))))].to(_DEV)
        batch = torch.repeat_interleave(torch.arange(case["graphs"], device=_DEV), sizes)
        start = torch.cumsum(sizes, 0) - sizes
        u = torch.randint(0, N, (E // 2,), generator=g, device=_DEV)
        n = sizes[batch[u]]
        hop = 1 + (torch.rand(E // 2, generator=g, device=_DEV, dtype=torch.float64) * (n - 1)).long()
        s = start[batch[u]]
        v = s + (u - s + hop) % n
        ei = torch.stack([torch.cat([u, v]), torch.cat([v, u])])
        return ei.contiguous(), batch
    M = (E - N) // 2
    loops = E - 2 * M
    if case["graph"] == "uniform":
        u, v = torch.randint(0, N, (2, M), generator=g, device=_DEV)
    else:
        u, v = _power_endpoints(N, M, g)
        relabel = torch.randperm(N, generator=g, device=_DEV)
        u, v = relabel[u], relabel[v]
    loop = torch.arange(loops, device=_DEV) % N
    order = torch.randperm(E, generator=g, device=_DEV)
    ei = torch.empty(2, E, dtype=torch.int64, device=_DEV)
    ei[0] = torch.cat([u, v, loop])[order]
    ei[1] = torch.cat([v, u, loop])[order]
    return ei, None


def _batch_sizes(case):
    """Graph sizes of 10 to 40 nodes, evenly spread."""
    return torch.linspace(10, 40, case["graphs"]).round().long()


def _sizes(case):
    if case["graph"] == "knn":
        n = case["clouds"] * case["points"]
        return n, n * min(case["k"], case["points"] - 1)
    if case["graph"] == "batch":
        n = int(_batch_sizes(case).sum())
        return n, 2 * round(n * 2.2)
    return case["N"], case["E"]


def _normal(g, shape, dtype=torch.float32, scale=1.0):
    return (torch.randn(*shape, generator=g, device=_DEV) * scale).to(dtype)


def _inputs(case, seed):
    """The seed's tensors: what `prepare` and `exact` both start from."""
    g = _gen(seed)
    N, E = _sizes(case)
    ei, batch = _edges(case, g)
    t = _T[case["dtype"]]
    d = {"N": N, "E": E, "ei": ei, "batch": batch}
    kind = case["kind"]
    if kind == "layer":
        d["x"] = _normal(g, (N, case["Fi"]), t)
        d["theta"] = _normal(g, (case["Fi"], case["F"]), t, case["Fi"] ** -0.5)
    elif kind == "gat":
        HC = case["H"] * case["C"]
        d["x"] = _normal(g, (N, HC), t)
        d["a_src"], d["a_dst"] = _normal(g, (N, case["H"])), _normal(g, (N, case["H"]))
        d["grad"] = _normal(g, (N, HC), t)
    elif kind == "graph":
        d["w"] = torch.rand(E, generator=g, device=_DEV) + 0.05
    else:
        d["x"] = _normal(g, (N, case["F"]), t)
    if kind in ("edgeconv", "weighted", "edge"):
        d["grad"] = _normal(g, (N, case["F"]), t)
    if kind == "weighted":
        d["w"] = torch.rand(E, generator=g, device=_DEV) + 0.05
    if kind == "edge":
        d["ea"] = _normal(g, (E, case["F"]), t)
    return d


def prepare(case, seed):
    d = _inputs(case, seed)
    kind, ei, N = case["kind"], d["ei"], d["N"]
    d["case"] = case
    if kind == "gcn_sum":
        d["csr"] = pyg.coo_to_csr(ei, N)
        del d["ei"]
    elif kind == "step":
        d["batch"] = torch.zeros(N, dtype=torch.int64, device=_DEV)  # one graph
    elif kind == "layer":
        csr = pyg.coo_to_csr(ei, N)
        csr.weight = pyg.gcn_norm_csr(csr)
        d["csr"] = csr
        del d["ei"]
    elif kind in ("edgeconv", "gat", "weighted", "edge"):
        d["graph"] = pyg.Graph(ei, N)
        if kind == "gat":
            d["graph"].map_t  # made once per graph
        for name in ("x", "a_src", "a_dst", "w", "ea"):
            if name in d:
                d[name].requires_grad_(True)
    return d


# --------------------------------------------------------------------- pass

def run(state):
    case = state["case"]
    kind = case["kind"]
    if kind == "gcn_sum":
        return pyg.gcn_propagate(state["x"], state["csr"])
    if kind == "layer":
        h = pyg.dense_transform(state["x"], state["theta"], out_dtype=state["x"].dtype)
        return pyg.propagate(h, csr=state["csr"], aggr="sum")[0]
    if kind == "step":
        bcsr = pyg.coo_to_csr_blocked(state["ei"], state["N"], case["B"])
        deg = pyg.degree_csr_blocks(bcsr)
        out = pyg.gcn_propagate_blocked(state["x"], None, bcsr)
        pool, _ = pyg.global_pool(out, state["batch"], 1, "mean")
        return {"rowptr": bcsr.rowptr, "col": bcsr.col, "deg": deg, "out": out, "pool": pool}
    if kind == "minibatch":
        csr = pyg.coo_to_csr(state["ei"], state["N"])
        h, _ = pyg.propagate(state["x"], csr=csr, aggr="mean")
        pool, arg = pyg.global_pool(h, state["batch"], case["graphs"], "max")
        return {"h": h, "pool": pool, "arg": arg}
    if kind == "edgeconv":
        out = pyg.Propagate.apply(state["x"], None, state["graph"], "max", "diff")
        (gx,) = torch.autograd.grad(out, [state["x"]], state["grad"])
        return {"out": out, "grad_x": gx}
    if kind == "gat":
        out = pyg.GATAttention.apply(state["x"], state["a_src"], state["a_dst"], state["graph"], 0.2)
        gx, gs, gd = torch.autograd.grad(out, [state["x"], state["a_src"], state["a_dst"]], state["grad"])
        return {"out": out, "grad_x": gx, "grad_src": gs, "grad_dst": gd}
    if kind == "weighted":
        out = pyg.Propagate.apply(state["x"], state["w"], state["graph"], case["aggr"], "src")
        gx, gw = torch.autograd.grad(out, [state["x"], state["w"]], state["grad"])
        return {"out": out, "grad_x": gx, "grad_w": gw}
    if kind == "edge":
        out = pyg.PropagateEdge.apply(state["x"], state["ea"], state["graph"], case["msg"], case["aggr"])
        gx, ge = torch.autograd.grad(out, [state["x"], state["ea"]], state["grad"])
        return {"out": out, "grad_x": gx, "grad_e": ge}
    if kind == "coo":
        out, arg = pyg.propagate(state["x"], state["ei"], aggr=case["aggr"])
        return {"out": out} if arg is None else {"out": out, "arg": arg}
    g = pyg.Graph(state["ei"], state["N"], state["w"])
    return {"rowptr": g.csr.rowptr, "col": g.csr.col, "perm": g.csr.perm, "w": g.csr.weight, "rowptr_t": g.csr_t.rowptr,
            "col_t": g.csr_t.col, "perm_t": g.csr_t.perm, "w_t": g.csr_t.weight, "map_t": g.map_t}


# -------------------------------------------------------------------- floor

def work(case):
    """Every input read once, every output written once; one multiply-add per
    edge and feature and direction."""
    N, E = _sizes(case)
    s = 2 if case["dtype"] == "bf16" else 4
    kind = case["kind"]
    F = case["H"] * case["C"] if kind == "gat" else case["F"]
    csr = 8 * (N + 1) + 4 * E
    if kind == "gcn_sum":
        return {"bytes": csr + 2 * N * F * s, "flops": 2 * E * F}
    if kind == "layer":
        Fi = case["Fi"]
        return {"bytes": csr + 4 * E + N * Fi * s + Fi * F * s + N * F * s, "flops": 2 * E * F + 2 * N * Fi * F}
    if kind == "step":
        return {"bytes": 16 * E + 8 * (case["B"] * N + 1) + 4 * E + 16 * N + 2 * N * F * s + F * s, "flops": 2 * E * F}
    if kind == "minibatch":
        G = case["graphs"]
        return {"bytes": 16 * E + 2 * N * F * s + 8 * N + G * F * (s + 8), "flops": E * F + N * F}
    if kind == "edgeconv":
        return {"bytes": csr + 8 * E + 4 * N * F * s, "flops": 3 * E * F}
    if kind == "gat":
        H = case["H"]
        return {"bytes": 2 * csr + 4 * N * F * s + 4 * N * H * 4, "flops": 6 * E * F + 12 * E * H}
    if kind == "weighted":
        return {"bytes": 2 * csr + 16 * E + 8 * E + 4 * N * F * s, "flops": 6 * E * F}
    if kind == "edge":
        return {"bytes": 2 * csr + 16 * E + 2 * E * F * s + 4 * N * F * s, "flops": 6 * E * F}
    if kind == "coo":
        return {"bytes": 16 * E + 2 * N * F * s + (8 * N * F if case["aggr"] == "max" else 0), "flops": E * F}
    return {"bytes": 16 * E + 4 * E + 2 * (8 * (N + 1) + 16 * E) + 4 * E, "flops": 0}


def tolerance(case):
    kind = case["kind"]
    if kind == "graph":
        return "exact"
    if kind == "coo" and case["aggr"] == "max":
        return "exact"
    if case["dtype"] == "bf16":  # one rounding is up to 2.3e-3 from 64 bits (two in a layer)
        return {"rel": 1e-2, "max": 0.05, "differ": 0.01}
    # up to 4.8e-7 from 64 bits (the logits' gradients, the 500-term products)
    return {"rel": 2e-6, "max": 2e-4, "differ": 1e-3}


# ----------------------------------------------------------------- 64 bits

_CHUNK = 1 << 29  # bytes of one gathered block of rows in 64 bits


def _blocks(E, F):
    step = max(1, _CHUNK // (8 * max(F, 1)))
    return [slice(a, min(E, a + step)) for a in range(0, E, step)]


def _scatter(N, F, dst, msg):
    """sum over edges of msg(slice) [n, F] into dst, in 64 bits."""
    out = torch.zeros(N, F, dtype=torch.float64, device=_DEV)
    for b in _blocks(dst.numel(), F):
        out.index_add_(0, dst[b], msg(b))
    return out


def _degree(dst, N):
    return torch.bincount(dst, minlength=N).double()


def _max_edge(x, src, dst, N, diff):
    """Max over incoming edges of the fp32 messages and the first edge that
    reaches it (E for none)."""
    E, F = src.numel(), x.shape[1]
    top = torch.full((N, F), -math.inf, device=_DEV)
    first = torch.full((N, F), E, dtype=torch.int64, device=_DEV)

    def msg(b):
        m = x[src[b]].float()
        return (m - x[dst[b]].float() if diff else m) + 0.0
    for b in _blocks(E, 2 * F):
        top.scatter_reduce_(0, dst[b].view(-1, 1).expand(-1, F), msg(b), "amax")
    for b in _blocks(E, 2 * F):
        k = torch.arange(b.start, b.stop, device=_DEV).view(-1, 1)
        k = torch.where(msg(b) == top[dst[b]], k, E)
        first.scatter_reduce_(0, dst[b].view(-1, 1).expand(-1, F), k, "amin")
    return torch.where(first < E, top, 0.0).double(), first


def exact(case, seed):
    d = _inputs(case, seed)
    kind, N, E = case["kind"], d["N"], d["E"]
    src, dst = d["ei"]
    if kind == "graph":
        return None
    x = d["x"]
    F = x.shape[1]
    x64 = x.double()
    if kind in ("gcn_sum", "step"):
        di = _degree(dst, N)
        di = torch.where(di > 0, di.rsqrt(), 0.0).view(-1, 1)
        xs = x64 * di
        out = _scatter(N, F, dst, lambda b: xs[src[b]]) * di
        if kind == "gcn_sum":
            return out
        return {"rowptr": None, "col": None, "deg": None, "out": out, "pool": out.mean(0, keepdim=True)}
    if kind == "layer":
        h = x64 @ d["theta"].double()
        di = _degree(dst, N).rsqrt().view(-1, 1)
        hs = torch.where(di.isfinite(), h * di, 0.0)
        out = _scatter(N, h.shape[1], dst, lambda b: hs[src[b]]) * di
        return torch.where(di.isfinite(), out, 0.0)
    if kind == "minibatch":
        h = _scatter(N, F, dst, lambda b: x64[src[b]]) / _degree(dst, N).clamp(min=1).view(-1, 1)
        pool = torch.full((case["graphs"], F), -math.inf, dtype=torch.float64, device=_DEV)
        pool.scatter_reduce_(0, d["batch"].view(-1, 1).expand(-1, F), h, "amax")
        return {"h": h, "pool": pool, "arg": None}
    if kind == "coo":
        if case["aggr"] == "max":
            out, first = _max_edge(x, src, dst, N, False)
            return {"out": out, "arg": None}
        out = _scatter(N, F, dst, lambda b: x64[src[b]])
        return {"out": out if case["aggr"] == "sum" else out / _degree(dst, N).clamp(min=1).view(-1, 1)}
    g64 = d["grad"].double()
    if kind == "edgeconv":
        out, first = _max_edge(x, src, dst, N, True)
        hit = first < E
        gv = torch.where(hit, g64, 0.0)
        cols = torch.arange(F, device=_DEV).expand(N, F)
        gx = -gv
        at = src[first.clamp(max=E - 1)]
        gx.reshape(-1).scatter_add_(0, (at * F + cols).reshape(-1), gv.reshape(-1))
        return {"out": out, "grad_x": gx}
    if kind == "weighted":
        w = d["w"].double().view(-1, 1)
        sc = 1.0 / _degree(dst, N).clamp(min=1).view(-1, 1) if case["aggr"] == "mean" else torch.ones(N, 1, device=_DEV)
        gs = g64 * sc
        out = _scatter(N, F, dst, lambda b: x64[src[b]] * w[b]) * sc
        gx = _scatter(N, F, src, lambda b: gs[dst[b]] * w[b])
        gw = torch.cat([(gs[dst[b]] * x64[src[b]]).sum(1) for b in _blocks(E, F)])
        return {"out": out, "grad_x": gx, "grad_w": gw}
    if kind == "edge":
        ea, how = d["ea"], case["msg"]
        sc = 1.0 / _degree(dst, N).clamp(min=1).view(-1, 1) if case["aggr"] == "mean" else torch.ones(N, 1, device=_DEV)
        gs = g64 * sc

        def msg(b):
            m = x64[src[b]]
            e = ea[b].double()
            return m * e if how == "edge_mul" else (m + e).clamp(min=0) if how == "edge_relu" else m + e

        def grads(b):
            dk = gs[dst[b]]
            if how == "edge_mul":
                return dk * ea[b].double(), dk * x64[src[b]]
            if how == "edge_relu":
                dk = torch.where(x64[src[b]] + ea[b].double() > 0, dk, 0.0)
            return dk, dk
        out = _scatter(N, F, dst, msg) * sc
        gx = _scatter(N, F, src, lambda b: grads(b)[0])
        ge = torch.cat([grads(b)[1] for b in _blocks(E, F)])
        return {"out": out, "grad_x": gx, "grad_e": ge}
    # gat
    H, C = case["H"], case["C"]
    a_s, a_d = d["a_src"].double(), d["a_dst"].double()

    def lrelu(b):
        v = a_s[src[b]] + a_d[dst[b]]
        return torch.where(v >= 0, v, 0.2 * v), torch.where(v >= 0, 1.0, 0.2)
    Z = _scatter(N, H, dst, lambda b: lrelu(b)[0].exp())

    def alpha(b):
        return lrelu(b)[0].exp() / Z[dst[b]]

    def spread(a, rows):  # [n, H] times [n, H*C]
        return (a.unsqueeze(2) * rows.view(-1, H, C)).reshape(-1, H * C)
    out = torch.zeros(N, F, dtype=torch.float64, device=_DEV)
    gx = torch.zeros_like(out)
    t = torch.zeros(N, H, dtype=torch.float64, device=_DEV)
    blocks = _blocks(E, F)
    for b in blocks:
        al, xr, gr = alpha(b), x64[src[b]], g64[dst[b]]
        out.index_add_(0, dst[b], spread(al, xr))
        gx.index_add_(0, src[b], spread(al, gr))
        t.index_add_(0, dst[b], al * (gr * xr).view(-1, H, C).sum(2))
    gs, gd = torch.zeros_like(t), torch.zeros_like(t)
    for b in blocks:
        al = alpha(b)
        ga = (g64[dst[b]] * x64[src[b]]).view(-1, H, C).sum(2)
        dv = al * (ga - t[dst[b]]) * lrelu(b)[1]
        gs.index_add_(0, src[b], dv)
        gd.index_add_(0, dst[b], dv)
    return {"out": out, "grad_x": gx, "grad_src": gs, "grad_dst": gd}
