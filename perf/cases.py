"""Performance cases of the gnnk operators: what they are, how they run and what they should give.

The graphs are seeded stand-ins of the workloads that this repository's
generator and benchmark use (a tiny uniform multigraph, a citation-like
power-law graph, R-MAT graphs with the node and edge counts of its two large
workloads, a relational multigraph, a constant in-degree graph), drawn on the
GPU, and a sampled neighbourhood block as a mini-batch loop makes it.  Edge
lists come in two orders: "sorted" by (destination, source), as this
repository's generator writes them, and "arrival", a random order of the
edges, as an edge list read from a file has it.
"""
import math

import torch

from paper_1909_01315_amd import gnnk, nn

SLOPE = 0.2
DTYPES = {"f32": torch.float32, "bf16": torch.bfloat16}

# the two R-MAT workloads: nodes, edges, levels
LARGE_N, LARGE_E = 232965, 114600000
PRODUCTS_N, PRODUCTS_E = 2449029, 61859140


def listed():
    return [
        # a training step of one aggregation on a tiny graph: launches and host time are all there is
        {"name": "tiny_gcn_step", "op": "gcn", "dir": "step", "graph": "uniform", "order": "sorted", "n_src": 1024,
         "n_dst": 1024, "e": 17408, "heads": 1, "feat": 16, "dtype": "f32", "ptr64": False},
        # inference of a hidden layer on a citation graph
        {"name": "citation_gcn_fwd", "op": "gcn", "dir": "fwd", "graph": "chunglu", "order": "sorted", "n_src": 20000,
         "n_dst": 20000, "e": 109170, "heads": 1, "feat": 256, "dtype": "f32", "ptr64": False},
        # a training step of the fused attention layer on a citation graph as it came from its file
        {"name": "citation_gat_step", "op": "gat_fused", "dir": "step", "graph": "chunglu", "order": "arrival",
         "n_src": 20000, "n_dst": 20000, "e": 109170, "heads": 8, "feat": 8, "dtype": "f32", "ptr64": False},
        # one layer of a mini-batch: the sampled block's graph is built, then aggregated
        {"name": "minibatch_sage", "op": "block_mean", "dir": "fwd", "graph": "block", "order": "sorted",
         "n_src": 90000, "n_dst": 10000, "e": 100000, "heads": 1, "feat": 100, "dtype": "f32", "ptr64": False},
        # relational layer: every (relation, source) row of the transformed table, both gradients
        {"name": "rgcn_step", "op": "rgcn", "dir": "step", "graph": "relational", "order": "sorted",
         "n_src": 5000000, "n_dst": 100000, "e": 2000000, "heads": 1, "feat": 64, "dtype": "f32", "ptr64": False},
        # the attention layer of the large graph as four operators and their gradients, the largest case
        {"name": "large_gat_step", "op": "gat", "dir": "step", "graph": "rmat", "order": "sorted", "n_src": LARGE_N,
         "n_dst": LARGE_N, "e": LARGE_E, "heads": 8, "feat": 16, "dtype": "f32", "ptr64": False},
        # the two headline operators of the benchmark
        {"name": "large_u_mul_e_fwd", "op": "attn_sum", "dir": "fwd", "graph": "rmat", "order": "sorted",
         "n_src": LARGE_N, "n_dst": LARGE_N, "e": LARGE_E, "heads": 8, "feat": 16, "dtype": "f32", "ptr64": False},
        {"name": "large_u_dot_v_fwd", "op": "dot", "dir": "fwd", "graph": "rmat", "order": "sorted",
         "n_src": LARGE_N, "n_dst": LARGE_N, "e": LARGE_E, "heads": 8, "feat": 16, "dtype": "f32", "ptr64": False},
        # the fused attention layer, trained on the large graph with edges in arrival order
        {"name": "large_gat_fused_step", "op": "gat_fused", "dir": "step", "graph": "rmat", "order": "arrival",
         "n_src": LARGE_N, "n_dst": LARGE_N, "e": LARGE_E, "heads": 8, "feat": 16, "dtype": "f32", "ptr64": False},
        # mean aggregation of input features, trained, on a very large graph in arrival order
        {"name": "products_sage_step", "op": "mean", "dir": "step", "graph": "rmat", "order": "arrival",
         "n_src": PRODUCTS_N, "n_dst": PRODUCTS_N, "e": PRODUCTS_E, "heads": 1, "feat": 100, "dtype": "f32",
         "ptr64": True},
        # max pooling in bf16 with its argmax gradient
        {"name": "products_max_bf16_step", "op": "max", "dir": "step", "graph": "rmat", "order": "sorted",
         "n_src": PRODUCTS_N, "n_dst": PRODUCTS_N, "e": PRODUCTS_E, "heads": 1, "feat": 100, "dtype": "bf16",
         "ptr64": True},
        # an output layer: an odd number of classes, on a constant in-degree graph
        {"name": "knn_mean_odd_step", "op": "mean", "dir": "step", "graph": "knn", "order": "sorted",
         "n_src": 262144, "n_dst": 262144, "e": 8388608, "heads": 1, "feat": 47, "dtype": "f32", "ptr64": False},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """Another case: any operator, graph family, order, width (odd ones among them) and type."""
    op = rng.choice(["gcn", "gcn", "mean", "mean", "max", "dot", "attn_sum", "gat", "gat_fused", "rgcn",
                     "block_mean"])
    dtype = rng.choice(["f32", "f32", "bf16"])
    order = rng.choice(["sorted", "arrival"])
    way = rng.choice(["fwd", "step", "step"])
    heads = 1
    if op in ("gat", "gat_fused", "attn_sum", "dot"):
        heads = rng.choice([1, 2, 3, 4, 8, 8])
        feat = rng.choice([8, 16, 32, 64, rng.randint(3, 63)])
    else:
        feat = rng.choice([16, 32, 64, 100, 128, 256, 512, _log_int(rng, 9, 602), _log_int(rng, 9, 602)])
    if op == "block_mean":
        n_dst = _log_int(rng, 500, 200000)
        fan = rng.randint(5, 25)
        return {"op": op, "dir": "fwd", "graph": "block", "order": "sorted", "n_src": n_dst * (fan - 1), "n_dst": n_dst,
                "e": n_dst * fan, "heads": 1, "feat": min(feat, 256), "dtype": dtype, "ptr64": False}
    if op == "rgcn":
        n = _log_int(rng, 5000, 100000)
        rel = rng.randint(5, 50)
        return {"op": op, "dir": way, "graph": "relational", "order": order, "n_src": n * rel, "n_dst": n,
                "e": n * rng.randint(4, 30), "heads": 1, "feat": min(feat, 128), "dtype": dtype, "ptr64": False}
    kind = rng.choice(["uniform", "chunglu", "rmat", "rmat", "knn"])
    if kind == "uniform":
        n = _log_int(rng, 500, 50000)
        e = n * rng.randint(4, 40)
    elif kind == "chunglu":
        n = _log_int(rng, 3000, 200000)
        e = n + int(n * rng.uniform(2.0, 9.0))
    elif kind == "knn":
        n = _log_int(rng, 10000, 400000)
        e = n * rng.choice([8, 15, 16, 20, 32])
    else:
        n = _log_int(rng, 50000, PRODUCTS_N)
        e = min(int(n * rng.uniform(10.0, 200.0)), PRODUCTS_E)
    # no drawn case costs more than the largest listed one
    most = LARGE_E * 128 // (2 if op in ("gat", "gat_fused") else 4)
    while e * heads * feat > most:
        if feat > 16:
            feat //= 2
        else:
            heads = max(1, heads // 2)
            e = min(e, most // (heads * feat))
    return {"op": op, "dir": way, "graph": kind, "order": order, "n_src": n, "n_dst": n, "e": e, "heads": heads,
            "feat": feat, "dtype": dtype, "ptr64": rng.random() < 0.25}


# ---------------------------------------------------------------------------
# inputs


def _gen(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed))
    return g


def _exactly(keys, e, gen):
    """e of the sorted distinct keys, in order."""
    drop = torch.randperm(keys.numel(), device="cuda", generator=gen)[: keys.numel() - e]
    keep = torch.ones(keys.numel(), dtype=torch.bool, device="cuda")
    keep[drop] = False
    return keys[keep]


def _rmat_keys(n, e, gen, abc=(0.57, 0.19, 0.19)):
    """Sorted distinct keys dst * n + src of an R-MAT graph, ids at random."""
    a, b, c = abc
    levels = max(1, (n - 1).bit_length())
    relabel = torch.randperm(n, device="cuda", generator=gen)
    keys = torch.empty(0, dtype=torch.int64, device="cuda")
    want = e
    while keys.numel() < e:
        m = int(1.3 * want) + 4096
        src = torch.zeros(m, dtype=torch.int32, device="cuda")
        dst = torch.zeros(m, dtype=torch.int32, device="cuda")
        for _ in range(levels):
            r = torch.rand(m, device="cuda", generator=gen)
            src = 2 * src + (r >= a + b)
            dst = 2 * dst + (((r >= a) & (r < a + b)) | (r >= a + b + c))
        ok = (src < n) & (dst < n)
        new = relabel[dst[ok].long()] * n + relabel[src[ok].long()]
        keys = torch.unique(torch.cat([keys, new]))
        want = max(2 * (e - keys.numel()), 4096)
    return _exactly(keys, e, gen)


def _chunglu_keys(n, e, gen):
    """Sorted keys dst * n + src: power-law endpoints (exponent 2.5), no duplicates, one self-loop per node."""
    w = torch.arange(1, n + 1, device="cuda", dtype=torch.float64) ** (-1.0 / 1.5)
    cum = torch.cumsum(w, 0)
    relabel = torch.randperm(n, device="cuda", generator=gen)
    keys = torch.empty(0, dtype=torch.int64, device="cuda")
    while keys.numel() < e - n:
        m = 2 * (e - n)
        u = torch.rand((2, m), device="cuda", dtype=torch.float64, generator=gen) * cum[-1]
        ends = relabel[torch.searchsorted(cum, u).clamp_(max=n - 1)]
        new = (ends[0] * n + ends[1])[ends[0] != ends[1]]
        keys = torch.unique(torch.cat([keys, new]))
    loops = torch.arange(n, device="cuda") * (n + 1)
    return torch.sort(torch.cat([_exactly(keys, e - n, gen), loops]))[0]


def _edges(case, gen):
    """(src, dst, edge type or None) int32 on the GPU, in the case's order."""
    kind, ns, nd, e = case["graph"], case["n_src"], case["n_dst"], case["e"]
    etype = None
    if kind == "block":
        # a sampler's block: each destination's draws side by side; the
        # destinations come first among the sources
        src = torch.randint(0, ns, (e,), device="cuda", generator=gen)
        return src.int(), torch.arange(nd, device="cuda").repeat_interleave(e // nd).int(), None
    if kind == "rmat":
        keys = _rmat_keys(ns, e, gen)
    elif kind == "chunglu":
        keys = _chunglu_keys(ns, e, gen)
    elif kind == "knn":
        src = torch.randint(0, ns, (e,), device="cuda", generator=gen)
        keys = torch.sort(torch.arange(nd, device="cuda").repeat_interleave(e // nd) * ns + src)[0]
    elif kind == "uniform":
        src = torch.randint(0, ns, (e,), device="cuda", generator=gen)
        dst = torch.randint(0, nd, (e,), device="cuda", generator=gen)
        keys = torch.sort(dst * ns + src)[0]
    else:  # relational: source id = edge type * nodes + node, types from a Zipf(1.2) law
        rel = ns // nd
        p = torch.arange(1, rel + 1, device="cuda", dtype=torch.float64) ** -1.2
        cum = torch.cumsum(p, 0)
        u = torch.rand(e, device="cuda", dtype=torch.float64, generator=gen) * cum[-1]
        et = torch.searchsorted(cum, u).clamp_(max=rel - 1)
        src = et * nd + torch.randint(0, nd, (e,), device="cuda", generator=gen)
        dst = torch.randint(0, nd, (e,), device="cuda", generator=gen)
        keys = torch.sort(dst * ns + src)[0]
    if case["order"] == "arrival":
        keys = keys[torch.randperm(e, device="cuda", generator=gen)]
    src, dst = keys % ns, keys // ns
    if kind == "relational":
        etype = (src // nd).int()
    return src.int(), dst.int(), etype


def _inputs(case, seed):
    """The tensors of a case, from its seed alone."""
    gen = _gen(seed)
    dt = DTYPES[case["dtype"]]
    H, F, e, ns, nd = case["heads"], case["feat"], case["e"], case["n_src"], case["n_dst"]
    op, step = case["op"], case["dir"] == "step"
    t = {}
    t["src"], t["dst"], etype = _edges(case, gen)

    def normal(*shape):
        return torch.randn(shape, device="cuda", generator=gen).to(dt)

    if op == "gcn":
        deg_s = torch.bincount(t["src"], minlength=ns).double()
        deg_d = torch.bincount(t["dst"], minlength=nd).double()
        w = torch.rsqrt(deg_s[t["src"].long()] * deg_d[t["dst"].long()])
        t["w"] = w.to(dt).view(e, 1, 1)
    elif op == "rgcn":
        t["w"] = nn.rel_norm(etype, t["dst"], ns // nd, nd).to(dt)
    elif op == "attn_sum":
        t["w"] = torch.rand((e, H, 1), device="cuda", generator=gen).to(dt)
    if op in ("gat", "gat_fused"):
        t["el"], t["er"] = normal(ns, H, 1), normal(nd, H, 1)
    t["x"] = normal(ns, H, F)
    if op == "dot":
        t["y"] = normal(nd, H, F)
    if step:
        t["dz"] = normal(e, H, 1) if op == "dot" else normal(nd, H, F)
    return t


# the tensors whose gradients a training step of each operator asks for
GRADS = {"gcn": ["x"], "mean": ["x"], "max": ["x"], "rgcn": ["x", "w"], "attn_sum": ["x", "w"], "dot": ["x", "y"],
         "gat": ["x", "el", "er"], "gat_fused": ["x", "el", "er"]}


def prepare(case, seed):
    t = _inputs(case, seed)
    state = {"case": case, "t": t}
    if case["op"] != "block_mean":
        state["g"] = gnnk.Graph.from_coo(t.pop("src"), t.pop("dst"), case["n_src"], case["n_dst"],
                                         ptr64=case["ptr64"])
        if case["dir"] == "step":
            for name in GRADS[case["op"]]:
                t[name].requires_grad_(True)
    return state


def run(state):
    case, t, op = state["case"], state["t"], state["case"]["op"]
    if op == "block_mean":
        g = gnnk.Graph.from_coo(t["src"], t["dst"], case["n_src"], case["n_dst"])
        return {"out": gnnk.gspmm(g, "copy_lhs", "mean", t["x"])}
    g = state["g"]
    if op in ("gcn", "rgcn", "attn_sum"):
        out = nn.gspmm(g, "mul", "sum", t["x"], t["w"])
    elif op in ("mean", "max"):
        out = nn.gspmm(g, "copy_lhs", op, t["x"])
    elif op == "dot":
        out = nn.gsddmm(g, "dot", t["x"], "u", t["y"], "v")
    elif op == "gat_fused":
        out = nn.gat_aggregate(g, t["x"], t["el"], t["er"], SLOPE)
    else:
        s = nn.leaky_relu(nn.gsddmm(g, "add", t["el"], "u", t["er"], "v"), SLOPE)
        out = nn.gspmm(g, "mul", "sum", t["x"], nn.edge_softmax(g, s))
    got = {"out": out}
    if case["dir"] == "step":
        names = GRADS[op]
        for name, grad in zip(names, torch.autograd.grad(out, [t[n] for n in names], t["dz"])):
            got["d_" + name] = grad
    return got


def work(case):
    """Bytes: every input and output once, and per pass over the graph its neighbour ids and row offsets (edge ids
    too where they are not the positions).  Operations: a multiply and an add per edge and column and direction."""
    H, F, e, ns, nd, op = case["heads"], case["feat"], case["e"], case["n_src"], case["n_dst"], case["op"]
    s = 2 if case["dtype"] == "bf16" else 4
    D = H * F
    ids = 4 if case["order"] == "sorted" else 8
    fwd = e * 4 + (nd + 1) * 4
    edge_in = {"gcn": 1, "rgcn": 1, "attn_sum": H}.get(op, 0)  # values per edge read by the forward
    if edge_in:
        fwd += e * (edge_in * s + ids - 4)
    fwd += ns * D * s
    fwd += (e * H + nd * D) * s if op == "dot" else nd * D * s
    if op in ("gat", "gat_fused"):
        fwd += (ns + nd) * H * s
    if op == "gat":  # four calls: each reads and writes its own edge tensors
        fwd += 6 * e * H * s
    if op == "block_mean":
        fwd += 8 * e  # the edge list
    flops = 2.0 * e * D
    total = fwd
    if case["dir"] == "step":
        flops *= 3 if len(GRADS[op]) > 1 else 2
        bwd = e * 8 + (ns + 1) * 4
        if op == "dot":
            bwd += e * H * s + (ns + nd) * D * s * 2
        else:
            bwd += (nd + ns) * D * s + e * edge_in * s
        if op in ("rgcn", "attn_sum"):
            bwd += e * edge_in * s + ns * D * s
        if op in ("gat", "gat_fused"):
            bwd += ns * D * s + 2 * (ns + nd) * H * s
        if op == "gat":
            bwd += 10 * e * H * s
        total += bwd
    return {"bytes": float(total), "flops": float(flops)}


def tolerance(case):
    """32-bit results: sums in another order in 32 bits (measured against exact(): 2.5e-8 for sums rounded once,
    1.4e-7 for the attention gradients).  16-bit results: one rounding each (1.7e-3 measured), and in the chain of
    four operators the scores, the attention and their gradients are rounded between the steps too."""
    if case["dtype"] == "bf16":
        return {"rel": 2e-2 if case["op"] == "gat" else 8e-3}
    return {"rel": 1e-5}


# ---------------------------------------------------------------------------
# the same results in 64 bits, by plain torch


class _Rows:
    """Edges grouped by one endpoint: sums and extrema of per-edge values."""

    def __init__(self, of, n):
        self.order = torch.argsort(of, stable=True)
        self.sizes = torch.bincount(of, minlength=n)

    def reduce(self, values, how="sum", initial=0.0):
        return torch.segment_reduce(values, how, lengths=self.sizes, axis=0, initial=initial, unsafe=True)


def _spmm(rows, gather, x, w):
    """out[r, h, :] = sum over the edges of r of w[e, h] * x[gather[e], h, :]; w (E, 1 or H) or None."""
    H, F = x.shape[1], x.shape[2]
    gi = gather[rows.order]
    wp = w[rows.order] if w is not None else None
    out = torch.empty((rows.sizes.numel(), H, F), dtype=torch.float64, device="cuda")
    for h in range(H):
        for c in range(0, F, 16):
            m = x[:, h, c:c + 16].double()[gi]
            if wp is not None:
                m *= wp[:, (h if wp.shape[1] > 1 else 0)].double().unsqueeze(1)
            out[:, h, c:c + 16] = rows.reduce(m)
    return out


def _dots(src, dst, x, y):
    """out[e, h] = x[src, h, :] . y[dst, h, :]"""
    H, F = x.shape[1], x.shape[2]
    out = torch.zeros((src.numel(), H), dtype=torch.float64, device="cuda")
    for h in range(H):
        for c in range(0, F, 16):
            out[:, h] += (x[:, h, c:c + 16].double()[src] * y[:, h, c:c + 16].double()[dst]).sum(1)
    return out


def _max(rows, src, dst, x, dz):
    """Maxima over the edges of each destination and, with dz, their gradient (to the first edge of equal ones)."""
    nd, F = rows.sizes.numel(), x.shape[2]
    out = torch.empty((nd, 1, F), dtype=torch.float64, device="cuda")
    dx = torch.zeros_like(x, dtype=torch.float64) if dz is not None else None
    so, do = src[rows.order], dst[rows.order]
    none = rows.sizes == 0
    e = src.numel()
    for c in range(0, F, 10):
        m = x[:, 0, c:c + 10].double()[so]
        best = rows.reduce(m, "max", initial=-math.inf)
        if dz is not None:
            at = torch.where(m == best[do], rows.order.double().unsqueeze(1), float(e))
            first = rows.reduce(at, "min", initial=float(e)).long()
            won = torch.where(first < e, src[first.clamp(max=e - 1)], 0)
            g = torch.where(first < e, dz[:, 0, c:c + 10].double(), 0.0)
            dx[:, 0, c:c + 10] = torch.zeros_like(x[:, 0, c:c + 10], dtype=torch.float64).scatter_add_(0, won, g)
        best[none] = 0.0
        out[:, 0, c:c + 10] = best
    return out, dx


def exact(case, seed):
    t = _inputs(case, seed)
    op, step = case["op"], case["dir"] == "step"
    src, dst = t["src"].long(), t["dst"].long()
    ns, nd = case["n_src"], case["n_dst"]
    into = _Rows(dst, nd)
    outof = _Rows(src, ns) if step else None
    x, dz = t["x"], t.get("dz")
    got = {}
    if op in ("mean", "block_mean"):
        per = into.sizes.clamp(min=1).double().view(-1, 1, 1)
        got["out"] = _spmm(into, src, x, None) / per
        if step:
            got["d_x"] = _spmm(outof, dst, dz.double() / per, None)
    elif op == "max":
        got["out"], dx = _max(into, src, dst, x, dz)
        if step:
            got["d_x"] = dx
    elif op in ("gcn", "rgcn", "attn_sum"):
        w = t["w"].squeeze(2)
        got["out"] = _spmm(into, src, x, w)
        if step:
            got["d_x"] = _spmm(outof, dst, dz, w)
            if op != "gcn":
                got["d_w"] = _dots(src, dst, x, dz).unsqueeze(2)
    elif op == "dot":
        got["out"] = _dots(src, dst, x, t["y"]).unsqueeze(2)
        if step:
            got["d_x"] = _spmm(outof, dst, t["y"], dz.squeeze(2))
            got["d_y"] = _spmm(into, src, x, dz.squeeze(2))
    else:
        z = t["el"].squeeze(2).double()[src] + t["er"].squeeze(2).double()[dst]
        slope = torch.where(z > 0, 1.0, SLOPE).double()
        a = z * slope
        top = into.reduce(a[into.order], "max", initial=-math.inf)
        a = torch.exp(a - top[dst])
        a /= into.reduce(a[into.order])[dst]
        got["out"] = _spmm(into, src, x, a)
        if step:
            got["d_x"] = _spmm(outof, dst, dz, a)
            ds = a * _dots(src, dst, x, dz)
            ds -= a * into.reduce(ds[into.order])[dst]
            ds *= slope
            got["d_el"] = outof.reduce(ds[outof.order]).unsqueeze(2)
            got["d_er"] = into.reduce(ds[into.order]).unsqueeze(2)
    return got
