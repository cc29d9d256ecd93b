"""The work that programs using this framework have it do, one case each.

A case is one solve through the public entry points: new initial values in,
the run to its stop rule, the values out. The graph, the problem handle and
the device arrays of the initial values are what such a program keeps.
"""
import math

import numpy as np
import torch

from paper_1710_05785_amd import daic

DEV = "cuda"


def listed():
    return [
        # shortest paths over a small network (a service answering one source
        # at a time): every microsecond is latency
        {"name": "sssp_1k_u32", "kind": "sssp", "graph": "powerlaw", "n": 1000, "state": "u32", "sched": "all"},
        # the 10,000-vertex power-law PageRank of the paper's example, all
        # pending vertices per round and the sampled priority queue
        {"name": "pagerank_10k_f64", "kind": "pagerank", "graph": "powerlaw", "n": 10000, "state": "f64",
         "sched": "all"},
        {"name": "pagerank_10k_f64_sampled", "kind": "pagerank", "graph": "powerlaw", "n": 10000, "state": "f64",
         "sched": "sampled", "q": 0.1},
        # label propagation on the paper's log-normal graphs: weighted sums
        # with per-vertex coefficients, a ragged vertex count
        {"name": "adsorption_300k_f32", "kind": "adsorption", "graph": "lognormal", "n": 300007, "state": "f32",
         "sched": "all"},
        # connected components of a symmetrized web-like graph
        {"name": "components_262k_i32", "kind": "components", "graph": "rmat", "n": 262144, "ef": 8, "state": "i32",
         "sched": "all"},
        # shortest paths with real weights on a log-normal graph
        {"name": "sssp_500k_f64", "kind": "sssp", "graph": "lognormal", "n": 500009, "state": "f64", "sched": "all"},
        # the RMAT-20 shortest paths workload, by sampled priority
        {"name": "sssp_rmat20_u32_sampled", "kind": "sssp", "graph": "rmat", "n": 1 << 20, "ef": 16, "state": "u32",
         "sched": "sampled", "q": 0.1},
        # personalized PageRank for many seeds on several uneven graphs at once
        {"name": "ppr_batch_12x64", "kind": "ppr", "graph": "rmat", "n": 8000, "ef": 8, "graphs": 12, "rhs": 64,
         "state": "f32_kahan"},
        # learned selection (the network scores the pending vertices)
        {"name": "pagerank_rmat20_learned", "kind": "pagerank", "graph": "rmat", "n": 1 << 20, "ef": 16,
         "state": "f32_kahan", "sched": "learned", "q": 0.1},
        # large graphs by exact priority and by sweeps over id blocks
        {"name": "pagerank_rmat22_exact", "kind": "pagerank", "graph": "rmat", "n": 1 << 22, "ef": 16,
         "state": "f32_kahan", "sched": "exact", "q": 0.1},
        {"name": "pagerank_rmat22_sweep", "kind": "pagerank", "graph": "rmat", "n": 1 << 22, "ef": 16,
         "state": "f32_kahan", "sched": "sweep", "q": 0.25},
        # the headline workload: RMAT-24, all pending vertices per round
        {"name": "pagerank_rmat24_f32k", "kind": "pagerank", "graph": "rmat", "n": 1 << 24, "ef": 16,
         "state": "f32_kahan", "sched": "all"},
    ]


def _size(rng, lo, hi):
    """A size spread over the logarithm of [lo, hi], odd ones among them."""
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["pagerank", "pagerank", "pagerank", "sssp", "sssp", "components", "adsorption", "katz", "ppr"])
    graph = rng.choice(["powerlaw", "lognormal", "rmat"])
    c = {"kind": kind, "graph": graph}
    if kind == "ppr":
        c.update(graph="rmat", n=_size(rng, 500, 12000), ef=rng.choice([4, 8, 16]), graphs=rng.randint(2, 16),
                 rhs=rng.choice([8, 17, 32, 64]), state=rng.choice(["f32", "f32_kahan"]))
        return c
    c["n"] = _size(rng, 500, 3000000)
    if graph == "rmat":
        c["ef"] = rng.choice([8, 16])
    if kind == "sssp":
        c.update(state=rng.choice(["u32", "f64"]), sched=rng.choice(["all", "sampled", "exact"]))
    elif kind == "components":
        c.update(state="i32", sched=rng.choice(["all", "sampled"]))
    elif kind == "pagerank":
        c.update(state=rng.choice(["f64", "f32", "f32_kahan"]),
                 sched=rng.choice(["all", "all", "sampled", "exact", "sweep", "learned"]))
    else:
        c.update(state=rng.choice(["f64", "f32"]), sched=rng.choice(["all", "all", "sampled", "sweep"]))
    if c["sched"] == "sweep":
        c["q"] = rng.choice([0.125, 0.25])
    elif c["sched"] != "all":
        c["q"] = rng.choice([0.05, 0.1, 0.2])
    return c


# ---------------------------------------------------------------------------
# Inputs, made on the device from the seed.
# ---------------------------------------------------------------------------
def _gen(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(int(seed) * 2654435761 % (1 << 62) + 1)
    return g


def _normal(gen, n, mu, sigma):
    return torch.exp(torch.randn(n, generator=gen, device=DEV, dtype=torch.float64) * sigma + mu)


def _edges(case, n, gen):
    """(source, target) of every edge, in no order."""
    kind = case["graph"]
    if kind == "rmat":  # a/b/c/d = .57/.19/.19/.05, ids scaled to [0, n)
        m, scale = n * case.get("ef", 16), max(1, (n - 1).bit_length())
        src = torch.zeros(m, dtype=torch.int64, device=DEV)
        dst = torch.zeros(m, dtype=torch.int64, device=DEV)
        for _ in range(scale):
            u = torch.rand(m, generator=gen, device=DEV)
            src.mul_(2).add_(u >= 0.76)
            dst.mul_(2).add_(((u >= 0.57) & (u < 0.76)) | (u >= 0.95))
        if n != 1 << scale:
            src = (src * n) >> scale
            dst = (dst * n) >> scale
        return src, dst
    if kind == "powerlaw":  # log-normal out-degrees, targets by a power law over permuted ids
        deg = torch.clamp(_normal(gen, n, 2.0, 1.0).long(), max=500)
        src = torch.repeat_interleave(torch.arange(n, device=DEV), deg)
        u = torch.rand(src.numel(), generator=gen, device=DEV, dtype=torch.float64)
        return src, torch.randperm(n, generator=gen, device=DEV)[(n * u ** 2.5).long().clamp_(max=n - 1)]
    # the paper's generator: log-normal in-degrees, uniform sources
    deg = torch.clamp(_normal(gen, n, -0.5, 2.3).long(), max=max(1, n // 4))
    dst = torch.repeat_interleave(torch.arange(n, device=DEV), deg)
    return torch.randint(0, n, (dst.numel(),), generator=gen, device=DEV), dst


def _csr(case, n, gen, symmetric=False):
    src, dst = _edges(case, n, gen)
    if symmetric:
        src, dst = torch.cat([src, dst]), torch.cat([dst, src])
    key = (src << 32) | dst
    del src, dst
    key = key.sort().values
    src = key >> 32
    row = torch.zeros(n + 1, dtype=torch.int64, device=DEV)
    row[1:] = torch.cumsum(torch.bincount(src, minlength=n), 0)
    del src
    return row, (key & 0xFFFFFFFF).to(torch.int32)


def _in_edges(row, col):
    """The edges by target: first edge of each, source and number of each edge."""
    n = row.numel() - 1
    sorted_dst, order = torch.sort(col, stable=True)
    offsets = torch.searchsorted(sorted_dst, torch.arange(n + 1, dtype=torch.int32, device=DEV))
    del sorted_dst
    src = torch.repeat_interleave(torch.arange(n, device=DEV), row[1:] - row[:-1])[order]
    return offsets, src, order


def _segment_sums(x, offsets):
    n, most = offsets.numel() - 1, 1 << 22  # targets of one call
    return torch.cat([torch.segment_reduce(x, "sum", offsets=offsets[i:min(n, i + most) + 1], unsafe=True, initial=0)
                      for i in range(0, n, most)])


def _weights(case, row, col, gen):
    m = col.numel()
    if case["kind"] == "sssp":
        if case["state"] == "u32":
            return torch.randint(1, 256, (m,), generator=gen, device=DEV, dtype=torch.int32)
        return _normal(gen, m, 0.0, 1.0)  # the paper's log-normal(0, 1) weights
    # Adsorption: log-normal(0.4, 0.8) weights, normalised over each receiver's in-edges
    w = _normal(gen, m, 0.4, 0.8)
    offsets, _, order = _in_edges(row, col)
    w = w / _segment_sums(w[order], offsets)[col.long()]
    return w.float() if case["state"].startswith("f32") else w


def _inputs(case, seed):
    """The arrays of a single-graph case: row, col, w, alpha, alpha_pv, v0, dv1."""
    gen = _gen(seed)
    n, kind = case["n"], case["kind"]
    row, col = _csr(case, n, gen, symmetric=kind == "components")
    s = {"row": row, "col": col, "w": None, "alpha": 0.0, "alpha_pv": None}
    if kind == "sssp":
        s["w"] = _weights(case, row, col, gen)
        source = int(torch.argmax(row[1:] - row[:-1]))  # a source that reaches much of the graph
        if case["state"] == "u32":
            s["v0"] = torch.full((n,), -1, dtype=torch.int32, device=DEV)  # 0xFFFFFFFF
        else:
            s["v0"] = torch.full((n,), math.inf, dtype=torch.float64, device=DEV)
        s["dv1"] = s["v0"].clone()
        s["dv1"][source] = 0
        return s
    if kind == "components":
        s["v0"] = torch.full((n,), -1, dtype=torch.int32, device=DEV)
        s["dv1"] = torch.arange(n, dtype=torch.int32, device=DEV)
        return s
    dt = torch.float64 if case["state"] == "f64" else torch.float32
    s["v0"] = torch.zeros(n, dtype=dt, device=DEV)
    if kind == "pagerank":
        s["alpha"] = 0.8
        s["dv1"] = torch.full((n,), 0.2, dtype=dt, device=DEV)
    elif kind == "katz":  # half of 1 / rho(A), rho by power iteration
        x = torch.ones(n, dtype=torch.float64, device=DEV)
        offsets, src, _ = _in_edges(row, col)
        rho = 1.0
        for _ in range(12):
            y = _segment_sums(x[src], offsets)
            rho = max(float(y.norm() / x.norm()), 1.0)
            x = y / max(float(y.norm()), 1e-300)
        s["alpha"] = round(0.5 / rho, 12)
        s["dv1"] = torch.rand(n, generator=gen, device=DEV, dtype=torch.float64).to(dt)
    else:  # adsorption: continuation probability of each sender, injected label mass
        s["w"] = _weights(case, row, col, gen)
        s["alpha_pv"] = (0.6 + 0.3 * torch.rand(n, generator=gen, device=DEV, dtype=torch.float64)).cpu().numpy()
        s["dv1"] = (0.2 * torch.rand(n, generator=gen, device=DEV, dtype=torch.float64)).to(dt)
    return s


def _sizes(case):
    """Vertices of each graph of a batch (uneven)."""
    n = case["n"]
    return [max(64, n * (g % 4 + 1) // 2 + 3 * g) for g in range(case["graphs"])]


def _batch_inputs(case, seed):
    gen = _gen(seed)
    graphs, p = [], []
    for n in _sizes(case):
        row, col = _csr(case, n, gen)
        graphs.append((row, col))
        # each right-hand side restarts at up to 32 seeds
        k = torch.randint(1, 33, (case["rhs"],), generator=gen, device=DEV)
        at = torch.randint(0, n, (case["rhs"], 32), generator=gen, device=DEV)
        on = (torch.arange(32, device=DEV)[None, :] < k[:, None]).double() / k[:, None]
        dv = torch.zeros(case["rhs"], n, dtype=torch.float64, device=DEV).scatter_add_(1, at, on * (1.0 - 0.85))
        p.append(dv.t().contiguous().cpu().numpy())
    return graphs, p


_OPS = {"pagerank": (daic.SUM, daic.G_DEG_SCALE), "katz": (daic.SUM, daic.G_SRC_SCALE),
        "adsorption": (daic.SUM, daic.G_EDGE_SCALE), "sssp": (daic.MIN, daic.G_EDGE_ADD),
        "components": (daic.MAX, daic.G_COPY)}


def prepare(case, seed):
    if case["kind"] == "ppr":
        graphs, p = _batch_inputs(case, seed)
        handles = [daic.Graph.from_device(row, col) for row, col in graphs]
        torch.cuda.synchronize()
        batch = daic.Batch(handles, case["rhs"], alpha=0.85, state=case["state"])
        return {"case": case, "batch": batch, "v0": [np.zeros_like(x) for x in p], "dv1": p}
    s = _inputs(case, seed)
    torch.cuda.synchronize()
    op, g = _OPS[case["kind"]]
    graph = daic.Graph.from_device(s["row"], s["col"], s["w"])
    problem = daic.Problem(graph, op, g, alpha=s["alpha"], alpha_pv=s["alpha_pv"], state=case["state"])
    opts = {"sched": case["sched"], "q": case.get("q", 1.0), "seed": 7}
    if op == daic.SUM:
        opts["eps"] = 1e-6 if case["n"] > 100000 or case["state"] != "f64" else 1e-9
    if case["sched"] == "learned":
        opts["model"] = daic.SchedModel(seed=11)
        opts["model"].set_features([-20.0, 0.0, 0.1], [8.0, 2.0, 0.2])
    # a single-precision result is kept in single precision
    out = torch.empty(case["n"], dtype=torch.float32) if case["state"].startswith("f32") else None
    return {"case": case, "problem": problem, "v0": s["v0"], "dv1": s["dv1"], "opts": opts, "out": out}


def run(state):
    if "batch" in state:
        b = state["batch"]
        for g in range(len(b.n)):
            b.set_init(g, state["v0"][g], state["dv1"][g])
        b.run(eps=1e-6)
        return [b.get(g).astype(np.float32) for g in range(len(b.n))]
    p = state["problem"]
    p.set_init_device(state["v0"], state["dv1"])
    p.run(**state["opts"])
    v = p.get()
    if state["out"] is None:
        return v
    return state["out"].copy_(torch.from_numpy(v))


def _mean_degree(case):
    if case["graph"] == "rmat":
        return case.get("ef", 16) * (2 if case["kind"] == "components" else 1)
    mean = 11.6 if case["graph"] == "powerlaw" else 7.5
    return mean * (2 if case["kind"] == "components" else 1)


def work(case):
    """The graph read once, the initial values read and the results written
    once, one multiply-add per edge."""
    if case["kind"] == "ppr":
        n = sum(_sizes(case))
        m = n * case["ef"]
        return {"bytes": 4.0 * (n + 1) + 4.0 * m + 3 * 8.0 * n * case["rhs"], "flops": 2.0 * m * case["rhs"]}
    n, size = case["n"], 8 if case["state"] == "f64" else 4
    m = n * _mean_degree(case)
    weight = 0 if case["kind"] in ("pagerank", "katz", "components") else size
    return {"bytes": 4.0 * (n + 1) + (4.0 + weight) * m + 3.0 * size * n, "flops": 2.0 * m}


# ---------------------------------------------------------------------------
# The same results in 64 bits, without the framework.
# ---------------------------------------------------------------------------
def _fixed_point(c, step):
    """x = c + step(x), by adding up the terms c, step(c), step(step(c)), ..."""
    x, d = c.clone(), c
    for _ in range(400):
        d = step(d)
        x += d
        if float(d.abs().sum()) <= 1e-15 * float(x.abs().sum()):
            break
    return x


def exact(case, seed):
    if case["kind"] == "ppr":
        graphs, p = _batch_inputs(case, seed)
        out = []
        for (row, col), dv in zip(graphs, p):
            deg = row[1:] - row[:-1]
            n = deg.numel()
            src = torch.repeat_interleave(torch.arange(n, device=DEV), deg)
            a = (0.85 / deg.clamp(min=1).double())[src]
            mat = torch.sparse_coo_tensor(torch.stack([col.long(), src]), a, (n, n)).coalesce()
            out.append(_fixed_point(torch.from_numpy(dv).to(DEV), lambda d: torch.sparse.mm(mat, d)).cpu().numpy())
        return out
    s = _inputs(case, seed)
    row, n = s["row"], case["n"]
    if case["kind"] in ("pagerank", "katz", "adsorption"):
        c = s["dv1"].double()
        deg = row[1:] - row[:-1]
        a = torch.full((n,), s["alpha"], dtype=torch.float64, device=DEV)
        if case["kind"] == "pagerank":
            a = a / deg.clamp(min=1)
        elif s["alpha_pv"] is not None:
            a = torch.from_numpy(s["alpha_pv"]).to(DEV)
        offsets, src, order = _in_edges(row, s["col"])
        w = None if s["w"] is None else s["w"].double()[order]
        del order
        v = _fixed_point(c, lambda d: _segment_sums((d * a)[src] if w is None else (d * a)[src] * w, offsets))
        return v.cpu() if case["state"] != "f64" else v.cpu().numpy()
    dst, deg = s["col"].long(), row[1:] - row[:-1]
    if case["kind"] == "components":
        v = torch.arange(n, dtype=torch.int64, device=DEV)
        for _ in range(n):
            new = v.clone().scatter_reduce_(0, dst, torch.repeat_interleave(v, deg), "amax")
            if torch.equal(new, v):
                break
            v = new
        return v.to(torch.int32).cpu().numpy()
    if case["state"] == "u32":
        v, inf, w = s["dv1"].long() & 0xFFFFFFFF, 0xFFFFFFFF, s["w"].long()
    else:
        v, inf, w = s["dv1"].clone(), math.inf, s["w"]
    for _ in range(n):
        new = v.clone().scatter_reduce_(0, dst, torch.repeat_interleave(v, deg) + w, "amin").clamp_(max=inf)
        if torch.equal(new, v):
            break
        v = new
    return v.cpu().numpy() if case["state"] == "f64" else v.cpu().numpy().astype(np.uint32)
