"""Runs of small problems in one workgroup against the per-round kernels and
the oracle: same rounds, updates and messages, min and max states bit for bit,
sums to rounding (FP64: the two forms add the same FP64 messages in another
order, in-degrees up to 16,383 and up to 40 rounds: below 1e-12 relative; FP32
states round each sum once per round in both: below 40 roundings of 6e-8)."""
import numpy as np
import pytest

import daic_gen
import oracle

pytestmark = pytest.mark.gpu

daic = pytest.importorskip("paper_1710_05785_amd.daic")


def graph(n, kind, seed=1):
    """CSR of a test graph: random targets, with a hub that every vertex points
    to ("hub"), or without any edge ("empty")."""
    rng = np.random.default_rng(seed + n)
    if kind == "empty" or n < 2:
        return np.zeros(n + 1, dtype=np.uint64), np.zeros(0, dtype=np.uint32)
    deg = rng.integers(0, 12, n)
    deg[rng.integers(0, n)] = min(4 * n, 3000)  # one large sender
    row = np.concatenate([[0], np.cumsum(deg)]).astype(np.uint64)
    col = (n * rng.random(int(row[-1])) ** 3).astype(np.uint32)
    if kind == "hub":
        first = row[:-1][deg > 0].astype(np.int64)
        col[first] = n // 3
    return row, col


def problem(case, row, col):
    n, m = row.size - 1, col.size
    rng = np.random.default_rng(7)
    kind, state = case
    if kind == "sssp":
        w = rng.integers(1, 4, m).astype(np.uint32) if state == "u32" else rng.integers(1, 4, m).astype(np.float64)
        p = daic.Problem(daic.Graph(row, col, w), daic.MIN, daic.G_EDGE_ADD, state=state)
        v0 = np.full(n, daic.INF_U32, dtype=np.uint32) if state == "u32" else np.full(n, np.inf)
        dv1 = v0.copy()
        dv1[0] = 0
        return p, v0, dv1
    if kind == "components":
        p = daic.Problem(daic.Graph(row, col), daic.MAX, daic.G_COPY, state="i32")
        return p, np.full(n, -1, dtype=np.int32), np.arange(n, dtype=np.int32)
    if kind == "pagerank":
        p = daic.Problem(daic.Graph(row, col), daic.SUM, daic.G_DEG_SCALE, alpha=0.8, state=state)
    elif kind == "katz":
        p = daic.Problem(daic.Graph(row, col), daic.SUM, daic.G_SRC_SCALE, alpha=1e-3, state=state)
    else:
        w = rng.random(m) * 0.05
        p = daic.Problem(daic.Graph(row, col, w.astype(np.float32) if state != "f64" else w), daic.SUM,
                         daic.G_EDGE_SCALE, alpha_pv=rng.random(n), state=state)
    # equal deltas: every priority ties in the first rounds
    return p, np.zeros(n), np.full(n, 0.25)


CASES = [("pagerank", "f64"), ("pagerank", "f32_kahan"), ("katz", "f32"), ("adsorption", "f64"), ("adsorption", "f32"),
         ("sssp", "u32"), ("sssp", "f64"), ("components", "i32")]
# one vertex, a partial and a full wave, rows of 1,024, every number of rows
# that has a kernel of its own and the first size of the next, the largest
SIZES = [1, 64, 1024, 1025, 2049, 4097, 8193, 10241, 12289, 16384]


@pytest.mark.parametrize("case", CASES, ids=lambda c: "-".join(c))
@pytest.mark.parametrize("n", SIZES)
def test_small_runs_match_round_kernels(case, n, monkeypatch):
    kind = "hub" if n in (1025, 10241, 16384) else "empty" if n == 64 else "random"
    row, col = graph(n, kind)
    p, v0, dv1 = problem(case, row, col)
    for sched, q in (("all", 1.0), ("exact", 0.13), ("sampled", 0.2), ("round_robin", 0.3)):
        got = []
        for small in (True, False):
            if small:
                monkeypatch.delenv("DAIC_NO_SMALL", raising=False)
            else:
                monkeypatch.setenv("DAIC_NO_SMALL", "1")
            p.set_init(v0, dv1)
            r1 = p.run(eps=1e-9, sched=sched, q=q, max_rounds=7, seed=3)  # stopped by the limit, ...
            mid = p.get(with_dv=True)
            r2 = p.run(eps=1e-9, sched=sched, q=q, max_rounds=33, seed=3)  # ... then resumed
            got.append((r1, mid, r2, p.get(with_dv=True)))
        for a, b in ((got[0][0], got[1][0]), (got[0][2], got[1][2])):
            assert a.status == b.status
            if case[0] in ("sssp", "components") or sched in ("all", "round_robin"):
                for k in ("rounds", "activations", "pushed_edges"):
                    assert a.stats[k] == b.stats[k], (sched, k, a.stats, b.stats)
        for a, b in ((got[0][1], got[1][1]), (got[0][3], got[1][3])):
            for x, y in zip(a, b):
                if case[0] in ("sssp", "components"):
                    assert np.array_equal(x, y), sched
                elif sched in ("all", "round_robin"):
                    tol = 1e-12 if case[1] == "f64" else 40 * 6e-8
                    assert np.abs(x - y).sum() <= tol * max(np.abs(y).sum(), 1e-3), sched


@pytest.mark.parametrize("sched", ["all", "exact", "sampled", "round_robin"])
def test_small_runs_reach_the_oracle(sched):
    g = daic_gen.powerlaw(n=5000, seed=4)
    v0, dv1 = oracle.pagerank_init(g.n, 0.8)
    p = daic.Problem(daic.Graph(g.row_ptr, g.col), daic.SUM, daic.G_DEG_SCALE, alpha=0.8, state="f64")
    p.set_init(v0, dv1)
    assert p.run(eps=1e-10, sched=sched, q=0.1, seed=1).converged
    ref, _, _ = oracle.jacobi_sum(g, oracle.G_DEG_SCALE, 0.8, dv1, eps=1e-13)
    assert np.abs(p.get() - ref).sum() <= 1e-9
    w = daic_gen.sssp_weights(g.m, seed=3)
    ps = daic.Problem(daic.Graph(g.row_ptr, g.col, w), daic.MIN, daic.G_EDGE_ADD, state="u32")
    ps.set_init(*oracle.sssp_init(g.n, 0))
    assert ps.run(sched=sched, q=0.1).converged
    assert np.array_equal(ps.get(), oracle.dijkstra(g, w, 0))


def test_small_run_longer_than_one_launch():
    """A path of 5,000 vertices takes 5,000 rounds: more than one launch holds."""
    n = 5000
    row = np.minimum(np.arange(n + 1), n - 1).astype(np.uint64)
    col = np.arange(1, n, dtype=np.uint32)
    p = daic.Problem(daic.Graph(row, col, np.full(n - 1, 3, dtype=np.uint32)), daic.MIN, daic.G_EDGE_ADD, state="u32")
    v0, dv1 = oracle.sssp_init(n, 0)
    p.set_init(v0, dv1)
    r = p.run(sched="all")
    assert r.converged
    assert (r.stats["rounds"], r.stats["activations"], r.stats["pushed_edges"]) == (n, n, n - 1)
    assert np.array_equal(p.get(), 3 * np.arange(n, dtype=np.uint32))
