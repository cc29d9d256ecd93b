"""What small problems keep from the per-round kernels when they run in one
workgroup: selections, counters and states under every rule (sums of powers of
two, which any order of additions gives exactly), messages over infinite
weights and below zero, and the run's time; and the per-round kernels
themselves at these sizes, which the default route no longer takes."""
import numpy as np
import pytest

import daic_gen
import test_gpu_parity as parity
from test_gpu_small import CASES, graph
from test_gpu_small import test_small_runs_match_round_kernels as match_round_kernels

pytestmark = pytest.mark.gpu

daic = pytest.importorskip("paper_1710_05785_amd.daic")

RULES = [("all", 1.0), ("exact", 0.13), ("exact", 0.5), ("sampled", 0.2), ("sampled", 0.6), ("round_robin", 0.3)]


def exact_sums(kind, state, n):
    """A sum problem whose deltas, factors and weights are powers of two."""
    rng = np.random.default_rng(n)
    row, col = graph(n, "hub" if n == 1025 else "random")
    if kind == "pagerank":  # out-degrees are powers of two
        deg = 2 ** rng.integers(0, 4, n)
        deg[rng.random(n) < 0.2] = 0
        row = np.concatenate([[0], np.cumsum(deg)]).astype(np.uint64)
        col = (n * rng.random(int(row[-1])) ** 2).astype(np.uint32)
        p = daic.Problem(daic.Graph(row, col), daic.SUM, daic.G_DEG_SCALE, alpha=0.5, state=state)
    elif kind == "katz":
        p = daic.Problem(daic.Graph(row, col), daic.SUM, daic.G_SRC_SCALE, alpha=0.5, state=state)
    else:
        w = 2.0 ** -rng.integers(1, 3, col.size)
        p = daic.Problem(daic.Graph(row, col, w.astype(np.float32) if state != "f64" else w), daic.SUM,
                         daic.G_EDGE_SCALE, alpha_pv=2.0 ** -rng.integers(0, 2, n), state=state)
    dv = 2.0 ** rng.integers(0, 3, n) * np.where(rng.random(n) < 0.3, -1, 1)
    dv[rng.random(n) < 0.1] = 0.0
    return p, np.zeros(n), dv


@pytest.mark.parametrize("state", ["f64", "f32", "f32_kahan"])
@pytest.mark.parametrize("kind", ["pagerank", "katz", "adsorption"])
@pytest.mark.parametrize("n", [1025, 5000, 9999, 16384])
def test_small_selections_of_sums(n, kind, state, monkeypatch):
    """FP32 sums of two rounds fit their 24 bits (4 x 4,000 messages of a
    target, a quarter each time), FP64 sums of six rounds their 53."""
    p, v0, dv1 = exact_sums(kind, state, n)
    for sched, q in RULES:
        for rounds in (1, 6 if state == "f64" else 2):
            got = []
            for small in (True, False):
                monkeypatch.delenv("DAIC_NO_SMALL", raising=False) if small else monkeypatch.setenv("DAIC_NO_SMALL", "1")
                p.set_init(v0, dv1)
                r = p.run(eps=0.0, sched=sched, q=q, max_rounds=rounds, seed=3)
                got.append(([r.status] + [r.stats[k] for k in ("rounds", "activations", "pushed_edges")],
                            p.get(with_dv=True)))
            assert got[0][0] == got[1][0], (sched, q, rounds)
            for x, y in zip(got[0][1], got[1][1]):
                np.testing.assert_array_equal(x, y, err_msg=f"{sched} {q} {rounds}")


@pytest.mark.parametrize("state", ["f64", "f32", "f32_kahan"])
@pytest.mark.parametrize("weight", [np.inf, -np.inf, np.nan])
def test_small_runs_send_nothing_over_silent_edges(weight, state):
    """A weight that is no number is read only when its sender sends: vertex
    n - 1, whose out-edges hold it, has no delta."""
    n = 1500
    row = np.arange(n + 1, dtype=np.uint64)  # a path, and the last vertex points into it
    row[-1] += 39
    col = np.concatenate([np.arange(1, n), np.arange(40)]).astype(np.uint32)
    col[n - 2] = 0
    w = np.full(col.size, 0.5)
    w[n - 1:] = weight
    p = daic.Problem(daic.Graph(row, col, w if state == "f64" else w.astype(np.float32)), daic.SUM, daic.G_EDGE_SCALE,
                     alpha=0.5, state=state)
    dv = np.zeros(n)
    dv[3] = 1.0
    for sched in ("all", "exact", "sampled", "round_robin"):
        p.set_init(np.zeros(n), dv)
        r = p.run(eps=1e-12, sched=sched, q=0.2 if sched != "all" else 1.0, seed=2)
        assert r.converged, sched
        v = p.get()
        ref = np.zeros(n)
        ref[3:23] = 0.25 ** np.arange(20)
        np.testing.assert_allclose(v[:23], ref[:23], rtol=1e-6, atol=0, err_msg=sched)
        assert np.isfinite(v).all(), sched


def test_small_runs_keep_distances_below_zero():
    """Starting distances may be negative (weights may not): a message that is
    no smaller than a pending one leaves it."""
    n = 4000
    src = np.concatenate([[0], np.arange(n)])
    dst = np.concatenate([[n - 1], (np.arange(n) * 7 + 1) % n])
    g = daic_gen.from_edges(n, src, dst)
    w = np.full(g.m, 5.0)
    p = daic.Problem(daic.Graph(g.row_ptr, g.col, w), daic.MIN, daic.G_EDGE_ADD, state="f64")
    v0 = np.full(n, np.inf)
    dv = v0.copy()
    dv[0], dv[n - 1] = 0.0, -3.0
    row, col = g.row_ptr.astype(np.int64), g.col.astype(np.int64)
    ref, tail = dv.copy(), np.repeat(np.arange(n), np.diff(row))
    for _ in range(n):
        new = ref.copy()
        np.minimum.at(new, col, ref[tail] + 5.0)
        if np.array_equal(new, ref):
            break
        ref = new
    for sched in ("exact", "all"):
        p.set_init(v0, dv)
        assert p.run(sched=sched, q=1.0 / n if sched == "exact" else 1.0).converged
        np.testing.assert_array_equal(p.get(), ref, err_msg=sched)


def test_time_of_a_first_small_run():
    """The layout that a problem's first run builds is no part of its rounds."""
    g = daic_gen.powerlaw(n=16000, seed=9)

    def make():
        p = daic.Problem(daic.Graph(g.row_ptr, g.col), daic.SUM, daic.G_DEG_SCALE, alpha=0.8, state="f64")
        p.set_init(np.zeros(g.n), np.full(g.n, 0.2))
        return p

    make().run(sched="all", max_rounds=3)  # (the kernel's code is loaded)
    times = []
    for _ in range(3):
        p = make()
        first = p.run(sched="all", max_rounds=3).stats["time_ms"]
        p.set_init(np.zeros(g.n), np.full(g.n, 0.2))
        times.append((first, p.run(sched="all", max_rounds=3).stats["time_ms"]))
    assert min(a for a, _ in times) <= 2 * max(b for _, b in times), times


@pytest.mark.parametrize("case", CASES, ids=lambda c: "-".join(c))
@pytest.mark.parametrize("n", [6144, 6145, 8192, 10240, 12288, 14336, 14337])
def test_small_runs_at_the_rows_of_their_kernels(case, n, monkeypatch):
    """The last size that each even number of rows of 1,024 holds, and the
    sizes at which some rules go to the round kernels."""
    match_round_kernels(case, n, monkeypatch)


@pytest.fixture
def rounds_apart(monkeypatch):
    monkeypatch.setenv("DAIC_NO_SMALL", "1")
    return monkeypatch


@pytest.mark.parametrize("n,ef", [(5, 2), (300, 3), (3000, 6)])
def test_fused_rounds_of_small_graphs(rounds_apart, n, ef):
    parity.test_fused_pull_small_graphs(daic, rounds_apart, n, ef)
    rng = np.random.default_rng(n)
    g = daic_gen.from_edges(n, rng.integers(0, n, n * ef), rng.integers(0, n, n * ef))
    p = daic.Problem(daic.Graph(g.row_ptr, g.col), daic.SUM, daic.G_DEG_SCALE, alpha=0.85, state="f64")
    p.set_init(np.zeros(n), np.full(n, 0.15))
    _, ks = p.profile(eps=1e-12, q=1.0, sched="all")
    assert {"tile_pull", "pull_fused"} & {k["name"] for k in ks}


@pytest.mark.parametrize("kind", ["sssp_u32", "sssp_f64", "cc_i32"])
@pytest.mark.parametrize("sched,q", [("all", 1.0), ("exact", 0.1), ("sampled", 0.1)])
def test_minmax_dense_rounds_of_a_partial_partition(rounds_apart, kind, sched, q):
    parity.test_minmax_dense_rounds_match_push(daic, rounds_apart, "powerlaw10k", kind, sched, q)


def test_profile_of_a_small_graph(rounds_apart):
    parity.test_profile_matches_run_and_accounts_the_pull(daic, rounds_apart)


@pytest.mark.parametrize("state,gk", [("f64", "deg"), ("f32_kahan", "deg"), ("f64", "edge")])
def test_pulls_of_dense_rounds_of_a_small_graph(rounds_apart, state, gk):
    parity.test_push_and_pull_rounds_agree(daic, rounds_apart, "pull_when_dense", state, gk)
