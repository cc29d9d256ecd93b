"""What small problems keep from the per-round kernels when they run in one
workgroup."""
import numpy as np
import pytest

import daic_gen
from test_gpu_small import CASES, test_small_runs_match_round_kernels as match_round_kernels

pytestmark = pytest.mark.gpu

daic = pytest.importorskip("paper_1710_05785_amd.daic")


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
