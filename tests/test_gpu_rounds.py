"""The kernels of a round at the sizes where their split changes: exact
selections at the edges of the radix passes' workgroups (4,096 keys), of their
grid (256 of them) and of the claim's blocks (2,048 of 256 vertices and the
first size with more); dense and push rounds of the same selections; sampled
thresholds among few pending vertices; scores beyond one group of 64 vertices
per wave; batches whose items and hub chunks are cut below, at and above their
smallest sizes. Selections, rounds of min problems and sums of powers of two
are compared exactly; batches in FP32 with the oracle's FP64 iteration to the
1e-5 of their residual."""
import numpy as np
import pytest

import daic_gen
import oracle

pytestmark = pytest.mark.gpu

daic = pytest.importorskip("paper_1710_05785_amd.daic")

SIZES = [4095, 4097, 524288, 524289, 1048577]


def edgeless(n):
    g = daic_gen.from_edges(n, [], [])
    return daic.Graph(g.row_ptr, g.col)


@pytest.mark.parametrize("state", ["f64", "f32", "u32"])
@pytest.mark.parametrize("n", SIZES)
def test_exact_selection_at_split_edges(n, state):
    rng = np.random.default_rng(n)
    if state == "u32":
        g = daic_gen.from_edges(n, [], [])
        p = daic.Problem(daic.Graph(g.row_ptr, g.col, np.zeros(0, dtype=np.uint32)), daic.MIN, daic.G_EDGE_ADD,
                         state="u32")
        v = rng.integers(1000, 1000000, n).astype(np.uint32)
        dv = v - rng.integers(0, 300, n).astype(np.uint32)  # priorities below 300, a fraction not pending
        pr = oracle.priority(oracle.OP_MIN, v, dv)
    else:
        p = daic.Problem(edgeless(n), daic.SUM, daic.G_SRC_SCALE, alpha=0.5, state=state)
        dv = rng.integers(0, 64, n) * 0.25 * np.where(rng.random(n) < 0.5, -1, 1)
        tail = rng.random(n) < 0.3  # distinct keys beside the ties
        dv[tail] = rng.random(int(tail.sum())).astype(np.float32)
        v, pr = np.zeros(n), np.abs(dv)
    p.set_init(v, dv)
    for q in (0.31, 1.5 / n, 0.999):
        sel, _ = p.select_frontier(q=q, sched="exact")
        np.testing.assert_array_equal(np.nonzero(sel)[0], oracle.topk_exact(pr, q))


@pytest.mark.parametrize("n", SIZES)
def test_dense_and_push_rounds_agree(n, monkeypatch):
    """Deltas and message factors are powers of two, so every sum is exact
    and the order of the additions does not show."""
    rng = np.random.default_rng(n + 1)
    m = 3 * n
    deg = np.full(n, 2)
    deg[rng.choice(n, 3, replace=False)] += (m - 2 * n) // 3  # rows of both bins, of many chunks
    row = np.concatenate([[0], np.cumsum(deg)]).astype(np.uint64)
    col = (n * rng.random(int(row[-1])) ** 2).astype(np.uint32)
    dv = 2.0 ** rng.integers(0, 4, n)
    dv[rng.random(n) < 0.1] = 0.0
    monkeypatch.setenv("DAIC_NO_SMALL", "1")
    for sched, q in (("exact", 0.37), ("sampled", 0.2), ("round_robin", 0.3)):
        got = []
        for push in (False, True):
            monkeypatch.setenv("DAIC_NO_PULL", "1") if push else monkeypatch.delenv("DAIC_NO_PULL", raising=False)
            p = daic.Problem(daic.Graph(row, col), daic.SUM, daic.G_SRC_SCALE, alpha=0.5, state="f64")
            p.set_init(np.zeros(n), dv)
            r = p.run(eps=0.0, sched=sched, q=q, max_rounds=3, seed=5)
            got.append((r.stats["rounds"], r.stats["activations"], r.stats["pushed_edges"], *p.get(with_dv=True)))
        assert got[0][:3] == got[1][:3], (sched, got[0][:3], got[1][:3])
        for x, y in zip(got[0][3:], got[1][3:]):
            np.testing.assert_array_equal(x, y)


@pytest.mark.parametrize("pending", [1, 50, 4096, 60000])
@pytest.mark.parametrize("state", ["f64", "f32"])
def test_sampled_threshold_of_a_narrow_frontier(state, pending):
    n = 100003
    rng = np.random.default_rng(pending)
    dv = np.zeros(n)
    at = rng.choice(n, pending, replace=False)
    dv[at] = rng.random(pending).astype(np.float32)
    p = daic.Problem(edgeless(n), daic.SUM, daic.G_SRC_SCALE, alpha=0.5, state=state)
    p.set_init(np.zeros(n), dv)
    for q, n_samples in ((0.1, 4096), (0.02, 1000), (0.5, 64)):
        for round_no in (0, 7):
            sel, _ = p.select_frontier(q=q, sched="sampled", seed=11, round_no=round_no, n_samples=n_samples)
            tau = oracle.sampled_threshold(dv, q, n_samples, 11, round_no)
            np.testing.assert_array_equal(sel, (dv >= tau) & (dv > 0))


@pytest.mark.parametrize("n", [63, 262144, 262209, 530001])
def test_scores_repeat_with_their_features(n):
    """Without edges a score depends on the vertex's delta alone: deltas of
    period 4,096 have scores of period 4,096."""
    dv = np.tile(np.random.default_rng(3).random(4096).astype(np.float32), n // 4096 + 1)[:n]
    dv[5::4096] = 0.0
    p = daic.Problem(edgeless(n), daic.SUM, daic.G_DEG_SCALE, alpha=0.85, state="f32")
    p.set_init(np.zeros(n), dv.astype(np.float64))
    m = daic.SchedModel(seed=34)
    m.set_features(np.array([-8.0, 0.1, 0.2], dtype=np.float32), np.array([5.0, 1.5, 0.5], dtype=np.float32))
    got = p.sched_score(m)
    assert (got[dv == 0] == 0).all() and (got[dv != 0] > 0).all()
    np.testing.assert_array_equal(got, np.resize(got[:4096], n))


@pytest.mark.parametrize("n,hubs", [(5, []), (700, [64]), (700, [65, 128, 129]), (9000, [1025, 8191]),
                                    (140001, [4097, 100, 64])])
def test_batches_cut_to_their_size(n, hubs):
    rng = np.random.default_rng(n)
    src, dst = [rng.integers(0, n, 4 * n)], [rng.integers(0, n, 4 * n)]
    for i, h in enumerate(hubs):  # (edges to a vertex that others reach seldom)
        src.append(rng.choice(n, min(h, n), replace=False))
        dst.append(np.full(src[-1].size, i))
    gs = [daic_gen.from_edges(n, np.concatenate(src), np.concatenate(dst)),
          daic_gen.from_edges(37, np.arange(37), (np.arange(37) * 5 + 1) % 37)]
    b = daic.Batch([daic.Graph(g.row_ptr, g.col) for g in gs], 3, alpha=0.85, state="f32")
    inits = []
    for i, g in enumerate(gs):
        dv1 = np.zeros((g.n, 3))
        dv1[rng.integers(0, g.n, 3), np.arange(3)] = 0.15
        inits.append(dv1)
        b.set_init(i, np.zeros((g.n, 3)), dv1)
    res, inst = b.run(eps=1e-7, rounds_per_check=4)
    assert res.converged and np.all(inst <= 1e-7)
    for i, g in enumerate(gs):
        v = b.get(i)
        for r in range(3):
            ref, _, _ = oracle.jacobi_sum(g, oracle.G_DEG_SCALE, 0.85, inits[i][:, r], eps=1e-14)
            assert np.abs(v[:, r] - ref).sum() <= 1e-5 * np.abs(ref).sum(), (i, r)
