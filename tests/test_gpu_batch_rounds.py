"""What a batch keeps whatever its size: dense rounds and sweeps that repeat bit
for bit where every hub's in-edges fit one item (1,024 in dense rounds, 256 in
sweeps), and as many rounds per graph launch as the caller asks for."""
import numpy as np
import pytest

import daic_gen

pytestmark = pytest.mark.gpu

daic = pytest.importorskip("paper_1710_05785_amd.daic")


def hub_graph(n, hubs, seed):
    """Three edges from every vertex, and targets with the given in-degrees."""
    rng = np.random.default_rng(seed)
    src, dst = [np.repeat(np.arange(n), 3)], [rng.integers(len(hubs), n, 3 * n)]
    for i, h in enumerate(hubs):
        src.append(rng.choice(n, h, replace=False))
        dst.append(np.full(h, i))
    return daic_gen.from_edges(n, np.concatenate(src), np.concatenate(dst))


def solve(gs, state, weighted, tune=False, **kw):
    rng = np.random.default_rng(5)
    ws = [rng.uniform(0.02, 0.04, g.m).astype(np.float32) if weighted else None for g in gs]
    b = daic.Batch([daic.Graph(g.row_ptr, g.col, w) for g, w in zip(gs, ws)], 19, alpha=0.85, state=state,
                   g=daic.G_EDGE_SCALE if weighted else None)
    for i, g in enumerate(gs):  # every vertex is pending: rounds are dense from the first on
        b.set_init(i, np.zeros((g.n, 19)), rng.random((g.n, 19)))
    if tune:
        b.tune()
    r, inst = b.run(**kw)
    return r, inst, [b.get(i) for i in range(len(gs))]


@pytest.mark.parametrize("weighted", [False, True])
@pytest.mark.parametrize("state", ["f32", "f32_kahan"])
@pytest.mark.parametrize("sched,q,hubs", [("all", 1.0, [65, 200, 333, 511, 512, 513, 700, 901, 1023, 1024] * 4),
                                          ("sweep", 0.25, [65, 100, 129, 193, 255, 256] * 6)])
def test_batches_repeat_bit_for_bit(sched, q, hubs, state, weighted):
    gs = [hub_graph(n, hubs, seed=n) for n in (1500, 4000, 2222)]
    for limit in (0, 9):  # to the stop rule, and stopped with messages in flight
        out = [solve(gs, state, weighted, eps=1e-5, sched=sched, q=q, max_rounds=limit) for _ in range(4)]
        for r, inst, vs in out[1:]:
            assert r.stats["rounds"] == out[0][0].stats["rounds"]
            np.testing.assert_array_equal(inst, out[0][1])
            for a, b in zip(vs, out[0][2]):
                np.testing.assert_array_equal(a, b)


@pytest.mark.parametrize("weighted", [False, True])
@pytest.mark.parametrize("sched,q", [("all", 1.0), ("sweep", 0.25)])
def test_lanes_of_hub_sums(sched, q, weighted, monkeypatch, tmp_path):
    """16, 32 and 64 lanes per vertex take the rows of a piece in one, two and
    four passes; targets of several pieces among them. Each sum is rounded in
    another order: 1e-5 holds 160 roundings of FP32."""
    gs = [hub_graph(n, [65, 300, 1024, 1025, 1500, 2100, 4000] * 3, seed=n) for n in (4500, 6001)]
    for limit in (0, 9):
        out = []
        for lanes in (16, 32, 64):
            cache = tmp_path / f"tuned{lanes}"
            cache.write_text(f"batch-fused N={sum(g.n for g in gs)} M={sum(g.m for g in gs)} G=2 kahan=1 "
                             f"weighted={int(weighted)} : 16 {lanes} 16 4096 64 8192\n")
            monkeypatch.setenv("DAIC_TUNE_CACHE", str(cache))
            out.append(solve(gs, "f32_kahan", weighted, tune=True, eps=1e-5, sched=sched, q=q, max_rounds=limit))
        for r, inst, vs in out[1:]:
            if limit:
                assert r.stats["rounds"] == out[0][0].stats["rounds"] == limit
            for a, b in zip(vs, out[0][2]):
                assert np.abs(a - b).sum() <= 1e-5 * np.abs(b).sum()


def graph_launches(f):
    from torch.profiler import ProfilerActivity, profile

    with profile(activities=[ProfilerActivity.CPU, ProfilerActivity.CUDA]) as prof:
        f()
    return sum(e.name == "hipGraphLaunch" for e in prof.events())


@pytest.mark.parametrize("dense", [False, True])
def test_rounds_of_a_launch(dense):
    """A path takes a round per vertex: one vertex pending at a time, or every
    vertex (dense rounds throughout)."""
    n = 256
    g = daic_gen.from_edges(n, np.arange(n - 1), np.arange(1, n))
    b = daic.Batch([daic.Graph(g.row_ptr, g.col)], 2, alpha=0.85, state="f32")
    dv = np.full((n, 2), 1.0 if dense else 0.0)
    dv[0] = 1.0

    def run(rounds, per_check):
        b.set_init(0, np.zeros((n, 2)), dv)
        r, _ = b.run(eps=0.0, rounds_per_check=per_check, max_rounds=rounds)
        assert r.stats["rounds"] == rounds

    for rounds, per_check, launches in ((100, 0, 1), (128, 0, 1), (100, 50, 2), (60, 20, 3), (24, 8, 3)):
        run(rounds, per_check)
        assert graph_launches(lambda: run(rounds, per_check)) == launches, (rounds, per_check)
