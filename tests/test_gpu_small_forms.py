"""What small problems keep from the per-round kernels when they run in one
workgroup."""
import numpy as np
import pytest

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
