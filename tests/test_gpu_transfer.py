"""State set from and read into host arrays: every element arrives, in the
stored precision, around the sizes at which a transfer takes another chunk (1
MiB) or another thread, for each element type, and from two threads at once."""
import threading

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

daic = pytest.importorskip("paper_1710_05785_amd.daic")

CHUNK8, CHUNK4 = 1 << 17, 1 << 18  # elements of 8 and 4 bytes in a chunk


def empty_graph(n):
    return daic.Graph(np.zeros(n + 1, dtype=np.uint64), np.zeros(0, dtype=np.uint32))


def weighted_graph(n):
    row = np.zeros(n + 1, dtype=np.uint64)
    row[1:] = 1
    return daic.Graph(row, np.zeros(1, dtype=np.uint32), np.ones(1, dtype=np.uint32))


def stored(x):
    """A double as F32_KAHAN keeps it: an FP32 value and the FP32 rounding."""
    y = x.astype(np.float32)
    return y.astype(np.float64) - (y.astype(np.float64) - x).astype(np.float32)


def roundtrip(n, state, seed=0):
    rng = np.random.default_rng(seed + n)
    if state == "u32":
        p = daic.Problem(weighted_graph(n), daic.MIN, daic.G_EDGE_ADD, state=state)
        v, dv = (rng.integers(0, 1 << 32, n, dtype=np.uint32) for _ in range(2))
        want = v, dv
    elif state == "i32":
        p = daic.Problem(empty_graph(n), daic.MAX, daic.G_COPY, state=state)
        v, dv = (rng.integers(-1, 1 << 31, n).astype(np.int32) for _ in range(2))
        want = v, dv
    else:
        p = daic.Problem(empty_graph(n), daic.SUM, daic.G_SRC_SCALE, alpha=0.5, state=state)
        v, dv = rng.standard_normal(n), rng.standard_normal(n)
        f32 = lambda x: x.astype(np.float32).astype(np.float64)  # noqa: E731
        want = (v, dv) if state == "f64" else (f32(v), f32(dv)) if state == "f32" else (stored(v), f32(dv))
    p.set_init(v, dv)
    got = p.get(with_dv=True)
    return all(np.array_equal(a, b) for a, b in zip(got, want)) and np.array_equal(p.get(), want[0])


@pytest.mark.parametrize("state", ["f64", "f32", "f32_kahan", "u32", "i32"])
def test_problem_state_roundtrip(state):
    chunk = CHUNK4 if state in ("u32", "i32") else CHUNK8
    for n in (1, 255, chunk - 1, chunk, chunk + 1, 2 * chunk, 4 * chunk + 1, 15 * chunk + 7, 33 * chunk - 5):
        assert roundtrip(n, state), n


@pytest.mark.parametrize("rhs", [1, 17, 64])
def test_batch_state_roundtrip(rhs):
    rng = np.random.default_rng(rhs)
    ns = [3, CHUNK8 // rhs, CHUNK8 // rhs + 1, 5 * CHUNK8 // rhs + 3]
    for state in ("f32", "f32_kahan"):
        b = daic.Batch([empty_graph(n) for n in ns], rhs, alpha=0.85, state=state)
        data = [(rng.standard_normal((n, rhs)), rng.standard_normal((n, rhs))) for n in ns]
        for g in (2, 0, 3, 1):
            b.set_init(g, *data[g])
        for g, (v, dv) in enumerate(data):
            gv, gdv, done = b.get_state(g)
            want = stored(v) if state == "f32_kahan" else v.astype(np.float32).astype(np.float64)
            assert np.array_equal(gv, want), (g, state)
            assert np.array_equal(gdv, dv.astype(np.float32).astype(np.float64)), (g, state)
            assert not done.any()


def test_transfers_from_two_threads():
    ok = [True, True]

    def work(i):
        for k in range(4):
            ok[i] = ok[i] and roundtrip(3 * CHUNK8 + 11 * i + k, "f32_kahan" if i else "f64", seed=i)

    ts = [threading.Thread(target=work, args=(i,)) for i in range(2)]
    for t in ts:
        t.start()
    for t in ts:
        t.join()
    assert ok == [True, True]
