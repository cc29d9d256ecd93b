"""Transfers of several threads run side by side: a small one does not wait for
the large ones of other threads, and no thread gets another's values."""
import threading
import time

import numpy as np
import pytest

from test_gpu_transfer import CHUNK8, empty_graph, roundtrip

pytestmark = pytest.mark.gpu

daic = pytest.importorskip("paper_1710_05785_amd.daic")


def problem(n):
    p = daic.Problem(empty_graph(n), daic.SUM, daic.G_SRC_SCALE, alpha=0.5, state="f64")
    p.set_init(np.arange(n, dtype=np.float64), np.zeros(n))
    return p


def test_small_reads_beside_large_ones():
    """A read waits for the kernels in flight when it begins: two chunks for
    each of a large read's eight threads at most, of its 256 chunks."""
    large, small = problem(256 * CHUNK8), problem(1000)
    stop, took = threading.Event(), []

    def read_large():
        while not stop.is_set():
            t = time.perf_counter()
            assert large.get()[-1] == 256 * CHUNK8 - 1
            took.append(time.perf_counter() - t)

    small.get()
    thread = threading.Thread(target=read_large)
    thread.start()
    while len(took) < 2:
        time.sleep(0.01)
    waits = []
    for _ in range(50):
        t = time.perf_counter()
        assert small.get()[-1] == 999
        waits.append(time.perf_counter() - t)
        time.sleep(0.001)
    stop.set()
    thread.join()
    assert np.median(waits) < 0.25 * np.median(took), (waits, took)


def test_many_threads_of_every_size():
    """More threads than chunks are kept for: one-chunk, two-chunk and many-chunk transfers."""
    ok = [True] * 12

    def work(i):
        for k in range(3):
            n = (100, CHUNK8 + 5, 21 * CHUNK8)[(i + k) % 3] + 7 * i
            ok[i] = ok[i] and roundtrip(n, "f32_kahan" if i % 2 else "f64", seed=i + k)

    ts = [threading.Thread(target=work, args=(i,)) for i in range(len(ok))]
    for t in ts:
        t.start()
    for t in ts:
        t.join()
    assert ok == [True] * len(ok)
