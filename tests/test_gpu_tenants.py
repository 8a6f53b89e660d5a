"""A small graph's updates beside another handle's long solves, one stream and
thread each: the results are the oracle's, and the updates do not wait for the
other's solves (an update that did would take half of one on average)."""
import threading
import time

import numpy as np
import pytest

import oracle as O
import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1000, 3000, 20011])
def test_updates_beside_long_solves(n):
    from paper_2511_05895_amd import mf
    g = W.random_graph(n, 8 * n, 1, 100, 91)
    rng = np.random.default_rng(1)
    ids = rng.choice(g.m, 100, replace=False)
    new = rng.integers(0, 100, 100).astype(np.int32)
    other = g.cap.copy()
    other[ids] = new
    want = [O.dinic(g, g.cap)[0], O.dinic(g, other)[0]]
    big = W.seg_grid(400, 92)
    with mf.MaxFlow(big) as A, mf.MaxFlow(g) as B:
        value = A.solve()
        begin = time.perf_counter()
        assert A.solve() == value
        long = time.perf_counter() - begin
        assert B.solve() == want[0]
        values, stop = [], threading.Event()

        def solves():
            while not stop.is_set():
                values.append(A.solve())
        other_thread = threading.Thread(target=solves)
        other_thread.start()
        times = []
        try:
            for i in range(40):
                begin = time.perf_counter()
                assert B.update(ids, new if i % 2 == 0 else g.cap[ids]) == want[1 - i % 2]
                times.append(time.perf_counter() - begin)
        finally:
            stop.set()
            other_thread.join()
        assert all(v == value for v in values)
        print(f"solve {1e3 * long:.1f} ms, updates beside it {1e3 * np.median(times):.2f} ms", flush=True)
        assert np.median(times) < 0.2 * long
