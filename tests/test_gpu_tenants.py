"""A small graph's updates beside another handle's or a batch's long solves, one
stream and thread each: the results are the oracle's, and the updates do not
wait for the other's solves (an update that did would take half of one on average).
Several handles of the small graph, the best counts: the runtime maps streams
onto a few hardware queues, and what shares one runs in order."""
import threading
import time

import numpy as np
import pytest

import oracle as O
import workloads as W

pytestmark = pytest.mark.gpu


def small(n):
    """Graph, a batch of 100 edges, and the values without and with it."""
    g = W.random_graph(n, 8 * n, 1, 100, 91)
    rng = np.random.default_rng(1)
    ids = rng.choice(g.m, 100, replace=False)
    new = rng.integers(0, 100, 100).astype(np.int32)
    other = g.cap.copy()
    other[ids] = new
    return g, ids, new, [O.dinic(g, g.cap)[0], O.dinic(g, other)[0]]


def updates_beside(solve, flows, g, ids, new, want):
    """Median time of updates of each of `flows` while a thread calls solve()
    again and again, the least of them, and the time of solve() alone."""
    value = solve()
    begin = time.perf_counter()
    assert np.array_equal(solve(), value)
    long = time.perf_counter() - begin
    for flow in flows:
        assert flow.solve() == want[0]
    values, stop = [], threading.Event()

    def solves():
        while not stop.is_set():
            values.append(solve())
    thread = threading.Thread(target=solves)
    thread.start()
    medians = []
    try:
        for flow in flows:
            times = []
            for i in range(30):
                begin = time.perf_counter()
                assert flow.update(ids, new if i % 2 == 0 else g.cap[ids]) == want[1 - i % 2]
                times.append(time.perf_counter() - begin)
            medians.append(float(np.median(times)))
    finally:
        stop.set()
        thread.join()
    assert all(np.array_equal(v, value) for v in values)
    print(f"solve {1e3 * long:.1f} ms, updates beside it (ms) {[round(1e3 * t, 2) for t in medians]}", flush=True)
    return min(medians), long


@pytest.mark.parametrize("n", [1000, 3000, 20011])
def test_updates_beside_long_solves(n):
    from paper_2511_05895_amd import mf
    g, ids, new, want = small(n)
    with mf.MaxFlow(W.seg_grid(400, 92)) as A, mf.MaxFlow(g) as B, mf.MaxFlow(g) as C, mf.MaxFlow(g) as D:
        median, long = updates_beside(A.solve, (B, C, D), g, ids, new, want)
    assert median < 0.2 * long


@pytest.mark.parametrize("n", [1000, 3000, 20011])
def test_updates_beside_a_batch(n):
    from paper_2511_05895_amd import mf
    g, ids, new, want = small(n)
    # as many instances as XCDs: every team is as large as it can be
    with mf.Batch([W.grid_instance(200, i) for i in range(8)]) as A, \
            mf.MaxFlow(g) as B, mf.MaxFlow(g) as C, mf.MaxFlow(g) as D:
        median, long = updates_beside(A.solve, (B, C, D), g, ids, new, want)
    assert median < 0.2 * long
