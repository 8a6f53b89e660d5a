"""Batches whose small instances fill the device while teams of workgroups want
it for the larger ones: the values are the oracle's, and the batch takes no
longer than its classes one after another (with half as much again for the
spread of the figures, and the millisecond that teams may wait for members)."""
import numpy as np
import pytest

import oracle as O
import workloads as W

pytestmark = pytest.mark.gpu

MIXES = {
    # more small instances than are resident at once, some just above the class bound
    "many": lambda: [W.grid_instance(40 + i % 30, 100 + i) for i in range(700)],
    # a few large ones behind them
    "few_large": lambda: [W.grid_instance(10 + i % 30, 200 + i) for i in range(600)] +
                         [W.grid_instance(120 + 10 * i, i) for i in range(8)],
    # random graphs around the class bound
    "random": lambda: [W.random_graph(100 + 4 * i, 800 + 32 * i, 1, 100, i, s=0, t=9) for i in range(300)],
}


@pytest.mark.parametrize("name", sorted(MIXES))
@pytest.mark.parametrize("blocks", [(256, 1024, 1024), (512, 1024)])
def test_mixed_batch(name, blocks):
    from paper_2511_05895_amd import mf
    gs = MIXES[name]()
    kw = dict(n_classes=len(blocks), block=list(blocks), class_max_arcs=[32768, 262144][:len(blocks) - 1])
    sizes = np.array([g.m for g in gs])
    check = sorted(set(np.argsort(-sizes)[:8].tolist()) | set(range(0, len(gs), 41)))
    want = [O.dinic(gs[i], gs[i].cap)[0] for i in check]
    with mf.Batch(gs, **kw) as B:
        ms = []
        for _ in range(6):
            values = B.solve()
            assert list(values[check]) == want
            ms.append(B.last_ms())
        parts = sum(min(B.solve_class(c) for _ in range(3)) for c in range(len(blocks)))
        assert list(B.values()[check]) == want
        print(f"{name} {blocks}: batch {min(ms):.2f} ms, classes one after another {parts:.2f} ms", flush=True)
        assert min(ms) <= 1.5 * parts + 1
