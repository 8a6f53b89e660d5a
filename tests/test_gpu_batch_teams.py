"""Batched instances solved by teams of workgroups of one XCD: merged size
classes, one class alone, classes of one workgroup beside them, more and fewer
instances than teams; against the oracle, on first solves, repeats and changed
capacities."""
import numpy as np
import pytest

import oracle as O
import workloads as W

from tests.graphs import from_edges
from tests.test_gpu_teams import hub_graph

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def mf():
    import torch
    assert torch.cuda.is_available()
    from paper_2511_05895_amd import mf as m
    return m


def instances(count):
    out = []
    for i in range(count):
        k = 700 + i
        if i % 4 == 0:
            out.append(W.seg_grid(5 + (11 * i) % 47, k))
        elif i % 4 == 1:
            out.append(W.random_graph(30 + 97 * i % 3000, 4 * (30 + 97 * i % 3000), 1, 100, k, s=0, t=9))
        elif i % 4 == 2:
            out.append(W.rmat(8 + i % 5, 8, k))
        else:
            out.append(from_edges(3, [(0, 1, 5), (1, 2, 4), (0, 0, 3)], 0, 2))
    if count > 8:
        out[7] = hub_graph(9001, 16)         # lists visited by wavefronts and workgroups
    return out


@pytest.mark.parametrize("count", [1, 3, 33, 150])
@pytest.mark.parametrize("blocks", [None, (256, 1024, 1024), (1024, 1024, 256), (1024,)])
def test_team_classes_match_oracle(mf, count, blocks):
    gs = instances(count)
    kw = {} if blocks is None else dict(n_classes=len(blocks), block=list(blocks))
    with mf.Batch(gs, **kw) as B:
        caps = [g.cap.copy() for g in gs]
        want = [O.dinic(g, g.cap)[0] for g in gs]
        assert list(B.solve()) == want
        assert list(B.solve()) == want
        for c in range(B.opts()["n_classes"]):
            B.solve_class(c)
        assert list(B.values()) == want
        rng = np.random.default_rng(5)
        for i in {0, count // 2, count - 1}:
            caps[i] = rng.integers(0, 50, gs[i].m)
            B.set_capacities(i, np.arange(gs[i].m), caps[i])
            want[i], side, _ = O.dinic(gs[i], caps[i])
        assert list(B.solve()) == want
        got, _ = B.min_cut(count - 1)
        assert np.array_equal(got, O.dinic(gs[count - 1], caps[count - 1])[1])
