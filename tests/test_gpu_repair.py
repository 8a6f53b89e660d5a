"""Batches at the edges of the solve kernel's own repair (1024 and 2048 edges,
source lists of up to 2048 arcs and longer ones), on one workgroup, on an
XCD's team and on one all over the device: against the oracle, parallel and
antiparallel edges included, and refused batches leave the state alone."""
import numpy as np
import pytest

import workloads as W

from tests.gpu_util import check_solved

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def mf():
    import torch
    assert torch.cuda.is_available()
    from paper_2511_05895_amd import mf as m
    return m


def graph(n, source_arcs, seed):
    """Random graph with pairs of vertices joined several times, both ways."""
    rng = np.random.default_rng(seed)
    m = 3 * n
    u, v = rng.integers(0, n, m), rng.integers(0, n, m)
    a, b = rng.integers(0, n, 300), rng.integers(0, n, 300)
    s_ends = 1 + rng.integers(0, n - 2, source_arcs)
    src = np.concatenate([u, a, a, b, np.zeros(source_arcs, int)])
    dst = np.concatenate([v, b, b, a, s_ends])
    keep = src != dst
    cap = rng.integers(0, 60, int(keep.sum()))
    return W.edges_to_csr(n, src[keep], dst[keep], cap, 0, n - 1)


@pytest.mark.parametrize("grid,source_arcs", [(1, 40), (0, 40), (0, 2600), (5, 40), (5, 2600)])
@pytest.mark.parametrize("raise_share", [0.0, 0.5, 1.0])
def test_batches_at_the_repairs_edges(mf, grid, source_arcs, raise_share):
    g = graph(9001, source_arcs, 21)
    cap = g.cap.copy()
    rng = np.random.default_rng(4)
    with mf.MaxFlow(g, grid_blocks=grid, flags=mf.MF_FLAG_DEBUG_CHECKS) as F:
        F.solve()
        for k in (0, 1, 1023, 1024, 1025, 2047, 2048, 2049, 6000):
            ids = rng.choice(g.m, k, replace=False)
            up = rng.random(k) < raise_share
            new = np.where(up, cap[ids] + rng.integers(0, 40, k), rng.integers(0, 1 + cap[ids])).astype(np.int32)
            F.update(ids, new)
            cap[ids] = new
            check_solved(F, g, cap)


@pytest.mark.parametrize("grid", [1, 0, 5])
@pytest.mark.parametrize("k", [2, 1024, 2048, 2049])
def test_refused_batches_leave_the_state(mf, grid, k):
    g = graph(9001, 40, 22)
    cap = g.cap.copy()
    rng = np.random.default_rng(6)
    with mf.MaxFlow(g, grid_blocks=grid, flags=mf.MF_FLAG_DEBUG_CHECKS) as F:
        F.solve()
        ids = rng.choice(g.m, k, replace=False)
        new = rng.integers(0, 50, k).astype(np.int32)
        for at, i, c, word in ((k - 1, g.m, 1, "out of range"), (0, -1, 1, "out of range"),
                               (k // 2, None, -1, "capacity"), (k - 1, ids[0], 1, "duplicate")):
            bad, caps = ids.copy(), new.copy()
            bad[at] = ids[at] if i is None else i
            caps[at] = c
            with pytest.raises(mf.MfError) as e:
                F.update(bad, caps)
            assert e.value.code == mf.MF_EINVAL and word in str(e.value)
            check_solved(F, g, cap)
        F.update(ids, new)
        cap[ids] = new
        check_solved(F, g, cap)
