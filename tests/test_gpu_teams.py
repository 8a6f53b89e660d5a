"""The solve kernel's teams against the oracle: one workgroup, workgroups of
one XCD (graphs of more than 8192 vertices by default) and workgroups all over
the device, on graphs small enough for the oracle."""
import numpy as np
import pytest

import oracle as O
import workloads as W

from tests.gpu_util import check_solved

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def mf():
    import torch
    assert torch.cuda.is_available()
    from paper_2511_05895_amd import mf as m
    return m


def hub_graph(n, seed):
    """Random graph with an inner vertex joined to most others (a list of more
    than 4096 arcs, visited by whole workgroups)."""
    rng = np.random.default_rng(seed)
    m = 4 * n
    src = np.concatenate([rng.integers(0, n, m), np.full(n // 2, 7), rng.integers(1, n - 1, n // 2)])
    dst = np.concatenate([rng.integers(0, n, m), rng.integers(1, n - 1, n // 2), np.full(n // 2, 7)])
    keep = src != dst
    cap = rng.integers(1, 60, int(keep.sum()))
    return W.edges_to_csr(n, src[keep], dst[keep], cap, 0, n - 1)


GRAPHS = {
    "grid90": lambda: W.seg_grid(90, 11),        # 8102 vertices: one workgroup
    "grid91": lambda: W.seg_grid(91, 12),        # 8283: a team
    "grid130": lambda: W.seg_grid(130, 13),
    "random9k": lambda: W.random_graph(9001, 72013, 1, 100, 14),
    "rmat14": lambda: W.rmat(14, 14, 15),
    "hub": lambda: hub_graph(12007, 16),
    "path": lambda: W.edges_to_csr(9000, np.arange(8999), np.arange(1, 9000), np.full(8999, 5), 0, 8999),
}


@pytest.mark.parametrize("name", sorted(GRAPHS))
@pytest.mark.parametrize("grid,mode", [(0, 0), (1, 0), (5, 0), (0, 1)])
def test_teams_match_oracle(mf, name, grid, mode):
    g = GRAPHS[name]()
    cap = g.cap.copy()
    with mf.MaxFlow(g, grid_blocks=grid, mode=mode, flags=mf.MF_FLAG_DEBUG_CHECKS) as F:
        F.solve()
        check_solved(F, g, cap)
        rng = np.random.default_rng(3)
        for k in (1, 65, 3000):
            ids, new = W.mixed_batch(cap, min(k, g.m), 100, rng)
            cap[ids] = new
            F.update(ids, new)
            check_solved(F, g, cap)
