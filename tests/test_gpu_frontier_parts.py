"""Breadth-first levels whose frontier has fewer items than the team has
wavefronts (cut into halves and quarters of an item), lists of every length
around an item's and a quarter's; against the oracle."""
import numpy as np
import pytest

import workloads as W

from tests.gpu_util import check_solved
from tests.test_gpu_list_lengths import lengths_graph

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def mf():
    import torch
    assert torch.cuda.is_available()
    from paper_2511_05895_amd import mf as m
    return m


@pytest.mark.parametrize("grid", [2, 9, 40, 200])
@pytest.mark.parametrize("s_side", [True, False])
@pytest.mark.parametrize("bottom_up", [0, -1])
def test_small_frontiers_of_hubs(mf, grid, s_side, bottom_up):
    g = lengths_graph(4301, s_side, 77)
    cap = g.cap.copy()
    with mf.MaxFlow(g, grid_blocks=grid, solo_items=-1, bottom_up=bottom_up, vertex_order=2,
                    flags=mf.MF_FLAG_DEBUG_CHECKS) as F:
        F.solve()
        check_solved(F, g, cap)
        rng = np.random.default_rng(9)
        for k in (5, 700):
            ids, new = W.mixed_batch(cap, k, 100, rng)
            cap[ids] = new
            F.update(ids, new)
            check_solved(F, g, cap)
