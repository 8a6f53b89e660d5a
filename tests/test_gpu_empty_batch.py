"""Empty update batches are accepted, also by a graph that has no edges."""
import numpy as np
import pytest

from tests.graphs import from_edges
from tests.gpu_util import check_solved

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("grid", [1, 0, 5])
@pytest.mark.parametrize("edges", [[], [(1, 1, 3)], [(0, 1, 4)]])
def test_empty_batches(edges, grid):
    import torch
    from paper_2511_05895_amd import mf
    g = from_edges(3, edges, 0, 1)
    ids, caps = np.zeros(0, np.int64), np.zeros(0, np.int32)
    with mf.MaxFlow(g, grid_blocks=grid, flags=mf.MF_FLAG_DEBUG_CHECKS) as F:
        want = F.solve()
        assert F.update(ids, caps) == want
        assert F.update_noalloc(ids, caps) == want
        assert F.update_device(torch.from_numpy(ids).cuda(), torch.from_numpy(caps).cuda()) == want
        check_solved(F, g, g.cap)
