"""Rounds that list and relabel far more vertices than the workgroups' LDS
holds, with short and with long arc lists, so that most entries go to the
global lists: against the oracle, on one workgroup, one XCD and the device."""
import numpy as np
import pytest

import workloads as W

from tests.gpu_util import check_solved

pytestmark = pytest.mark.gpu


def fan(mids, hubs, seed):
    """s, `mids` vertices, `hubs` vertices (each joined to all of the former), t.
    Less can leave the middle than enters it."""
    rng = np.random.default_rng(seed)
    m, h = 1 + np.arange(mids), 1 + mids + np.arange(hubs)
    t = 1 + mids + hubs
    src = np.concatenate([np.zeros(mids, int), np.repeat(m, hubs), h])
    dst = np.concatenate([m, np.tile(h, mids), np.full(hubs, t)])
    cap = np.concatenate([rng.integers(1, 100, mids), rng.integers(0, 100 // hubs + 2, mids * hubs),
                          np.full(hubs, 20 * mids // hubs)])
    return W.edges_to_csr(t + 1, src, dst, cap, 0, t)


@pytest.mark.parametrize("grid", [1, 0, 5])
@pytest.mark.parametrize("flags", [0, 1])
# short lists and huge hubs; lists of 41 arcs, more of them than LDS entries
@pytest.mark.parametrize("mids,hubs", [(60_000, 1), (60_000, 3), (40_001, 40), (3_000, 40)])
def test_lists_beyond_the_stage(mids, hubs, grid, flags):
    from paper_2511_05895_amd import mf
    assert mf.MF_FLAG_GAP == 1
    g = fan(mids, hubs, 71)
    cap = g.cap.copy()
    with mf.MaxFlow(g, grid_blocks=grid, flags=flags | mf.MF_FLAG_DEBUG_CHECKS) as F:
        F.solve()
        check_solved(F, g, cap, exact_heights=not flags)
        ids, new = W.mixed_batch(cap, g.m // 3, 100, np.random.default_rng(2))
        cap[ids] = new
        F.update(ids, new)
        check_solved(F, g, cap, exact_heights=not flags)
