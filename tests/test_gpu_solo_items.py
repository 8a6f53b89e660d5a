"""Levels and round lists at the largest size that one workgroup of a team all
over the device works on alone (512 items or vertices, whatever solo_items
asks for): layers of 511, 512 and 513 vertices between s and t."""
import numpy as np
import pytest

import workloads as W

from tests.gpu_util import check_solved

pytestmark = pytest.mark.gpu


def layers(widths, seed):
    """s, then layers of the given widths, then t; every vertex joined to three
    of the next layer (s and t to all of theirs)."""
    rng = np.random.default_rng(seed)
    src, dst, at, prev = [], [], 1, np.array([0])
    for w in widths:
        cur = at + np.arange(w)
        at += w
        if prev.size == 1:
            src.append(np.repeat(prev, w))
            dst.append(cur)
        else:
            src.append(np.repeat(prev, 3))
            dst.append(cur[rng.integers(0, w, 3 * prev.size)])
        prev = cur
    src.append(prev)
    dst.append(np.full(prev.size, at))
    src, dst = np.concatenate(src), np.concatenate(dst)
    return W.edges_to_csr(at + 1, src, dst, rng.integers(1, 40, src.size), 0, at)


@pytest.mark.parametrize("solo", [511, 512, 513, 1 << 20])
@pytest.mark.parametrize("bottom_up", [-1, 0])
def test_layers_at_the_limit(solo, bottom_up):
    from paper_2511_05895_amd import mf
    g = layers([511, 512, 513, 40, 512, 513, 511, 700, 512], 61)
    cap = g.cap.copy()
    with mf.MaxFlow(g, grid_blocks=5, solo_items=solo, bottom_up=bottom_up, flags=mf.MF_FLAG_DEBUG_CHECKS) as F:
        F.solve()
        check_solved(F, g, cap)
        rng = np.random.default_rng(9)
        for k in (512, 2500):
            ids, new = W.mixed_batch(cap, k, 60, rng)
            cap[ids] = new
            F.update(ids, new)
            check_solved(F, g, cap)
