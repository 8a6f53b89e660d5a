"""Which workgroups solve a graph by default: one up to 2^14 arcs, those of one
XCD but four up to 2^22, one per 2^16 arcs beyond, where two vertices count as an arc at
least.  Graphs at the edges of the rule, against the oracle."""
import numpy as np
import pytest

import workloads as W

from tests.gpu_util import check_solved

pytestmark = pytest.mark.gpu


def distinct_pairs(n, pairs, seed, used=None):
    """Graph of exactly `pairs` joined vertex pairs (2 * pairs arcs) among the
    first `used` of n vertices; s and t are two of them."""
    used = used or n
    rng = np.random.default_rng(seed)
    key = np.unique(np.sort(rng.integers(0, used, (2 * pairs + 64, 2)), axis=1) @ np.array([used, 1]))
    key = rng.permutation(key[key // used != key % used])[:pairs]
    assert key.size == pairs
    u, v = key // used, key % used
    turn = rng.random(pairs) < 0.5
    return W.edges_to_csr(n, np.where(turn, u, v), np.where(turn, v, u), rng.integers(1, 100, pairs), 0, used - 1)


CASES = {
    # n, joined pairs, vertices they lie among; workgroups (x: those of one XCD)
    "one, by arcs": (3000, 1 << 13, None, 1),
    "xcd, by arcs": (3000, (1 << 13) + 1, None, "x"),
    "one, by vertices": ((1 << 15) + 1, 2000, 900, 1),
    "xcd, by vertices": ((1 << 15) + 2, 2000, 900, "x"),
    "xcd, most arcs": (200_003, 1 << 21, None, "x"),
    "device, by arcs": (200_003, (1 << 21) + 1, None, 65),
    "xcd, most vertices": ((1 << 23) + 1, 2000, 900, "x"),
    "device, by vertices": ((1 << 23) + 2, 2000, 900, 65),
}


@pytest.mark.parametrize("name", list(CASES))
def test_default_team(name):
    import torch
    from paper_2511_05895_amd import mf
    n, pairs, used, blocks = CASES[name]
    if blocks == "x":
        blocks = torch.cuda.get_device_properties(0).multi_processor_count // 8 - 4
    g = distinct_pairs(n, pairs, 55, used)
    cap = g.cap.copy()
    with mf.MaxFlow(g) as F:
        F.solve()
        assert F.num_arcs == 2 * pairs
        assert F.stats()["grid_blocks"] == blocks
        check_solved(F, g, cap, full=False)
        ids, new = W.mixed_batch(cap, 300, 100, np.random.default_rng(7))
        cap[ids] = new
        F.update(ids, new)
        check_solved(F, g, cap, full=False)
