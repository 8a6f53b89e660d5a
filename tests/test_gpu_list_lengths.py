"""Arc lists at the edges of the kernels' splits (8, 64, 256 and 4096 arcs),
as relabelled vertices, as ends of changed edges and as ends of cut edges;
numbers of vertices of every remainder of 4; against the oracle."""
import numpy as np
import pytest

import workloads as W

from tests.gpu_util import check_solved

pytestmark = pytest.mark.gpu

LENGTHS = [1, 7, 8, 9, 31, 32, 33, 63, 64, 65, 127, 128, 129, 255, 256, 257, 1023, 1025, 4095, 4096, 4097, 4200]


@pytest.fixture(scope="module")
def mf():
    import torch
    assert torch.cuda.is_available()
    from paper_2511_05895_amd import mf as m
    return m


def lengths_graph(n, s_side, seed):
    """A vertex of every length, joined both ways to a random graph; the
    narrow edges out of them (s_side) or into them are the cut."""
    rng = np.random.default_rng(seed)
    src, dst, cap = [], [], []
    k = len(LENGTHS)
    for i, deg in enumerate(LENGTHS):
        u = 1 + i
        other = k + 2 + rng.choice(n - k - 3, max(deg - 1, 0), replace=False)
        src += [0 if s_side else u] + ([u] * len(other) if s_side else list(other))
        dst += [u if s_side else n - 1] + (list(other) if s_side else [u] * len(other))
        cap += [10 ** 6] + list(rng.integers(0, 4, len(other)))
    m = 3 * n
    a, b = rng.integers(k + 2, n - 1, m), rng.integers(k + 2, n - 1, m)
    keep = a != b
    ends = np.arange(k + 2, n - 1, 3)
    far = np.full(len(ends), n - 1 if s_side else 0)
    src = np.concatenate([src, a[keep], ends if s_side else far])
    dst = np.concatenate([dst, b[keep], far if s_side else ends])
    cap = np.concatenate([cap, rng.integers(1, 30, int(keep.sum())), rng.integers(1, 90, len(ends))])
    return W.edges_to_csr(n, src, dst, cap, 0, n - 1)


@pytest.mark.parametrize("n", [4300, 4301, 9002, 9003])
@pytest.mark.parametrize("s_side", [True, False])
@pytest.mark.parametrize("order,gap", [(1, False), (2, False), (2, True)])
def test_list_lengths_match_oracle(mf, n, s_side, order, gap):
    g = lengths_graph(n, s_side, n)
    cap = g.cap.copy()
    flags = mf.MF_FLAG_DEBUG_CHECKS | (mf.MF_FLAG_GAP if gap else 0)
    with mf.MaxFlow(g, vertex_order=order, flags=flags) as F:
        F.solve()
        check_solved(F, g, cap)
        rng = np.random.default_rng(9)
        for k in (3, 900):
            ids, new = W.mixed_batch(cap, k, 100, rng)
            cap[ids] = new
            F.update(ids, new)
            check_solved(F, g, cap)
