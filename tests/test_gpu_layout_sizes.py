"""The device build of the arc layout at the edges of its kernels: numbers of
half-edges around a sort tile (4096) and a wavefront's share of it (1024), keys
of one to four digits, hubs that draw most edges, multi-edges and self-loops;
against a layout made on the host."""
import numpy as np
import pytest

import workloads as W

from tests.gpu_util import check_layout, check_solved

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def mf():
    import torch
    assert torch.cuda.is_available()
    from paper_2511_05895_amd import mf as m
    return m


def edges(n, m, hubs, loops, seed):
    rng = np.random.default_rng(seed)
    src, dst = rng.integers(0, n, m), rng.integers(0, n, m)
    at_hub = rng.random(m) < hubs
    dst[at_hub] = rng.integers(0, min(n, 3), int(at_hub.sum()))
    if not loops:
        dst = np.where(src == dst, (dst + 1) % n, dst)
    return W.edges_to_csr(n, src, dst, rng.integers(0, 50, m), 0, n - 1)


@pytest.mark.parametrize("n", [2, 16, 17, 256, 257, 5000, 70000])
@pytest.mark.parametrize("m", [1, 31, 511, 512, 513, 2047, 2048, 2049, 4096, 9001, 66000])
@pytest.mark.parametrize("hubs,loops", [(0.0, False), (0.7, True)])
def test_layout_sizes(mf, n, m, hubs, loops):
    g = edges(n, m, hubs, loops, 1000 * n + m)
    for order in (1, 2):
        with mf.MaxFlow(g, vertex_order=order, flags=mf.MF_FLAG_DEBUG_CHECKS) as F:
            check_layout(F, g, g.cap)
            if n * m <= 257 * 9001:
                F.solve()
                check_solved(F, g, g.cap)
