"""The BFS direction rule counts every reached arc once, also those of a level
that a run in LDS hands back because it holds too many arcs.

A chain of fans leads to t: one vertex, `a` vertices, `b` vertices joined to
each of them, one vertex, and so on; the level of the `a` vertices ends the run
that finds it.  Beside it lies a component that nothing reaches, with more than
14 times the arcs of the largest level: as long as the reached arcs are counted
right, no level is large enough to be worth a look at all other vertices, and
the pass reads the arcs of the vertices it reaches and no others."""
import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu


def fans(a, b, sections, dead_edges, seed):
    step = 1 + a + b
    src, dst = [], []
    for i in range(sections):
        c = 1 + i * step                      # c of section 0 is t
        mid, low, up = c + 1 + np.arange(a), c + 1 + a + np.arange(b), c + step
        src += [mid, np.repeat(low, a), np.full(b, up)]
        dst += [np.full(a, c), np.tile(mid, b), low]
    reached = 1 + sections * step
    n_dead = dead_edges // 10
    rng = np.random.default_rng(seed)
    u, v = rng.integers(0, n_dead, dead_edges), rng.integers(0, n_dead, dead_edges)
    src.append(1 + reached + u[u != v])
    dst.append(1 + reached + v[u != v])
    src, dst = np.concatenate(src), np.concatenate(dst)
    return W.edges_to_csr(1 + reached + n_dead, src, dst, np.ones(src.size, np.int64), 0, 1), reached


# the first by one XCD's team (a run ends above 65536 arcs), the second by
# workgroups of the whole device (8192)
@pytest.mark.parametrize("grid,a,b,dead_edges", [(0, 300, 230, 600_000), (5, 100, 90, 80_000)])
def test_a_handed_back_level_counts_once(grid, a, b, dead_edges):
    from paper_2511_05895_amd import mf
    sections = 19
    g, reached = fans(a, b, sections, dead_edges, 41)
    with mf.MaxFlow(g, grid_blocks=grid) as F:
        assert F.solve() == 0
        st = F.stats()
        rp = F.export_graph()[0]
    levels = a * (1 + b), b * (1 + a)
    assert rp[-1] - rp[1 + reached] > 14 * max(levels)
    assert st["global_relabels"] == 1 and st["bfs_vertices"] == reached
    assert st["bfs_arcs"] == rp[1 + reached] - rp[1]
