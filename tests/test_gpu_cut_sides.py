"""Minimum cuts whose sink side is small or nearly the whole graph, hubs
included, on graphs around the sizes at which the kernel changes how many
vertices a wavefront takes, with lists at the lengths at which they are split;
against the oracle."""
import numpy as np
import pytest

import oracle as O
import workloads as W

pytestmark = pytest.mark.gpu


def stars(n, degrees, seed):
    """Vertices of exactly the given degrees among the first, spokes after them;
    s is joined to the centres, spokes lead to t."""
    rng = np.random.default_rng(seed)
    c = 2 + np.arange(len(degrees))
    src, dst = [np.zeros(c.size, int)], [c]
    for v, d in zip(c, degrees):  # one arc is s's
        src.append(np.full(d - 1, v))
        dst.append(rng.choice(np.arange(2 + c.size, n), d - 1, replace=False))
    spokes = np.arange(2 + c.size, n)
    src.append(spokes)
    dst.append(np.ones(spokes.size, int))
    src, dst = np.concatenate(src), np.concatenate(dst)
    return W.edges_to_csr(n, src, dst, rng.integers(1, 50, src.size), 0, 1)


LENGTHS = [1, 2, 8, 15, 16, 17, 31, 63, 64, 65, 255, 256]


@pytest.mark.parametrize("n", [301, 2047, 2560, 32767, 32768, 33280])
@pytest.mark.parametrize("longest", [256, 257, 300])
@pytest.mark.parametrize("at", ["s", "t", "-"])
def test_cut(n, longest, at):
    from paper_2511_05895_amd import mf
    degrees = [d for d in LENGTHS if d < n - 20] + ([longest] if longest < n - 20 else [])
    g = stars(n, degrees * (4 if n > 400 else 1), 81)
    cap = g.cap.copy()
    if at == "s":
        cap[g.row_ptr[g.s]:g.row_ptr[g.s + 1]] = 1
    elif at == "t":
        cap[g.col == g.t] = 1
        cap[g.row_ptr[g.s]:g.row_ptr[g.s + 1]] = 30000
    with mf.MaxFlow(W.Graph(g.n, g.row_ptr, g.col, cap, g.s, g.t)) as F:
        value = F.solve()
        want, side_o, _ = O.dinic(g, cap)
        for _ in range(2):
            side, cut = F.min_cut()
            assert value == want == cut
            assert np.array_equal(side, side_o)
