"""mf_resume ends at a maximum flow also when arcs out of the source are still
residual: the state that a solve kernel leaves when it stops while repairing a
batch, before it came to the source.  Made here by importing states: the flow
from before source arcs were raised, with the raised residuals, and no flow at
all."""
import numpy as np
import pytest

import oracle as O
from tests.gpu_util import check_solved
from tests.test_gpu_repair import graph

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("grid,source_arcs", [(1, 40), (0, 40), (0, 2600), (5, 2600)])
@pytest.mark.parametrize("flags", [0, 2])
def test_resume_pushes_what_the_source_still_has(grid, source_arcs, flags):
    from paper_2511_05895_amd import mf
    assert mf.MF_FLAG_PUSH_PULL == 2
    g = graph(9001, source_arcs, 31)
    rng = np.random.default_rng(8)
    with mf.MaxFlow(g, grid_blocks=grid, flags=flags | mf.MF_FLAG_DEBUG_CHECKS) as F:
        F.solve()
        cap, cf, e, _, ecap = F.export_state()
        # source edges raised, their flow left as it is
        arcs = O.PairGraph.build(g, g.cap).edge2arc
        ids = np.arange(g.row_ptr[g.s], g.row_ptr[g.s + 1])
        ids = ids[arcs[ids] >= 0]
        up = rng.integers(1, 60, ids.size)
        now = ecap.copy()
        now[ids] += up
        np.add.at(cap, arcs[ids], up)
        np.add.at(cf, arcs[ids], up)
        F.import_state(cap, cf, e, now)
        F.resume()
        check_solved(F, g, now)
        # no flow at all
        pg = O.PairGraph.build(g, now)
        F.import_state(pg.cap, pg.cap, np.zeros(g.n, np.int64), now)
        F.resume()
        check_solved(F, g, now)
        # and updates go on from there
        F.update(ids, g.cap[ids])
        now[ids] = g.cap[ids]
        check_solved(F, g, now, exact_heights=not flags)
