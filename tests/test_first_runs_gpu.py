"""The first run of each workgroup in a phase: half of its share of the worklist,
rounded up to whole wavefronts' entries, also where the division is exact."""
import numpy as np
import pytest

import graphgen as gg

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nf,run", [(2, 64), (32 * 64 - 1, 64), (32 * 64, 64), (32 * 64 + 1, 128),
                                    (32 * 128, 128), (32 * 192 + 5, 256), (32 * 256, 256), (50_000, 256)])
def test_first_runs(nf, run):
    from paper_1911_09135_amd import alb

    wgs = 16
    g = gg.from_edges(nf, np.arange(nf), (np.arange(nf) + 1) % nf)  # one edge each
    dg = alb.Graph(g.off, g.col)
    r = alb.trace_round(dg, np.arange(nf, dtype=np.int32), off=g.off, mode="twc", launch="host", grid_wgs=wgs)
    first = min(nf, wgs * run)  # entries of the fixed runs; later ones are claimed
    assert np.array_equal(r["edge_thread"][:first] // 256, np.arange(first) // run)
    assert (r["edge_hits"] == 1).all()
    dg.close()
