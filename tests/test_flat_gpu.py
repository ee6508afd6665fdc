"""Rounds over lists of many runs on graphs whose longest list is below, at and
above a wavefront's length: the first keep their entries' order, the others
spread it."""
import numpy as np
import pytest

import graphgen as gg
import oracle

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("longest", [63, 64, 65])
def test_longest_list(longest):
    from paper_1911_09135_amd import alb

    n = 60_000  # more than one run of 256 for each workgroup of the automatic grid
    v = np.arange(n)
    src = np.concatenate([v, np.full(longest - 2, 7)])
    dst = np.concatenate([(v + 1) % n, np.arange(100, 100 + longest - 2)])
    g = gg.undirected(n, src, dst).with_weights(3)
    assert int(g.degrees().max()) == longest
    dg = alb.Graph(g.off, g.col, g.w, symmetric=True)
    for wg in (64, 256, 1024):
        o = dict(wg_size=wg, grid_wgs=16)
        assert np.array_equal(alb.cc(dg, **o)[0], oracle.cc(g))
        for k in (3, 4):
            assert np.array_equal(alb.kcore(dg, k, **o)[0], oracle.kcore(g, k))
        x, _ = alb.pagerank(dg, 0.85, 3, **o)
        assert np.array_equal(x, alb.pagerank(dg, 0.85, 3, launch="host")[0])
    star = [gg.from_edges(n, np.zeros(longest, np.int64), np.arange(1, longest + 1), np.ones(longest, np.int64)), g]
    sources, members = [0, 9, n // 2], [0, 1, 1]
    both = alb.GraphSet(star)
    for q, x in enumerate(alb.sssp_batch(both, members, sources, grid_wgs=16)[0]):
        assert np.array_equal(x, oracle.sssp(star[members[q]], sources[q]))
    for h in (dg, both):
        h.close()
