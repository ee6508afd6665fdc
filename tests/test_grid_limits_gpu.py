"""Explicit grids that a call accepts: at least these workgroups per CU, for
every operator and workgroup size."""
import numpy as np
import pytest

import graphgen as gg
import oracle

pytestmark = pytest.mark.gpu

PER_CU = {64: 16, 256: 4, 1024: 1}


@pytest.fixture(scope="module")
def handles():
    from paper_1911_09135_amd import alb

    # a hub of 1,200 edges and a ring
    n = 3000
    src = np.concatenate([np.arange(n), np.zeros(1200, np.int64)])
    dst = np.concatenate([(np.arange(n) + 1) % n, np.arange(2, 1202)])
    g = gg.undirected(n, src, dst).with_weights(3)
    return g, alb.Graph(g.off, g.col, g.w, symmetric=True, build_transpose=True), alb.GraphSet([g])


@pytest.mark.parametrize("wg", [64, 256, 1024])
@pytest.mark.parametrize("op", ["bfs", "sssp", "cc", "kcore", "pagerank", "pagerank_pull", "bfs_batch", "sssp_batch"])
def test_full_grids(handles, op, wg):
    import torch

    from paper_1911_09135_amd import alb

    g, dg, gs = handles
    per_cu = 20 if wg == 64 and op in ("kcore", "pagerank_pull") else PER_CU[wg]
    o = dict(wg_size=wg, grid_wgs=per_cu * torch.cuda.get_device_properties(0).multi_processor_count)
    if op in ("bfs", "sssp"):
        assert np.array_equal(getattr(alb, op)(dg, 5, **o)[0], getattr(oracle, op)(g, 5))
    elif op == "cc":
        assert np.array_equal(alb.cc(dg, **o)[0], oracle.cc(g))
    elif op == "kcore":
        for k in (2, 3, 4):
            assert np.array_equal(alb.kcore(dg, k, **o)[0], oracle.kcore(g, k))
    elif op.startswith("pagerank"):
        want = alb.pagerank(dg, 0.85, 3)[0]
        assert np.array_equal(getattr(alb, op)(dg, 0.85, 3, **o)[0], want)
    else:
        outs, _ = getattr(alb, op)(gs, [0, 0], [5, 7], **o)
        for x, s in zip(outs, (5, 7)):
            assert np.array_equal(x, getattr(oracle, op[:-6])(g, s))


def test_automatic_grid_of_pull_pagerank_in_bins():
    """At most four waves per SIMD, however many edges ask for more."""
    import torch

    from paper_1911_09135_amd import alb

    n, m = 1 << 12, 1 << 28  # 2 * cbrt(m) = 1,290 workgroups
    off = (np.arange(n + 1, dtype=np.int64) * (m // n)).astype(np.int32)
    col = np.tile(np.arange(n, dtype=np.int32), m // n)
    with alb.Graph(off, col, build_transpose=True) as dg:
        del col
        for o in ({}, {"grid_wgs": alb.GRID_ALL}):
            _, st = alb.pagerank_pull(dg, 0.85, 1, mode="twc", **o)
            assert st["launched_threads"] <= 1024 * torch.cuda.get_device_properties(0).multi_processor_count
            assert st["edges_examined"] == m
