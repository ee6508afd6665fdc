"""Launches whose grid is small for the graph's vertices: labels are set up and
results written by kernels of their own, beyond 24 vertices a thread (BFS: 96, k-core: 12).
Both sides of the line, repeated calls in turn with calls of the other kind,
every kind of output."""
import numpy as np
import pytest

import graphgen as gg
import oracle

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [12 * 256, 12 * 256 + 1, 24 * 256, 24 * 256 + 1, 96 * 256, 96 * 256 + 1, 70_001])
def test_both_sides_of_the_line(n):
    import torch

    from paper_1911_09135_amd import alb

    rng = np.random.default_rng(n)
    g = gg.undirected(n, rng.integers(0, n, 2 * n), rng.integers(0, n, 2 * n)).with_weights(3)
    dg = alb.Graph(g.off, g.col, g.w, symmetric=True)
    pin = torch.empty(n, dtype=torch.int32, pin_memory=True)
    dev = torch.empty(n, dtype=torch.int32, device="cuda")
    refs = {"bfs": oracle.bfs(g, 7), "sssp": oracle.sssp(g, 7), "cc": oracle.cc(g), "kcore": oracle.kcore(g, 3)}
    calls = {"bfs": lambda **o: alb.bfs(dg, 7, **o), "sssp": lambda **o: alb.sssp(dg, 7, **o),
             "cc": lambda **o: alb.cc(dg, **o), "kcore": lambda **o: alb.kcore(dg, 3, **o)}
    for grid in (1, 0, 1, 1, 2):
        for name, call in calls.items():
            for opts in ({}, {"visited_filter": True}, {"mode": "twc"}, {"threshold": 64}):
                for out in (None, pin.numpy(), dev):
                    if out is not None:
                        out[:] = -7
                    got, st = call(out=out, grid_wgs=grid, **opts)
                    got = got.cpu().numpy() if out is dev else got
                    assert np.array_equal(got, refs[name]), (grid, name, opts)
                    assert st["device_ms"] >= st["kernel_ms"] > 0
        dev.fill_(-7)
        alb.sssp_noalloc(dg, 7, dev, grid_wgs=grid)
        assert np.array_equal(dev.cpu().numpy(), refs["sssp"])
    with pytest.raises(alb.AlbError) as e:  # a launch that failed, then a whole one
        alb.sssp(dg, 7, out=pin.numpy(), grid_wgs=1, worklist_capacity=4)
    assert e.value.status == alb.ALB_E_OVERFLOW
    assert np.array_equal(calls["sssp"](grid_wgs=1)[0], refs["sssp"])
    dg.close()


def test_few_edges_over_many_vertices():
    from paper_1911_09135_amd import alb

    n, m = 3_000_000, 2000
    rng = np.random.default_rng(2)
    g = gg.undirected(n, rng.integers(0, 900, m), rng.integers(0, 900, m)).with_weights(3)
    dg = alb.Graph(g.off, g.col, g.w, symmetric=True)
    assert np.array_equal(alb.sssp(dg, 5)[0], oracle.sssp(g, 5))
    assert np.array_equal(alb.bfs(dg, 5)[0], oracle.bfs(g, 5))
    assert np.array_equal(alb.cc(dg)[0], oracle.cc(g))
    assert np.array_equal(alb.kcore(dg, 3)[0], oracle.kcore(g, 3))
    dg.close()
