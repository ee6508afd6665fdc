"""Worklist pushes at the edges of their LDS staging: a wavefront stages 1,024
vertex ids (512 pairs in a batch) and writes a full area out with a
reservation of its own; what is left at a phase's end goes out with one
reservation per workgroup."""
import numpy as np
import pytest

import graphgen as gg
import oracle

pytestmark = pytest.mark.gpu


def hub_then_pairs(d, seed):
    """Vertex 0 -> 1..d, and each of those -> one private second-level vertex, weights from the seed."""
    leaf = np.arange(1, d + 1)
    src = np.concatenate([np.zeros(d, np.int64), leaf])
    dst = np.concatenate([leaf, leaf + d])
    return gg.from_edges(2 * d + 1, src, dst).with_weights(seed)


@pytest.mark.parametrize("wg", [64, 256, 1024])
@pytest.mark.parametrize("grid", [1, 3])
@pytest.mark.parametrize("d", [1, 63, 511, 512, 513, 1023, 1024, 1025, 4097, 70001])
def test_staging_edges(d, grid, wg):
    import torch

    from paper_1911_09135_amd import alb

    g = hub_then_pairs(d, d)
    ref_b, ref_s = oracle.bfs(g, 0), oracle.sssp(g, 0)
    dg = alb.Graph.from_csr(g)
    out = torch.empty(g.n, dtype=torch.int32, device="cuda")
    for opts in ({"mode": "twc"}, {"threshold": 64}, {"mode": "lb_all"}, {"launch": "host"}):
        _, st = alb.bfs(dg, 0, out=out, wg_size=wg, grid_wgs=grid, **opts)
        assert np.array_equal(out.cpu().numpy(), ref_b), opts
        assert st["pushes"] == 2 * d and st["frontier_vertices"] == 2 * d + 1
        alb.sssp(dg, 0, out=out, wg_size=wg, grid_wgs=grid, **opts)
        assert np.array_equal(out.cpu().numpy(), ref_s), opts
    dg.close()
    gs = alb.GraphSet([g, g])
    outs, _ = alb.sssp_batch(gs, [0, 1, 0], [0, 0, 1], wg_size=wg, grid_wgs=grid)
    for o, ref in zip(outs, (ref_s, ref_s, oracle.sssp(g, 1))):
        assert np.array_equal(o, ref)
    gs.close()
