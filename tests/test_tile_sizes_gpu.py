"""Tiles of PageRank sized by the graph: one of 512 to 2,048 rows and in-edges
per workgroup, or as many equal ones of up to 4,096 on each.  Graphs on both
sides of every line, ranks against the bins' path (the same bits)."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

HELD = 1024  # workgroups of the tiles on 256 CUs


@pytest.mark.parametrize("items", [320 * 512, 320 * 512 + 1, 320 * 1024 + 1, 320 * 1792, 320 * 1792 + 1, HELD * 2048,
                                   HELD * 2048 + 1, HELD * 4096, HELD * 4096 + 1, HELD * 8192 + 1])
def test_tile_sizes(items):
    from paper_1911_09135_amd import alb

    n = items // 5
    m = items - n
    rng = np.random.default_rng(items)
    src = np.sort(rng.integers(0, n, m))
    col = rng.integers(0, n, m)
    col[rng.integers(0, m, m // 10)] = n // 3  # a row over many tiles
    col[rng.integers(0, m, m // 50)] = n - 1
    off = np.searchsorted(src, np.arange(n + 1)).astype(np.int32)
    with alb.Graph(off, col.astype(np.int32), build_transpose=True) as dg:
        for it in (1, 4):
            bins, _ = alb.pagerank_pull(dg, 0.85, it, threshold=64)
            for call in (alb.pagerank_pull, alb.pagerank):
                x, st = call(dg, 0.85, it)
                assert np.array_equal(x, bins), (call, it)
                assert st["edges_examined"] == m * it
