"""PageRank in tiles of 4,096 rows and in-edges, merged: rows that end on a
tile's edge, rows longer than a tile and than a workgroup's run of tiles,
stretches of rows without in-edges, sizes around one tile."""
import numpy as np
import pytest

import graphgen as gg
import oracle

pytestmark = pytest.mark.gpu


def in_degrees(deg, seed):
    """A graph whose vertex v has deg[v] in-edges from vertices spread over all."""
    deg = np.asarray(deg, np.int64)
    n = deg.size
    rng = np.random.default_rng(seed)
    dst = np.repeat(np.arange(n), deg)
    start = rng.integers(0, n, n)
    first = np.cumsum(deg) - deg
    src = (np.repeat(start, deg) + np.arange(dst.size) - np.repeat(first, deg)) % n
    off = np.zeros(n + 1, np.int64)
    np.add.at(off, src + 1, 1)
    order = np.argsort(src, kind="stable")
    return gg.Graph(n, np.cumsum(off).astype(np.int32), dst[order].astype(np.int32))


CASES = {
    "one": [0], "loop": [1], "short_tile": [1] * 2047, "full_tile": [1] * 2048, "tile_and_one": [1] * 2049,
    "edge_at_tile_end": [4095] + [0] * 5000, "row_of_a_tile": [4096] + [0] * 4999 + [1],
    "empty_tiles": [0] * 9000 + [3] * 10 + [0] * 9000, "long_rows": [0, 9000, 1, 9500, 0, 0, 9999] + [1] * 9993,
    "hubs_apart": ([20000] + [2] * 3000) * 2 + [0] * 15000,
}


@pytest.mark.parametrize("name", list(CASES))
@pytest.mark.parametrize("iterations", [1, 2, 7])
def test_tiles_against_the_bins(name, iterations):
    from paper_1911_09135_amd import alb

    g = in_degrees(CASES[name], 5)
    dg = alb.Graph(g.off, g.col, build_transpose=True)
    plain = alb.Graph(g.off, g.col)
    ref = oracle.pagerank(g, 0.85, iterations)
    bins, bst = alb.pagerank_pull(dg, 0.85, iterations, threshold=64)
    for h, call in ((dg, alb.pagerank_pull), (dg, alb.pagerank), (plain, alb.pagerank)):
        x, st = call(h, 0.85, iterations)
        assert np.array_equal(x, bins), call
        assert st["rounds"] == iterations and st["edges_examined"] == g.m * iterations
        assert st["frontier_vertices"] == g.n * iterations
    # every sum is exact, an fp32 rounding per contribution and per rank
    assert np.abs(bins - ref).max() <= (iterations + 1) * 4 * np.finfo(np.float32).eps * ref.max()
    dg.close()
    plain.close()
