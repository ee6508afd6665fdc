"""Push PageRank in tiles on handles without in-edges: the device lays them out
(edges into bins of destinations, each bin sorted).  Ranks against the bins'
path, which adds in another order but exactly, so the bits are the same."""
import numpy as np
import pytest

import graphgen as gg
import oracle
from test_pagerank_tiles_gpu import CASES, in_degrees

pytestmark = pytest.mark.gpu


def check(alb, dg, iterations):
    held = dg.device_bytes()
    bins, _ = alb.pagerank(dg, 0.85, iterations, threshold=64)
    one_ws = dg.device_bytes()
    x, st = alb.pagerank(dg, 0.85, iterations)
    assert dg.device_bytes() >= one_ws + 12 * dg.m and one_ws > held  # it did lay them out
    assert np.array_equal(x, bins)
    assert st["rounds"] == iterations and st["edges_examined"] == dg.m * iterations
    return x


@pytest.mark.parametrize("name", list(CASES))
def test_rows_of_the_tiles(name):
    from paper_1911_09135_amd import alb

    g = in_degrees(CASES[name], 5)
    with alb.Graph(g.off, g.col) as dg:
        x = check(alb, dg, 12)
    ref = oracle.pagerank(g, 0.85, 12)
    # every sum is exact, an fp32 rounding per contribution and per rank
    assert np.abs(x - ref).max() <= 13 * 4 * np.finfo(np.float32).eps * ref.max()


# destinations per bin: 64 up to 2^16 vertices, then as many as give 1,024 bins,
# 4,096 from 2^22 vertices on, up to 8,192 bins, then 8,192 destinations
@pytest.mark.parametrize("n", [63, 64, 65, 1 << 16, (1 << 16) + 1, (1 << 22) + 1, (1 << 22) + (3 << 18), 1 << 25,
                               (1 << 25) + 1])
def test_bins_of_destinations(n):
    from paper_1911_09135_amd import alb

    m = 300_000
    rng = np.random.default_rng(n)
    src = np.sort(rng.integers(0, n, m))
    col = rng.integers(0, n, m)
    col[::3] = n - 1  # a third of the edges in the last bin, on one vertex
    col[1::3] = rng.integers(n // 2, n // 2 + min(n // 2, 5000), col[1::3].size)
    off = np.searchsorted(src, np.arange(n + 1)).astype(np.int32)
    with alb.Graph(off, col.astype(np.int32)) as dg:
        check(alb, dg, 10)


def test_more_edges_than_one_group_of_steps():
    """Beyond 2^29 edges a workgroup scatters more than 2^20 of them."""
    from paper_1911_09135_amd import alb

    n, m = 1 << 16, 512 * ((1 << 20) + 600)
    off = (np.arange(n + 1, dtype=np.int64) * m // n).astype(np.int32)
    col = np.empty(m, np.int32)
    for a in range(0, m, 1 << 26):
        i = np.arange(a, min(a + (1 << 26), m), dtype=np.uint32)
        i *= np.uint32(2654435761)
        i >>= np.uint32(16)
        col[a:a + i.size] = i
    with alb.Graph(off, col) as dg:
        del col
        check(alb, dg, 2)
