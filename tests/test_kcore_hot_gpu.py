"""k-core with hubs: neighbours of 1,024 edges or more are counted in an LDS
table of 1,024 slots before they are lowered.  Degrees on both sides of the
mark, more hubs than slots, hubs that leave the core by one decrement."""
import numpy as np
import pytest

import graphgen as gg
import oracle

pytestmark = pytest.mark.gpu


def hubs(n_hubs, leaves, deg, seed):
    """n_hubs hubs (a ring among themselves), `leaves` leaves with `deg` hub neighbours each."""
    rng = np.random.default_rng(seed)
    leaf = np.repeat(np.arange(leaves), deg)
    hub = (np.repeat(rng.integers(0, n_hubs, leaves), deg) + np.tile(np.arange(deg), leaves)) % n_hubs
    ring = np.arange(n_hubs)
    src = np.concatenate([leaf + n_hubs, ring])
    dst = np.concatenate([hub, (ring + 1) % n_hubs])
    return gg.undirected(n_hubs + leaves, src, dst)


@pytest.mark.parametrize("n_hubs,leaves,deg,ks", [
    (3, 1023, 1, [1, 2, 3]), (2, 2046, 1, [1, 2, 1022, 1024, 1025]), (1, 5000, 1, [1, 2]),
    (40, 60000, 3, [3, 4, 100, 4000]), (3000, 120000, 30, [30, 31, 33, 1000])])
def test_hot_neighbours(n_hubs, leaves, deg, ks):
    from paper_1911_09135_amd import alb

    g = hubs(n_hubs, leaves, min(deg, n_hubs), n_hubs)
    dg = alb.Graph.from_csr(g, symmetric=True)
    for k in ks:
        ref = oracle.kcore(g, k)
        for opts in ({}, {"wg_size": 64}, {"wg_size": 1024}, {"grid_wgs": 1}, {"mode": "twc"}, {"threshold": 64},
                     {"mode": "lb_all"}, {"launch": "host"}, {"visited_filter": True}):
            out, st = alb.kcore(dg, k, **opts)
            assert np.array_equal(out, ref), (k, opts)
            assert st["pushes"] + int((g.degrees() < k).sum()) == int((ref == 0).sum()), (k, opts)
    dg.close()
