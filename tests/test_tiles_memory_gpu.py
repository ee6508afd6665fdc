"""Device memory of PageRank in tiles: what a handle reports while calls run
beside each other."""
import threading

import numpy as np
import pytest

import graphgen as gg

pytestmark = pytest.mark.gpu


def run_together(calls):
    gate, errors = threading.Barrier(len(calls)), []

    def body(f):
        gate.wait()
        try:
            f()
        except Exception as e:  # seen by the test's thread
            errors.append(e)

    ts = [threading.Thread(target=body, args=(f,)) for f in calls]
    for t in ts:
        t.start()
    for t in ts:
        t.join()
    assert not errors, errors


def test_info_beside_first_calls():
    from paper_1911_09135_amd import alb

    g = gg.rmat(14, 8, seed=2)
    with alb.Graph(g.off, g.col) as dg:
        ref, _ = alb.pagerank(dg, 0.85, 12)
    for _ in range(5):
        with alb.Graph(g.off, g.col) as dg:
            bare, seen = dg.device_bytes(), []
            run_together([lambda: seen.append(alb.pagerank(dg, 0.85, 12)[0])] * 4 +
                         [lambda: [dg.device_bytes() for _ in range(200)]] * 2)
            assert all(np.array_equal(x, ref) for x in seen) and len(seen) == 4
            assert dg.device_bytes() > bare
