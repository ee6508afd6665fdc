"""Device memory of PageRank in tiles: what a handle reports while calls run
beside each other, and giving a kept layout back."""
import os
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


def test_kept_layouts_are_given_back_for_other_allocations():
    from paper_1911_09135_amd import alb

    g, h = gg.rmat(14, 8, seed=2), gg.rmat(12, 8, seed=3).with_weights(4)
    with alb.Graph(g.off, g.col) as dg, alb.Graph(g.off, g.col) as eg:
        alb.bfs(dg, 0)
        alb.bfs(eg, 0)
        before = dg.device_bytes()
        assert eg.device_bytes() == before
        ref, _ = alb.pagerank(dg, 0.85, 12)
        alb.pagerank(eg, 0.85, 12)
        held = dg.device_bytes()
        assert held >= before + 12 * g.m
        for _ in range(3):  # the layout serves later calls
            alb.pagerank(dg, 0.85, 12)
        assert dg.device_bytes() == held == eg.device_bytes()
        os.environ["ALB_INJECT_ALLOC_FAILURE"] = "tiles"  # no room while a layout is kept
        try:
            with alb.Graph(h.off, h.col, h.w) as other:
                alb.sssp(other, 0)
        finally:
            os.environ.pop("ALB_INJECT_ALLOC_FAILURE")
        assert dg.device_bytes() == before == eg.device_bytes()
        assert np.array_equal(alb.pagerank(dg, 0.85, 12)[0], ref)
        assert dg.device_bytes() == held
