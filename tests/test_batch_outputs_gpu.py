"""Host outputs of a batch that share memory: the queries' results are written
in their order, so the last query's stay, whether the memory is pinned or not."""
import numpy as np
import pytest

import graphgen as gg
import oracle

pytestmark = pytest.mark.gpu


def host(n, pin):
    import torch

    return torch.full((n,), -7, dtype=torch.int32, pin_memory=pin).numpy()


@pytest.mark.parametrize("pin", [True, False])
@pytest.mark.parametrize("plan", [False, True])
def test_shared_outputs_keep_the_last_query(pin, plan):
    from paper_1911_09135_amd import alb

    g = gg.rmat(15, 8, seed=4).with_weights(5)
    n = g.n
    gs = alb.GraphSet([g])
    sources = [int(v) for v in np.flatnonzero(g.degrees() > 0)[[0, 50, 400, 900, 1500, 2200, 3100]]]
    refs = [oracle.sssp(g, s) for s in sources]
    block = host(4 * n, pin)
    want = np.full(4 * n, -7, np.int32)
    # one array three times, an array that overlaps it, two that only touch, one apart
    at = [0, 0, n // 2, 0, 2 * n, 3 * n, n + n // 2]
    for a, ref in zip(at, refs):
        want[a:a + n] = ref
    outs = [block[a:a + n] for a in at]
    if plan:
        p = alb.BatchPlan(gs, "sssp", [0] * len(at), sources, outs=outs)
        for _ in range(3):
            block[:] = -7
            p.run()
            assert np.array_equal(block, want)
        p.close()
    else:
        alb.sssp_batch(gs, [0] * len(at), sources, outs=outs)
        assert np.array_equal(block, want)
    gs.close()


@pytest.mark.parametrize("n", [(1 << 18) - 1, 1 << 18, (1 << 18) + 1])
@pytest.mark.parametrize("plan", [False, True])
def test_outputs_around_the_size_that_is_written(n, plan):
    """Beside other batches the launch writes pinned outputs of up to 2^18 vertices only."""
    from paper_1911_09135_amd import alb

    rng = np.random.default_rng(n)
    big = gg.from_edges(n, rng.integers(0, n, 4 * n), rng.integers(0, n, 4 * n), rng.integers(1, 9, 4 * n))
    small = gg.rmat(9, 8, seed=1).with_weights(2)
    gs = alb.GraphSet([big, small])
    members, sources = [0, 1, 0], [0, 0, n - 1]
    outs = [host(n, True), host(small.n, True), host(n, False)]
    refs = [oracle.sssp((big, small)[m], s) for m, s in zip(members, sources)]
    p = alb.BatchPlan(gs, "sssp", members, sources, outs=outs) if plan else None
    for _ in range(2):
        for o in outs:
            o[:] = -7
        p.run() if plan else alb.sssp_batch(gs, members, sources, outs=outs)
        assert all(np.array_equal(o, ref) for o, ref in zip(outs, refs))
    if plan:
        p.close()
    gs.close()


def test_large_outputs_beside_other_batches():
    """Two threads' batches and plans on one set, members beyond 2^18 vertices."""
    import threading

    from paper_1911_09135_amd import alb

    n = (1 << 18) + 77
    rng = np.random.default_rng(1)
    g = gg.from_edges(n, rng.integers(0, n, 4 * n), rng.integers(0, n, 4 * n), rng.integers(1, 9, 4 * n))
    gs = alb.GraphSet([g])
    refs = {s: oracle.sssp(g, s) for s in (0, 5, n - 1)}
    bad = []

    def work(sources, plan):
        import torch

        stream = torch.cuda.Stream()
        outs = [host(n, True) for _ in sources]
        p = alb.BatchPlan(gs, "sssp", [0] * len(sources), sources, outs=outs, stream=stream) if plan else None
        for _ in range(8):
            for o in outs:
                o[:] = -7
            p.run() if plan else alb.sssp_batch(gs, [0] * len(sources), sources, outs=outs, stream=stream)
            bad.extend(s for o, s in zip(outs, sources) if not np.array_equal(o, refs[s]))
        if plan:
            p.close()

    threads = [threading.Thread(target=work, args=a) for a in (([0, 5], False), ([n - 1], False), ([5, 0], True))]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not bad
    gs.close()
