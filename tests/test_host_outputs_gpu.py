"""Host outputs that the launch writes itself: pinned arrays (also views into
one, and sizes around the staged ones) and pageable ones, for single queries,
batches and plans."""
import numpy as np
import pytest

import graphgen as gg
import oracle

pytestmark = pytest.mark.gpu


def pinned(n, dtype, lead=0):
    import torch

    t = torch.empty(n + lead, dtype=dtype, pin_memory=True)
    t.fill_(-7)
    return t.numpy()[lead:]


@pytest.mark.parametrize("n", [1, 2, 1000, 65535, 65536, 65537, 200001])
def test_single_queries(n):
    import torch

    from paper_1911_09135_amd import alb

    rng = np.random.default_rng(n)
    g = gg.undirected(n, rng.integers(0, n, 4 * n), rng.integers(0, n, 4 * n)).with_weights(3)
    dg = alb.Graph(g.off, g.col, g.w, symmetric=True, build_transpose=True)
    refs = {"bfs": oracle.bfs(g, 0), "sssp": oracle.sssp(g, 0), "cc": oracle.cc(g), "kcore": oracle.kcore(g, 4)}
    calls = {"bfs": lambda o: alb.bfs(dg, 0, out=o), "sssp": lambda o: alb.sssp(dg, 0, out=o),
             "cc": lambda o: alb.cc(dg, out=o), "kcore": lambda o: alb.kcore(dg, 4, out=o)}
    for name, call in calls.items():
        for out in (None, np.full(n, -7, np.int32), pinned(n, torch.int32), pinned(n, torch.int32, 3)):
            assert np.array_equal(call(out)[0], refs[name]), name
    on_device = torch.empty(n, dtype=torch.float32, device="cuda")
    for call in (alb.pagerank, alb.pagerank_pull):
        want = call(dg, 0.85, 12, out=on_device)[0].cpu().numpy()
        for out in (None, np.empty(n, np.float32), pinned(n, torch.float32), pinned(n, torch.float32, 5)):
            assert np.array_equal(call(dg, 0.85, 12, out=out)[0], want)
    dg.close()


def test_batches_and_plans_mix_outputs():
    import torch

    from paper_1911_09135_amd import alb

    graphs = [gg.rmat(s, 8, seed=s).with_weights(s) for s in (6, 9, 11)]
    gs = alb.GraphSet(graphs)
    members, sources = [0, 1, 2, 2, 1], [0, 0, 0, 5, 3]
    refs = [oracle.sssp(graphs[m], s) for m, s in zip(members, sources)]

    def outputs():
        made = [pinned(graphs[0].n, torch.int32), np.full(graphs[1].n, -7, np.int32)]
        made += [pinned(graphs[2].n, torch.int32, 3), np.full(graphs[2].n, -7, np.int32)]
        return made + [pinned(graphs[1].n, torch.int32)]

    for o, ref in zip(alb.sssp_batch(gs, members, sources, outs=outputs())[0], refs):
        assert np.array_equal(o, ref)
    plan = alb.BatchPlan(gs, "sssp", members, sources, outs=outputs())
    for _ in range(3):
        for o in plan.outs:
            o[:] = -7
        for o, ref in zip(plan.run()[0], refs):
            assert np.array_equal(o, ref)
        alb.bfs_batch(gs, [0, 1], [0, 0])  # other work between the replays
    plan.close()
    gs.close()
