"""A call that fails leaves host outputs as they were, also where the launch
writes them itself (pinned memory)."""
import numpy as np
import pytest

import graphgen as gg
import oracle

pytestmark = pytest.mark.gpu


def outputs(graphs, members, pin):
    import torch

    return [torch.full((graphs[m].n,), -7, dtype=torch.int32, pin_memory=pin).numpy() for m in members]


@pytest.mark.parametrize("pin", [True, False])
@pytest.mark.parametrize("algo", ["bfs", "sssp"])
def test_overflowing_batches_and_plans(algo, pin):
    from paper_1911_09135_amd import alb

    graphs = [gg.rmat(12, 8, seed=1).with_weights(2), gg.rmat(14, 8, seed=3).with_weights(4)]
    gs = alb.GraphSet(graphs)
    members, sources = [0, 1, 1], [0, 0, 9]
    call = alb.bfs_batch if algo == "bfs" else alb.sssp_batch
    outs = outputs(graphs, members, pin)
    with pytest.raises(alb.AlbError) as e:
        call(gs, members, sources, outs=outs, worklist_capacity=16)
    assert e.value.status == alb.ALB_E_OVERFLOW
    plan = alb.BatchPlan(gs, algo, members, sources, outs=outs, worklist_capacity=16)
    for _ in range(2):
        with pytest.raises(alb.AlbError) as e:
            plan.run()
        assert e.value.status == alb.ALB_E_OVERFLOW
    plan.close()
    assert all((o == -7).all() for o in outs)
    call(gs, members, sources, outs=outs)  # and the next call is whole
    for o, m, s in zip(outs, members, sources):
        assert np.array_equal(o, getattr(oracle, algo)(graphs[m], s))
    gs.close()


@pytest.mark.parametrize("pin", [True, False])
def test_overflowing_queries(pin):
    from paper_1911_09135_amd import alb

    g = gg.undirected(3000, *np.random.default_rng(1).integers(0, 3000, (2, 40000))).with_weights(3)
    dg = alb.Graph(g.off, g.col, g.w, symmetric=True)
    (out,) = outputs([g], [0], pin)
    for call in (alb.bfs, alb.sssp):
        with pytest.raises(alb.AlbError) as e:
            call(dg, 0, out=out, worklist_capacity=8)
        assert e.value.status == alb.ALB_E_OVERFLOW
        assert (out == -7).all()
    dg.close()
