"""Per-call evaluation at the edge between launches that pass descriptors of up
to 8 queries and of up to 32: every query's costs and stage costs equal, bit for
bit, those of the query evaluated alone."""
import numpy as np
import pytest

from synth import draw_query, model_params
from tests import gpucase as gc

pytestmark = pytest.mark.gpu


def _costs(cm, model, prec, queries):
    import torch
    kw = {"in_scale": 16.0} if prec == "fp8" else {}
    batch, cost = cm.pack_queries(queries, prec, **kw)
    ws = gc.workspace_for(cm, queries)
    stage = torch.zeros(sum(q.n_stages * q.n_cands for q in queries), device="cuda")
    cm.cm_eval_batch(model, prec, batch, ws, cost)
    plain = cost.clone()
    cm.cm_eval_stages(model, prec, batch, ws, cost, stage)
    torch.cuda.synchronize()
    ws.close()
    n = sum(q.n_cands for q in queries)
    return [t.view(torch.int32).cpu().numpy() for t in (plain[:n], cost[:n], stage)]


@pytest.mark.parametrize("prec", ["fp32", "bf16", "fp8"])
@pytest.mark.parametrize("n", [7, 8, 9, 33])
def test_queries_of_a_batch_equal_the_query_alone(prec, n):
    import torch
    assert torch.cuda.is_available()
    import paper_2012_07145_amd as cm
    rng = np.random.default_rng(n)
    queries = [draw_query(rng, int(rng.integers(1, 70)), int(rng.integers(1, 80)))
               for _ in range(n)]
    model = cm.cm_model_create(model_params(bias=True))
    cm.cm_model_prepare_fp8(model, 16.0, 8.0)
    together = _costs(cm, model, prec, queries)
    alone = [_costs(cm, model, prec, [q]) for q in queries]
    for j in range(3):
        assert np.array_equal(together[j], np.concatenate([a[j] for a in alone]))
    model.close()


SPREAD_SHAPES = [
    [(5, 1)], [(8, 31)], [(16, 32)], [(17, 33)], [(32, 200)], [(33, 8192)], [(64, 8193)],
    [(64, 257)], [(65, 40)], [(20, 4100), (3, 60), (64, 0), (120, 33)], [(9, 1), (8, 0)],
    [(7 + 4 * j, 17 * j) for j in range(15)],
]


@pytest.mark.parametrize("prec", ["bf16", "fp8"])
@pytest.mark.parametrize("shapes", SPREAD_SHAPES, ids=lambda s: "x".join(map(str, s[0])))
def test_small_calls_spread_over_the_waves(prec, shapes):
    """Calls of few row tiles, whose stages all waves of a workgroup share, against
    the form with stage costs, which never does: the same bits, at the edges of
    the stage split, of the tiles and of the rule (256 tiles)."""
    import torch
    assert torch.cuda.is_available()
    import paper_2012_07145_amd as cm
    rng = np.random.default_rng(78)
    queries = [draw_query(rng, S, N) for S, N in shapes]
    model = cm.cm_model_create(model_params(bias=True))
    cm.cm_model_prepare_fp8(model, 16.0, 8.0)
    plain, with_stages, _ = _costs(cm, model, prec, queries)
    assert np.array_equal(plain, with_stages)
    model.close()
