"""Steps of up to 32 queries, whose descriptors go to the kernels by value,
and of more, which go through the slot's block: both equal the per-call path
bit for bit, at the edge between the two, in both precisions, with the step's
own hoist and with given rows, under either value of use_graph, and with slots
reused between batches of either kind."""
import numpy as np
import pytest

from synth import draw_query, model_params
from tests import gpucase as gc

pytestmark = pytest.mark.gpu

IN_SCALE = 16.0
K = 8


@pytest.fixture(scope="module")
def cm():
    import torch
    assert torch.cuda.is_available()
    import paper_2012_07145_amd as cm
    return cm


@pytest.fixture(scope="module")
def model(cm):
    m = cm.cm_model_create(model_params(bias=True))
    cm.cm_model_prepare_fp8(m, IN_SCALE, 8.0)
    yield m
    m.close()


def _queries(n, seed):
    rng = np.random.default_rng(seed)
    return [draw_query(rng, int(rng.integers(1, 40)), int(rng.integers(0, 90))) for _ in range(n)]


def _pack(cm, prec, queries):
    kw = {"in_scale": IN_SCALE} if prec == "fp8" else {}
    return cm.pack_queries(queries, prec, **kw)[0]


def _outs(batch):
    import torch
    n = batch.n_queries * K
    return (torch.full((max(1, batch.n_cands),), -5.0, device="cuda"),
            torch.full((n,), -7, dtype=torch.int32, device="cuda"),
            torch.full((n,), 7.0, device="cuda"))


def _per_call(cm, model, prec, batch, queries):
    import torch
    ws = gc.workspace_for(cm, queries, K)
    cost, idx, val = _outs(batch)
    cm.cm_eval_batch(model, prec, batch, ws, cost)
    cm.cm_topk_per_query(cost, batch, K, ws, idx, val)
    torch.cuda.synchronize()
    ws.close()
    return cost, idx, val


def _same(got, want, n):
    import torch
    torch.cuda.synchronize()
    assert torch.equal(got[0][:n].view(torch.int32), want[0][:n].view(torch.int32))
    assert torch.equal(got[1], want[1])
    assert torch.equal(got[2].view(torch.int32), want[2].view(torch.int32))


@pytest.mark.parametrize("graph", [1, 0])
@pytest.mark.parametrize("prec", ["bf16", "fp8"])
def test_step_by_value_and_by_block(cm, model, prec, graph):
    import torch
    sizes = [1, 31, 32, 33, 32, 40, 2]
    step = cm.cm_step_create(model, prec, max_queries=40, max_stages=2000, max_cands=8000,
                             max_k=K, slots=2)
    cm.cm_step_set_config(step, 0, 1, graph)
    for j, n in enumerate(sizes):
        queries = _queries(n, 50 + j)
        batch = _pack(cm, prec, queries)
        want = _per_call(cm, model, prec, batch, queries)
        U = torch.empty(sum(q.n_stages for q in queries) * 32, device="cuda")
        cm.cm_hoist_stages(model, prec, batch, U)
        for rows in (None, U):
            got = _outs(batch)
            cm.cm_step_run(step, batch, rows, K, *got)
            _same(got, want, batch.n_cands)
    step.close()


SPREAD_SHAPES = [
    [(1, 16)], [(3, 200)], [(4, 8192)], [(4, 8193)], [(5, 1)], [(8, 31)], [(16, 32)], [(17, 33)], [(32, 200)], [(33, 8192)], [(64, 8193)],
    [(64, 257)], [(65, 40)], [(20, 4100), (3, 60), (64, 0), (120, 33)], [(9, 0)],
    [(7 + 4 * j, 17 * j) for j in range(15)],
]


@pytest.mark.parametrize("prec", ["bf16", "fp8"])
@pytest.mark.parametrize("shapes", SPREAD_SHAPES, ids=lambda s: "x".join(map(str, s[0])))
def test_small_batches_spread_over_the_waves(cm, model, prec, shapes):
    """Batches of few row tiles, whose stages all waves of a workgroup share: the
    bits of the per-call path at the edges of the stage split, of the tiles and
    of the rule (256 tiles), beside queries that are not spread, and with
    several tiles per task."""
    import torch
    rng = np.random.default_rng(77)
    queries = [draw_query(rng, S, N) for S, N in shapes]
    batch = _pack(cm, prec, queries)
    want = _per_call(cm, model, prec, batch, queries)
    step = cm.cm_step_create(model, prec, max_queries=len(queries),
                             max_stages=sum(S for S, _ in shapes),
                             max_cands=max(1, sum(N for _, N in shapes)), max_k=K, slots=2)
    for tiles in (1, 2, 8):
        cm.cm_step_set_config(step, 0, tiles, 1)
        got = _outs(batch)
        cm.cm_step_run(step, batch, None, K, *got)
        _same(got, want, batch.n_cands)
    step.close()
