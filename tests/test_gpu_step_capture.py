"""A step recorded by a stream under capture: every replay runs the batch that
was recorded, whatever other batches the step has run since on the same slots,
and recording takes nothing from the step's later runs."""
import numpy as np
import pytest

from synth import draw_query, model_params
from tests import gpucase as gc

pytestmark = pytest.mark.gpu

K = 8


def _queries(n, seed):
    rng = np.random.default_rng(seed)
    return [draw_query(rng, int(rng.integers(1, 40)), int(rng.integers(0, 90))) for _ in range(n)]


def _outs(batch):
    import torch
    n = batch.n_queries * K
    return (torch.full((max(1, batch.n_cands),), -5.0, device="cuda"),
            torch.full((n,), -7, dtype=torch.int32, device="cuda"),
            torch.full((n,), 7.0, device="cuda"))


def _per_call(cm, model, prec, batch, queries):
    import torch
    ws = gc.workspace_for(cm, queries, K)
    out = _outs(batch)
    cm.cm_eval_batch(model, prec, batch, ws, out[0])
    cm.cm_topk_per_query(out[0], batch, K, ws, out[1], out[2])
    torch.cuda.synchronize()
    ws.close()
    return out


def _same(got, want):
    import torch
    torch.cuda.synchronize()
    for g, w in zip(got, want):
        assert torch.equal(g.view(torch.int32), w.view(torch.int32))


@pytest.mark.parametrize("own_hoist", [True, False])
@pytest.mark.parametrize("n", [1, 32, 33, 70, 256])  # by value; one, several and many parts of a block
@pytest.mark.parametrize("prec", ["bf16", "fp8"])
def test_recorded_step_replays_its_own_batch(prec, n, own_hoist):
    import torch
    import paper_2012_07145_amd as cm
    model = cm.cm_model_create(model_params(bias=True))
    kw = {}
    if prec == "fp8":
        cm.cm_model_prepare_fp8(model, 16.0, 8.0)
        kw = {"in_scale": 16.0}
    step = cm.cm_step_create(model, prec, max_queries=256, max_stages=12000, max_cands=30000,
                             max_k=K, slots=2)
    batches = []
    for size, seed in ((n, 1), (40, 2), (256, 3), (3, 4)):
        qs = _queries(size, seed)
        b = cm.pack_queries(qs, prec, **kw)[0]
        batches.append((b, _outs(b), _per_call(cm, model, prec, b, qs)))
    rec, rec_out, rec_want = batches[0]
    U = None
    if not own_hoist:
        U = torch.empty(sum(q[0] for q in rec.queries) * 32, device="cuda")
        cm.cm_hoist_stages(model, prec, rec, U)

    def others():
        # every slot, with batches of both kinds
        for b, out, want in batches[1:] + batches[1:]:
            cm.cm_step_run(step, b, None, K, *out)
            _same(out, want)
            assert cm.cm_step_kernel_time(step) > 0

    others()
    torch.cuda.synchronize()
    graph, stream = torch.cuda.CUDAGraph(), torch.cuda.Stream()
    with torch.cuda.graph(graph, stream=stream):
        cm.cm_step_run(step, rec, U, K, *rec_out, stream=torch.cuda.current_stream())
    assert int(rec_out[1][0]) == -7  # recorded, not run
    for _ in range(3):
        others()
        for out, sentinel in zip(rec_out, (-5.0, -7, 7.0)):
            out.fill_(sentinel)
        graph.replay()
        _same(rec_out, rec_want)
    # a second recording, with runs still in flight while it is made
    cm.cm_step_run(step, batches[2][0], None, K, *batches[2][1])
    cm.cm_step_run(step, batches[1][0], None, K, *batches[1][1])
    graph2 = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph2, stream=stream):
        cm.cm_step_run(step, rec, U, K, *rec_out, stream=torch.cuda.current_stream())
    for g in (graph2, graph):
        others()
        for out in rec_out:
            out.zero_()
        g.replay()
        _same(rec_out, rec_want)
    step.close()
    model.close()
