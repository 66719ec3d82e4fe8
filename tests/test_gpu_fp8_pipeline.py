"""FP8 evaluator: the load pipeline of three buffers (per call and in the
persistent step) at every remainder of its loop and of its chunks of staged
rows gives the bits of the two-buffer form that per-stage costs take, and of
the oracle's form within its bound elsewhere."""
import numpy as np
import pytest

from synth import draw_query, model_params
from tests import gpucase as gc

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N", [1, 33, 300])
def test_three_buffers_equal_two(oracle_mod, N):
    import torch
    import paper_2012_07145_amd as cm
    rng = np.random.default_rng(N)
    m = cm.cm_model_create(model_params(bias=True))
    cm.cm_model_prepare_fp8(m, 16.0, 8.0)
    # stages per part 1 .. 16 and more than one chunk of rows in a part
    qs = [draw_query(rng, S, N) for S in list(range(1, 19)) + [30, 31, 32, 33, 61, 64, 65, 120, 128,
                                                               129, 250]]
    codes = [oracle_mod.fp8_codes(q.sched, 16.0) for q in qs]
    codes[3].reshape(-1)[5] = 0x7F  # a NaN input
    batch, cost = gc.pack_fp8(cm, qs, codes)
    ws = gc.workspace_for(cm, qs)
    cm.cm_eval_batch(m, "fp8", batch, ws, cost)
    staged = torch.zeros_like(cost)
    stage = torch.empty(sum(q.n_stages * N for q in qs), device="cuda")
    cm.cm_eval_stages(m, "fp8", batch, ws, staged, stage)
    step = cm.cm_step_create(m, "fp8", max_queries=len(qs), max_stages=sum(q.n_stages for q in qs),
                             max_cands=N * len(qs), max_k=8)
    stepped = torch.zeros_like(cost)
    idx = torch.empty(len(qs) * 8, dtype=torch.int32, device="cuda")
    val = torch.empty(len(qs) * 8, device="cuda")
    for _ in range(3):
        stepped.zero_()
        cm.cm_step_run(step, batch, None, 8, stepped, idx, val)
        torch.cuda.synchronize()
        assert torch.equal(stepped.view(torch.int32), cost.view(torch.int32))
    assert torch.equal(staged.view(torch.int32), cost.view(torch.int32))
    assert torch.isnan(cost).sum() == 1
    ws.close()
    step.close()
    m.close()
