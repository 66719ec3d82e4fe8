"""Float32 evaluator on the GPU at the edges of its work split: tiles of 16
candidates, stages shared by 8 waves, sums carried over chunks of 128 stages,
and more tiles than the grid's workgroups -- costs and per-stage costs against
the oracle.

Tolerance: a coefficient is a chain of at most 40 + 24 + 32 float32 fused
multiply-adds whose terms' magnitudes add up to at most about 20 for these
weights (hidden units of up to 10 against 32 weights of variance 1/32), so
its error stays below 96 * 2^-24 * 20 = 1.1e-4, and a stage's or query's cost
error below that times the sum of its cost terms.  The typical candidate is
held to 1e-6 relative.
"""
import numpy as np
import pytest

from synth import draw_query, model_params
from tests import gpucase as gc

pytestmark = pytest.mark.gpu

COEF_TOL, MEDIAN_TOL = 1.1e-4, 1e-6

SHAPES = [
    [(1, 1)], [(7, 15)], [(8, 16)], [(9, 17)],
    [(127, 16), (128, 17), (129, 33), (300, 5)],   # chunk edges, several queries
    [(2, 9700), (130, 20), (1, 31)],               # more tiles than workgroups
]


@pytest.mark.parametrize("shapes", SHAPES, ids=lambda s: "+".join(f"{a}x{b}" for a, b in s))
def test_fp32_split_edges(oracle_mod, shapes):
    import torch
    import paper_2012_07145_amd as cm
    rng = np.random.default_rng(sum(a * 7919 + b for a, b in shapes))
    params = model_params(bias=True)
    m = cm.cm_model_create(params)
    qs = [draw_query(rng, S, N) for S, N in shapes]
    ws = gc.workspace_for(cm, qs)
    batch, cost = cm.pack_queries(qs, "fp32")
    rows = sum(q.n_stages * q.n_cands for q in qs)
    stage = torch.full((rows + 4,), -7.0, device="cuda")
    cm.cm_eval_batch(m, "fp32", batch, ws, cost)
    plain = cost.clone()
    cost.fill_(-3.0)
    cm.cm_eval_stages(m, "fp32", batch, ws, cost, stage)
    torch.cuda.synchronize()
    assert torch.equal(plain, cost)
    assert (stage[rows:] == -7.0).all()
    c, st = cost.cpu().numpy(), stage.cpu().numpy()
    for q, d in zip(qs, batch.queries):
        S, N = q.n_stages, q.n_cands
        ref, refs = oracle_mod.eval_query(params, q.pipe, q.sched, q.terms, stage_costs=True)
        tsum = q.terms.astype(np.float64).sum(axis=2)
        got = st[d[4] // 8:d[4] // 8 + S * N].reshape(S, N).astype(np.float64)
        assert np.all(np.abs(got - refs) <= COEF_TOL * tsum), (S, N)
        mine = c[d[5]:d[5] + N].astype(np.float64)
        assert np.all(np.abs(mine - ref) <= COEF_TOL * tsum.sum(axis=0)), (S, N)
        assert np.median(gc.rel_err(mine, ref)) <= MEDIAN_TOL, (S, N)
    ws.close()


def _log_values():
    """Values of every exponent, ends and special values of float32, and runs of
    neighbours (among which are the roundings nearest to a tie)."""
    rng = np.random.default_rng(14)
    bits = [rng.integers(e << 23, (e + 1) << 23, 400) for e in range(1, 255)]
    for x in (2.0 ** -28, 2.0 ** -6, 0.5, 1.0, 3.0, 7.0, 15.0, 55.0, 63.0, 1e4, 65535.0, 2.0 ** 64):
        at = int(np.float32(x).view(np.uint32))
        bits.append(np.arange(at - 4000, at + 4000))
    bits.append([0, 0x80000000, 1, 0x007fffff, 0x7f7fffff, 0xbf000000, 0xbe000001, 0xbf7fffff,
                 0xbf800000, 0xc0000000, 0x7fc00000, 0xb8000000])
    v = np.concatenate([np.asarray(b, np.int64) for b in bits]).astype(np.uint32)
    return v.view(np.float32)


@pytest.mark.parametrize("mix", ["alone", "beside_plain", "beside_zero"])
def test_fp32_log_has_the_bits_of_log1pf(mix):
    """The logarithm of a schedule feature (short form and gathered log1pf)
    against that of an algorithm feature (log1pf), each routed to the stage's
    cost with unit weights: one value per stage, the same bits, whatever values
    are beside it in its wave."""
    import torch
    import paper_2012_07145_amd as cm
    from synth import Query
    from tests import cmcases as cc
    x = _log_values()
    S, N = x.size, 3
    sched = np.zeros((S, N, 40), np.float32)
    if mix == "beside_plain":
        sched[:] = np.exp(np.random.default_rng(3).normal(4.0, 2.0, (S, N, 40)))
    sched[:, 1, 0] = x
    terms = np.zeros((S, N, 8), np.float32)
    terms[:, :, 0] = 1.0
    got = {}
    for route in ("sched", "pipe"):
        pipe = np.zeros((S, 56), np.float32)
        if route == "pipe":
            pipe[:, 0] = x
        q = Query(pipe, sched if route == "sched" else np.zeros_like(sched), terms)
        if mix == "alone" and route == "sched":
            q.sched[:, 0], q.sched[:, 2] = -0.25, 1e6  # neighbours that log1pf takes
        m = cm.cm_model_create(cc.log_params(route))
        ws = gc.workspace_for(cm, [q])
        batch, cost = cm.pack_queries([q], "fp32")
        stage = torch.empty(S * N, device="cuda")
        cm.cm_eval_stages(m, "fp32", batch, ws, cost, stage)
        torch.cuda.synchronize()
        got[route] = stage.view(S, N)[:, 1].cpu().numpy()
        ws.close()
        m.close()
    same = got["sched"].view(np.uint32) == got["pipe"].view(np.uint32)
    same |= np.isnan(got["sched"]) & np.isnan(got["pipe"])
    assert np.all(same), (x[~same][:5], got["sched"][~same][:5], got["pipe"][~same][:5])


def test_fp32_log_has_the_bits_of_log1pf_for_every_feature_to_65536():
    """The same over every float32 from 0 to 65,536, which takes in all values of
    the short form: the logarithm of a schedule feature, routed to the cost,
    against that of an algorithm feature, routed to the hoisted row."""
    import torch
    import paper_2012_07145_amd as cm
    from tests import cmcases as cc
    end = 0x47800000
    n = 1 << 24
    sched, pipe = torch.zeros(n, 40, device="cuda"), torch.zeros(n, 56, device="cuda")
    terms = torch.zeros(n, 8, device="cuda")
    terms[:, 0] = 1.0
    cost, U = torch.empty(n, device="cuda"), torch.empty(n, 32, device="cuda")
    by_sched, by_pipe = (cm.cm_model_create(cc.log_params(r)) for r in ("sched", "pipe"))
    ws = cm.cm_workspace_create(1, 1, n, n, 1)
    zero_pipe = torch.zeros(56, device="cuda")
    one_stage = cm.Batch([(1, n, 0, 0, 0, 0)], zero_pipe, sched, terms)
    stages = cm.Batch([(n, 0, 0, 0, 0, 0)], pipe, sched, terms)
    for first in range(0, end, n):
        bits = torch.arange(first, first + n, dtype=torch.int32, device="cuda").clamp_(max=end)
        x = bits.view(torch.float32)
        sched[:, 0] = x
        pipe[:, 0] = x
        cm.cm_eval_batch(by_sched, "fp32", one_stage, ws, cost)
        cm.cm_hoist_stages(by_pipe, "fp32", stages, U)
        off = torch.nonzero(cost.view(torch.int32) != U[:, 0].contiguous().view(torch.int32))
        assert off.numel() == 0, (off.numel(), x[off[:5, 0]], cost[off[:5, 0]], U[off[:5, 0], 0])
    assert bits.max() == end and abs(float(cost.max()) - np.log(65537.0)) < 1e-5
    ws.close()
    by_sched.close()
    by_pipe.close()
    del sched, pipe, terms, U
    torch.cuda.empty_cache()
