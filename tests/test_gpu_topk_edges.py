"""Beam selection (cm_topk_per_query) at the edges of its work split -- waves,
the sizes at which the threshold starts, tiles of both workgroup sizes, merge
rounds -- for costs in orders that defeat the threshold; bit-exact against the
oracle's selection."""
import numpy as np
import pytest

from tests import gpucase as gc

pytestmark = pytest.mark.gpu

SIZES = [0, 1, 63, 64, 65, 255, 256, 257, 300, 1023, 1024, 1025, 2000, 4096, 4097, 16383, 16384,
         16385, 33000]


def _costs(kind, n, rng):
    if kind == "random":
        return rng.lognormal(8, 1, n).astype(np.float32)
    if kind == "ascending":
        return np.arange(n, dtype=np.float32)
    if kind == "descending":
        return -np.arange(n, dtype=np.float32)
    if kind == "equal":
        return np.full(n, 3.5, np.float32)
    c = rng.choice([0.0, -0.0, 1.0, -1.0, np.nan, np.inf, -np.inf, 3.4e38, -3.4e38, 1e-45], size=n)
    return c.astype(np.float32)


@pytest.mark.parametrize("k", [1, 2, 32, 33, 200, 256])
@pytest.mark.parametrize("kind", ["random", "ascending", "descending", "equal", "special"])
def test_topk_edges(oracle_mod, kind, k):
    import torch
    import paper_2012_07145_amd as cm
    rng = np.random.default_rng(k)
    z = torch.zeros(1, device="cuda")
    # every size alone (its own workgroup size), then all in one batch
    for sizes in [[n] for n in SIZES] + [SIZES]:
        costs = [_costs(kind, n, rng) for n in sizes]
        descs, off = [], 0
        for c in costs:
            descs.append((1, c.size, 0, 0, 0, off))
            off += c.size
        flat = torch.from_numpy(np.concatenate(costs + [np.zeros(1, np.float32)])).cuda()
        idx, val = gc.gpu_topk(cm, flat, cm.Batch(descs, z, z, z), k)
        for j, c in enumerate(costs):
            gc.assert_select_bit_exact(oracle_mod, c, idx[j], val[j], k)


def test_topk_many_merge_rounds(oracle_mod):
    """200 tiles of 16,384: their lists take several merge rounds at k = 256."""
    import torch
    import paper_2012_07145_amd as cm
    rng = np.random.default_rng(9)
    z = torch.zeros(1, device="cuda")
    n = 200 * 16384 + 5
    for c in (rng.lognormal(8, 1, n).astype(np.float32), -np.arange(n, dtype=np.float32)):
        idx, val = gc.gpu_topk(cm, torch.from_numpy(c).cuda(),
                               cm.Batch([(1, n, 0, 0, 0, 0)], z, z, z), 256)
        gc.assert_select_bit_exact(oracle_mod, c, idx[0], val[0], 256)


def _ordered_costs(kind, n, rng):
    e = np.arange(n)
    if kind == "columns of 1024":      # few threads hold all the smallest: 16 each
        return ((e % 1024) * 16 + e // 1024 % 16).astype(np.float32)
    if kind == "columns of 512":
        return ((e % 512) * 32 + e // 512 % 32).astype(np.float32)
    if kind == "blocks":               # whole waves of the smallest, last
        return (-(e // 64)).astype(np.float32)
    if kind == "three values":
        return rng.integers(0, 3, n).astype(np.float32)
    if kind == "one below":            # all equal but the last
        return np.where(e == n - 1, 1.0, 2.0).astype(np.float32)
    return np.where(rng.random(n) < 0.02, rng.random(n), np.inf).astype(np.float32)


@pytest.mark.parametrize("k", [1, 31, 64, 256])
@pytest.mark.parametrize("kind", ["columns of 1024", "columns of 512", "blocks", "three values",
                                  "one below", "mostly infinite"])
def test_topk_of_ordered_and_equal_costs(oracle_mod, kind, k):
    """Costs for which the first threshold lets too many pass, some of which the
    second does not thin out either."""
    import torch
    import paper_2012_07145_amd as cm
    rng = np.random.default_rng(k)
    z = torch.zeros(1, device="cuda")
    sizes = [k + 255, k + 256, k + 257, 2 * k + 1, 1000, 4096, 9000, 16384, 40000]
    costs = [_ordered_costs(kind, n, rng) for n in sizes]
    descs, off = [], 0
    for c in costs:
        descs.append((1, c.size, 0, 0, 0, off))
        off += c.size
    flat = torch.from_numpy(np.concatenate(costs)).cuda()
    idx, val = gc.gpu_topk(cm, flat, cm.Batch(descs, z, z, z), k)
    for j, c in enumerate(costs):
        gc.assert_select_bit_exact(oracle_mod, c, idx[j], val[j], k)


@pytest.mark.parametrize("k", [1, 32, 256])
@pytest.mark.parametrize("kind", ["columns of 1024", "columns of 512", "blocks", "three values",
                                  "one below"])
def test_step_of_ordered_and_equal_costs(oracle_mod, kind, k):
    """The same costs out of the persistent step's evaluation: one stage, equal
    features, terms in the order of the kind."""
    import torch
    import paper_2012_07145_amd as cm
    from synth import Query, model_params
    rng = np.random.default_rng(k)
    queries = []
    for n in (300, 2 * k + 257, 1000, 4096, 9000):
        c = _ordered_costs(kind, n, rng)
        terms = np.repeat((c - c.min() + 1)[None, :, None], 8, axis=2).astype(np.float32)
        queries.append(Query(np.ones((1, 56), np.float32), np.full((1, n, 40), 3.0, np.float32),
                             terms))
    model = cm.cm_model_create(model_params(bias=True))
    batch, cost = cm.pack_queries(queries, "bf16")
    step = cm.cm_step_create(model, "bf16", max_queries=5, max_stages=5, max_cands=cost.numel(),
                             max_k=k)
    idx = torch.zeros(5 * k, dtype=torch.int32, device="cuda")
    val = torch.zeros(5 * k, device="cuda")
    cm.cm_step_run(step, batch, None, k, cost, idx, val)
    torch.cuda.synchronize()
    got, i, v = cost.cpu().numpy(), idx.cpu().numpy(), val.cpu().numpy()
    for j, d in enumerate(batch.queries):
        c = got[d[5]:d[5] + d[1]]
        order = np.argsort(queries[j].terms[0, :, 0], kind="stable")
        assert c.min() > 0 and np.all(np.diff(c[order]) >= 0)
        gc.assert_select_bit_exact(oracle_mod, c, i[j * k:(j + 1) * k], v[j * k:(j + 1) * k], k)
    step.close()
    model.close()
