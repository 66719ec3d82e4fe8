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
