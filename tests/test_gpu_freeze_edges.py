"""Freezing (cm_freeze_stages) at the stage counts where its work split
changes -- threads per stage, rounds of 1,024 stages, LDS chunks of 2,048 keys
-- bit-exact against the oracle's rule, with ties, NaN and signed zeros."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("S", [1, 2, 15, 16, 17, 32, 33, 512, 513, 1024, 1025, 2048, 2049, 4100])
def test_freeze_stage_count_edges(oracle_mod, S):
    import torch
    import paper_2012_07145_amd as cm
    rng = np.random.default_rng(S)
    N, c = 3, 1
    v = rng.normal(size=(S, N))
    v = np.where(rng.random((S, N)) < 0.3, rng.choice([0.0, -0.0, 1.0, np.nan, np.inf], size=(S, N)),
                 v).astype(np.float32)
    z = torch.zeros(1, device="cuda")
    batch = cm.Batch([(S, N, 0, 0, 0, 0)], z, z, z)
    frozen = torch.full((S + 8,), 7, dtype=torch.uint8, device="cuda")
    cm.cm_freeze_stages(torch.from_numpy(v.ravel()).cuda(), batch,
                        torch.tensor([c], dtype=torch.int32, device="cuda"), 1, frozen)
    torch.cuda.synchronize()
    got = frozen.cpu().numpy()
    assert np.array_equal(got[:S], oracle_mod.freeze(v[:, c].astype(np.float64)))
    assert np.all(got[S:] == 7)
