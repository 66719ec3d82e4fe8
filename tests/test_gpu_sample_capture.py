"""cm_sample_buckets recorded by a stream under capture: a replay draws for the
batch that was recorded, whatever the sampler has been called with since, and
recording takes nothing from the sampler's later calls.  Bit-exact against the
oracle."""
import numpy as np
import pytest

from tests.test_gpu_sample import bucket_hashes, check, run

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nq,top", [(3, 900), (3, 5000), (65, 900), (65, 3000), (300, 2000)])
def test_recorded_sampling_replays_its_own_batch(oracle_mod, nq, top):
    import torch
    import paper_2012_07145_amd as cm
    rng = np.random.default_rng(nq + top)

    def draw(n, most):
        hs = [bucket_hashes(rng, int(rng.integers(1, most + 1))) for _ in range(n)]
        hs[0] = bucket_hashes(rng, most)
        return hs, rng.integers(0, 2 ** 64, n, dtype=np.uint64)

    rec, rec_seeds = draw(nq, top)
    others = [draw(5, 4000), draw(80, 1000), draw(130, 2500)]
    total = max(sum(h.size for h in hs) for hs, _ in [(rec, 0)] + others)
    sp = cm.cm_sampler_create(300, total)

    def call_others():
        for hs, seeds in others:
            sel, cnt, descs = run(cm, sp, hs, seeds)
            check(oracle_mod, hs, seeds, sel, cnt, descs)

    descs, off = [], 0
    for h in rec:
        descs.append((1, h.size, 0, 0, 0, off))
        off += h.size
    z = torch.zeros(1, device="cuda")
    batch = cm.Batch(descs, z, z, z)
    hashes = torch.from_numpy(np.concatenate(rec).view(np.int64).copy()).cuda()
    sel = torch.full((total + 1,), -5, dtype=torch.int32, device="cuda")
    cnt = torch.full((nq,), -5, dtype=torch.int32, device="cuda")
    call_others()
    graph, stream = torch.cuda.CUDAGraph(), torch.cuda.Stream()
    with torch.cuda.graph(graph, stream=stream):
        cm.cm_sample_buckets(sp, batch, hashes, rec_seeds, sel, cnt,
                             stream=torch.cuda.current_stream())
    assert int(cnt[0]) == -5  # recorded, not run
    for _ in range(3):
        call_others()
        sel.fill_(-5)
        cnt.fill_(-5)
        graph.replay()
        torch.cuda.synchronize()
        check(oracle_mod, rec, rec_seeds, sel.cpu().numpy(), cnt.cpu().numpy(), descs)
        assert int(sel[off]) == -5
    sp.close()
