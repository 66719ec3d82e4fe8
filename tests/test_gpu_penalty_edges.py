"""Known-bad penalty (cm_penalize_known_bad) where its work split changes: bad
sets around the 1,024 hashes that it keeps in LDS and far above, candidate
counts around its workgroups, empty queries and more queries than a launch
holds -- bit-exact against the oracle."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_bad", [1, 2, 1023, 1024, 1025, 2047, 2049, 3000, 100_003])
def test_penalty_set_sizes(oracle_mod, n_bad):
    import torch
    import paper_2012_07145_amd as cm
    rng = np.random.default_rng(n_bad)
    bad = np.sort(rng.integers(0, 2 ** 64, n_bad, dtype=np.uint64))
    bad[0], bad[-1] = 0, 2 ** 64 - 1
    bad[n_bad // 2:n_bad // 2 + 40] = bad[n_bad // 2]   # a run of equal hashes
    sizes = [0, 1, 255, 256, 257, 0, 3000] + [int(rng.integers(0, 600)) for _ in range(35)] + [0]
    costs, hashes, descs, off = [], [], [], 0
    near = np.concatenate([bad - np.uint64(1), bad, bad + np.uint64(1)])
    for n in sizes:
        h = np.where(rng.random(n) < 0.5, rng.choice(near, n),
                     rng.integers(0, 2 ** 64, n, dtype=np.uint64))
        costs.append(rng.lognormal(8, 1, n).astype(np.float32))
        hashes.append(h)
        descs.append((1, n, 0, 0, 0, off))
        off += n
    z = torch.zeros(1, device="cuda")
    c = torch.from_numpy(np.concatenate(costs + [np.zeros(1, np.float32)])).cuda()
    h = torch.from_numpy(np.concatenate(hashes).view(np.int64)).cuda()
    cm.cm_penalize_known_bad(cm.Batch(descs, z, z, z), h, torch.from_numpy(bad.view(np.int64)).cuda(),
                             1234.5, c)
    torch.cuda.synchronize()
    got = c.cpu().numpy()
    for d, cc, hh in zip(descs, costs, hashes):
        want = oracle_mod.penalize(cc, hh, bad, 1234.5)
        assert np.array_equal(got[d[5]:d[5] + d[1]].view(np.uint32), want.view(np.uint32))
    assert got[-1] == 0.0


def test_penalty_more_candidates_than_a_launch_takes():
    """More than 2^32 candidates in one call: every query's first and last ones
    are reached, and no other cost changes."""
    import torch
    import paper_2012_07145_amd as cm
    sizes = [3, 2 ** 31 - 1, 0, 2 ** 31 - 1, 1000]
    total, descs = 0, []
    for n in sizes:
        descs.append((1, n, 0, 0, 0, total))
        total += n
    if torch.cuda.mem_get_info()[0] < 14 * total:
        pytest.skip("needs 60 GB of device memory")
    bad = torch.tensor([5, 77], device="cuda")
    h = torch.zeros(total, dtype=torch.int64, device="cuda")
    c = torch.zeros(total, device="cuda")
    hits = sorted({d[5] + e for d in descs if d[1] for e in (0, d[1] // 2, d[1] - 1)})
    h[torch.tensor(hits, device="cuda")] = 77
    z = torch.zeros(1, device="cuda")
    cm.cm_penalize_known_bad(cm.Batch(descs, z, z, z), h, bad, 2.5, c)
    found = torch.cat([torch.nonzero(p).view(-1) + j * (1 << 28)
                       for j, p in enumerate(torch.split(c, 1 << 28))]).cpu().numpy()
    assert np.array_equal(found, hits)
    assert bool((c[torch.tensor(hits, device="cuda")] == 2.5).all())
    del h, c
    torch.cuda.empty_cache()


@pytest.mark.parametrize("n", [511, 512, 513, 1023, 1024, 1025])
def test_penalty_workgroup_edges(oracle_mod, n):
    import torch
    import paper_2012_07145_amd as cm
    rng = np.random.default_rng(n)
    bad = np.sort(rng.integers(0, 2 ** 64, 1500, dtype=np.uint64))
    descs, costs, hashes = [], [], []
    for j in range(3):
        descs.append((1, n, 0, 0, 0, j * n))
        costs.append(rng.lognormal(8, 1, n).astype(np.float32))
        hashes.append(np.where(rng.random(n) < 0.5, rng.choice(bad, n), bad[0] + np.uint64(1)))
        hashes[-1][-1] = bad[-1]
    z = torch.zeros(1, device="cuda")
    c = torch.from_numpy(np.concatenate(costs)).cuda()
    h = torch.from_numpy(np.concatenate(hashes).view(np.int64)).cuda()
    cm.cm_penalize_known_bad(cm.Batch(descs, z, z, z), h,
                             torch.from_numpy(bad.view(np.int64)).cuda(), -7.25, c)
    got = c.cpu().numpy()
    for j in range(3):
        want = oracle_mod.penalize(costs[j], hashes[j], bad, -7.25)
        assert np.array_equal(got[j * n:(j + 1) * n].view(np.uint32), want.view(np.uint32))
