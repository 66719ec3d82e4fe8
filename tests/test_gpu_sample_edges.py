"""Hierarchical sampling (cm_sample_buckets) at the edges of its work split:
chunks of 1,024 options, lists of whole buckets (up to 32 members) and of
candidates, the hash value that marks an empty slot, and buckets whose
candidate list comes out short; bit-exact against the oracle, several calls on
one sampler."""
import numpy as np
import pytest

from tests.test_gpu_sample import bucket_hashes, check, run

pytestmark = pytest.mark.gpu

FULL = np.uint64(2 ** 64 - 1)


@pytest.fixture(scope="module")
def cm():
    import torch
    assert torch.cuda.is_available()
    import paper_2012_07145_amd as cm
    return cm


@pytest.mark.parametrize("n", [1, 2, 511, 1023, 1024, 1025, 2049, 9000])
@pytest.mark.parametrize("kind", ["distinct", "equal", "marker", "dense", "low"])
def test_sample_chunk_edges(cm, oracle_mod, n, kind):
    rng = np.random.default_rng(n)
    h = {"distinct": rng.permutation(n).astype(np.uint64) * np.uint64(0x9E3779B97F4A7C15),
         "equal": np.full(n, 12345, np.uint64),
         "marker": np.where(rng.random(n) < 0.5, FULL, np.uint64(7)),
         "dense": rng.integers(0, max(1, n // 100) + 1, n).astype(np.uint64),
         "low": rng.integers(0, 2 * n, n).astype(np.uint64)}[kind]
    sp = cm.cm_sampler_create(2, n)
    for seed in (5, 6):  # the second call finds the table as the first left it
        sel, cnt, descs = run(cm, sp, [h], [seed])
        check(oracle_mod, [h], [seed], sel, cnt, descs)
        assert sel[-1] == -5
    sp.close()


def test_sample_bucket_sizes(cm, oracle_mod):
    """Buckets of every size at which the representatives or the list change."""
    rng = np.random.default_rng(3)
    sizes = [1, 2, 3, 4, 5, 8, 9, 31, 32, 33, 34, 64, 65, 128, 129, 255, 256, 257, 1024, 1025, 4000]
    parts = [np.repeat(rng.integers(0, 2 ** 64, 20, dtype=np.uint64), b) for b in sizes]
    hashes = [rng.permutation(p) for p in parts] + [rng.permutation(np.concatenate(parts))]
    seeds = rng.integers(0, 2 ** 64, len(hashes), dtype=np.uint64)
    sp = cm.cm_sampler_create(len(hashes), sum(h.size for h in hashes))
    sel, cnt, descs = run(cm, sp, hashes, seeds)
    check(oracle_mod, hashes, seeds, sel, cnt, descs)
    sp.close()


# (bucket size, seed) for which fewer members than representatives fall under
# the bound of the candidates (found by a search over 6e7 seeds)
SHORT = [(256, 3359416), (256, 6203968), (200, 6634266), (512, 29459833)]


@pytest.mark.parametrize("others", [0, 300, 3000])  # one chunk (a launch of its own) and several
def test_sample_short_candidate_lists(cm, oracle_mod, others):
    hashes = [np.full(b, 99, np.uint64) for b, _ in SHORT]
    seeds = np.array([s for _, s in SHORT], np.uint64)
    # the bucket's options come first, so their keys are the search's
    rng = np.random.default_rng(4)
    if others:
        hashes = [np.concatenate([h, bucket_hashes(rng, others)]) for h in hashes]
    sp = cm.cm_sampler_create(len(hashes), sum(h.size for h in hashes))
    sel, cnt, descs = run(cm, sp, hashes, seeds)
    check(oracle_mod, hashes, seeds, sel, cnt, descs)
    sp.close()


@pytest.mark.parametrize("nq", [1, 64, 65, 130])
def test_sample_small_queries(cm, oracle_mod, nq):
    """Every query within one chunk: a single launch, with descriptors by value
    and from memory; larger queries on the same sampler in between."""
    rng = np.random.default_rng(nq)
    sizes = [int(rng.integers(0, 1025)) for _ in range(nq)]
    sizes[0] = 1024
    hashes = [bucket_hashes(rng, n) if n else np.zeros(0, np.uint64) for n in sizes]
    for j in range(0, nq, 3):
        hashes[j] = rng.integers(0, 5, sizes[j]).astype(np.uint64)
        hashes[j][:: 7] = FULL
    seeds = rng.integers(0, 2 ** 64, nq, dtype=np.uint64)
    sp = cm.cm_sampler_create(nq, max(sum(sizes), 5000))
    for _ in range(2):
        sel, cnt, descs = run(cm, sp, hashes, seeds)
        check(oracle_mod, hashes, seeds, sel, cnt, descs)
        assert sel[-1] == -5
        big = [bucket_hashes(rng, 4000)]
        sel, cnt, descs = run(cm, sp, big, [7])
        check(oracle_mod, big, [7], sel, cnt, descs)
    sp.close()


def test_sample_many_queries_some_empty(cm, oracle_mod):
    rng = np.random.default_rng(5)
    sizes = [0, 0, 3] + [int(rng.integers(0, 2500)) for _ in range(190)] + [0, 1, 0]
    hashes = [bucket_hashes(rng, n) if n else np.zeros(0, np.uint64) for n in sizes]
    seeds = rng.integers(0, 2 ** 64, len(sizes), dtype=np.uint64)
    sp = cm.cm_sampler_create(200, sum(sizes))
    for part in (slice(None), slice(60, 70), slice(0, 2)):
        hs, ss = hashes[part], seeds[part]
        sel, cnt, descs = run(cm, sp, hs, ss)
        check(oracle_mod, hs, ss, sel, cnt, descs)
    sp.close()


@pytest.mark.parametrize("nq", [4095, 4096, 4097, 9001])
def test_sample_thousands_of_queries(cm, oracle_mod, nq):
    """A chunk finds its query by votes over 64 of them at a time: the edges of
    two and three rounds, with empty queries at both ends and in between."""
    rng = np.random.default_rng(nq)
    sizes = rng.integers(0, 4, nq)
    sizes[rng.integers(0, nq, 40)] = rng.integers(1000, 3100, 40)
    sizes[[0, nq - 1]] = 0
    sizes[[1, 64, 4094, nq - 2]] = [1025, 2048, 1500, 1024]
    pool = rng.integers(0, 2 ** 64, 900, dtype=np.uint64)
    hashes = [rng.choice(pool[: max(1, n // 3)], n) for n in sizes]
    seeds = rng.integers(0, 2 ** 64, nq, dtype=np.uint64)
    sp = cm.cm_sampler_create(nq, int(sizes.sum()))
    sel, cnt, descs = run(cm, sp, hashes, seeds)
    check(oracle_mod, hashes, seeds, sel, cnt, descs)
    assert sel[-1] == -5
    sp.close()


# options of a query ahead, so that the second query's chunks start inside a
# group of 512, on its edge and one after it
@pytest.mark.parametrize("ahead", [1000, 511 * 1024, 512 * 1024, 512 * 1024 + 1])
@pytest.mark.parametrize("chunks", [1024, 1025, 1026, 1700])
def test_sample_many_chunks(cm, oracle_mod, ahead, chunks):
    """A query of more than two groups of chunks: what is kept ahead of a chunk
    is summed by groups."""
    rng = np.random.default_rng(chunks)
    sizes = [ahead, chunks * 1024 - 7, 3000]
    hashes = [rng.integers(0, max(1, n // 3), n).astype(np.uint64) for n in sizes]
    seeds = rng.integers(0, 2 ** 64, len(sizes), dtype=np.uint64)
    sp = cm.cm_sampler_create(len(sizes), sum(sizes))
    for _ in range(2):
        sel, cnt, descs = run(cm, sp, hashes, seeds)
        check(oracle_mod, hashes, seeds, sel, cnt, descs)
        assert sel[-1] == -5
    sp.close()


@pytest.mark.parametrize("largest", [1, 2500])  # one kernel for the call, and several
def test_sample_more_queries_than_a_launch_takes(cm, oracle_mod, largest):
    """2^23 workgroups of 512 threads are more than one launch holds."""
    import torch
    from paper_2012_07145_amd import _lib
    import ctypes
    nq = (1 << 23) + 5
    rng = np.random.default_rng(largest)
    n = rng.integers(0, 2, nq).astype(np.int32)
    big = [0, 12345, (1 << 22) - 1, 1 << 22, nq - 1]
    n[big] = largest
    off = np.zeros(nq, np.int64)
    np.cumsum(n[:-1], out=off[1:])
    total = int(n.sum())
    names = [f for f, _ in _lib.cm_query._fields_]
    q = np.zeros(nq, np.dtype({"names": names,
                               "formats": [np.int32, np.int32] + [np.int64] * (len(names) - 2),
                               "offsets": [getattr(_lib.cm_query, f).offset for f in names],
                               "itemsize": ctypes.sizeof(_lib.cm_query)}))
    q["n_stages"], q["n_cands"], q["cost_off"] = 1, n, off
    z = torch.zeros(1, device="cuda")
    batch = cm.Batch([], z, z, z)
    batch.c.n_queries = nq
    batch.c.queries = ctypes.cast(q.ctypes.data, type(batch.c.queries))
    hashes = rng.integers(0, 50, total).astype(np.uint64)
    seeds = rng.integers(0, 2 ** 64, nq, dtype=np.uint64)
    sp = cm.cm_sampler_create(nq, total)
    sel = torch.full((total + 1,), -5, dtype=torch.int32, device="cuda")
    cnt = torch.full((nq,), -5, dtype=torch.int32, device="cuda")
    cm.cm_sample_buckets(sp, batch, torch.from_numpy(hashes.view(np.int64)).cuda(), seeds, sel, cnt)
    torch.cuda.synchronize()
    sel, cnt = sel.cpu().numpy(), cnt.cpu().numpy()
    small = np.ones(nq, bool)
    small[big] = False
    assert np.array_equal(cnt[small], n[small])  # a lone option is kept
    assert not sel[off[small & (n == 1)]].any()
    for j in big:
        want = oracle_mod.sample(hashes[off[j]:off[j] + n[j]], int(seeds[j]))
        assert cnt[j] == want.size
        assert np.array_equal(sel[off[j]:off[j] + want.size], want)
    sp.close()


# (bucket size, its first option, seed), found as SHORT was: buckets over
# several chunks
SHORT_LONG = [(2048, 0, 91014303), (2048, 0, 20063815), (4096, 0, 16937571), (300, 900, 81182720)]


@pytest.mark.parametrize("others", [0, 3000, 300_000])
def test_sample_short_candidate_lists_over_chunks(cm, oracle_mod, others):
    rng = np.random.default_rng(6)
    hashes, seeds = [], []
    for b, first, seed in SHORT_LONG + [(b, 0, s) for b, s in SHORT]:
        h = np.concatenate([rng.integers(0, 40, first).astype(np.uint64) + np.uint64(100),
                            np.full(b, 99, np.uint64), bucket_hashes(rng, others) if others else
                            np.zeros(0, np.uint64)])
        hashes.append(h)
        seeds.append(seed)
    seeds = np.array(seeds, np.uint64)
    sp = cm.cm_sampler_create(len(hashes), sum(h.size for h in hashes))
    for _ in range(2):
        sel, cnt, descs = run(cm, sp, hashes, seeds)
        check(oracle_mod, hashes, seeds, sel, cnt, descs)
        assert sel[-1] == -5
    sp.close()
