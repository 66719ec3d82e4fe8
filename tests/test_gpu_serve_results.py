"""wait_all_results: the beams of a batch of requests equal the beams of the
same requests waited for one by one, for no request, one and many, with k below
the server's k."""
import numpy as np
import pytest

from synth import draw_query, model_params

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [0, 1, 37])
def test_wait_all_results_equals_wait(n):
    import torch
    import paper_2012_07145_amd as cm
    rng = np.random.default_rng(n)
    m = cm.cm_model_create(model_params(bias=True))
    srv = cm.cm_server_create(m, k=32, max_slots=2, max_sessions=max(n, 1), max_stages=16,
                              max_batch_queries=16)
    qs = [draw_query(rng, int(rng.integers(1, 12)), int(rng.integers(1, 300))) for _ in range(n)]
    sched = [torch.from_numpy(q.sched).cuda().to(torch.bfloat16) for q in qs]
    terms = [torch.from_numpy(q.terms).cuda() for q in qs]
    sids = [srv.session_open(q.pipe) for q in qs]
    ks = [32 if j % 3 else 5 for j in range(n)]
    one = [srv.wait(srv.submit(sids[j], qs[j].n_cands, sched[j], terms[j], ks[j])) for j in range(n)]
    tickets = srv.submit_batch(sids, [q.n_cands for q in qs], [x.data_ptr() for x in sched],
                               [t.data_ptr() for t in terms], ks) if n else np.zeros(0, np.uint64)
    beams = srv.wait_all_results(tickets)
    assert len(beams) == n
    for (i, v), (wi, wv, _), k in zip(beams, one, ks):
        assert i.dtype == np.int32 and v.dtype == np.float32 and i.shape == v.shape == (k,)
        assert np.array_equal(i, wi) and np.array_equal(v, wv)
    srv.close()
    m.close()
