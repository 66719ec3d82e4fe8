"""The calls that a search using this library makes, over the sizes it makes them at.

A search scores the candidate schedules of a beam step and keeps the k best
(cm_eval_batch and cm_topk_per_query, or the persistent step, or a server),
draws the candidates from hash buckets first (cm_sample_buckets), and between
passes freezes stages and penalizes states it has seen.  Stage counts run
from 3 to 120, candidates of a query from 16 to 4,096 in a serving mix and up
to 65,536 in one large query.  Features, terms and weights follow the
distributions of the repository's synthetic workloads.
"""
import math

import numpy as np
import torch

import paper_2012_07145_amd as cm

# scales of the FP8 form: the ones that the FP8 tests use for these distributions
IN_SCALE, ACT_SCALE = 16.0, 8.0
PENALTY = 1e5

PARAM_LAYOUT = (("W_p", (24, 56)), ("b_p", (24,)), ("W_s", (24, 40)), ("b_s", (24,)),
                ("W_1", (32, 48)), ("b_1", (32,)), ("W_2", (8, 32)), ("b_2", (8,)))


def _case(name, kind, prec, nq, s_lo, s_hi, n_lo, n_hi, k, sizes, hoisted=False):
    return {"name": name, "kind": kind, "prec": prec, "nq": nq, "s_lo": s_lo, "s_hi": s_hi,
            "n_lo": n_lo, "n_hi": n_hi, "k": k, "sizes": sizes, "hoisted": hoisted}


def listed():
    return [
        # a first beam step of a short pipeline: the smallest call, latency only
        _case("score_fp32_4x64", "score", "fp32", 1, 4, 4, 64, 64, 8, 1),
        # a beam of 32 states with 200 children each, in the float32 form
        _case("score_fp32_30x6400", "score", "fp32", 1, 30, 30, 6400, 6400, 32, 2),
        # one very large query (an exhaustive pass over a pipeline's options)
        _case("score_bf16_64x65536", "score", "bf16", 1, 64, 64, 65536, 65536, 32, 3),
        # the same in the 8-bit form, from raw float32 features: they are
        # encoded once and scored once
        _case("encode_fp8_64x65536", "encode", "fp8", 1, 64, 64, 65536, 65536, 32, 3),
        # one session's beam step through the persistent step, a few hundred children
        _case("step_bf16_20x200", "step", "bf16", 1, 20, 20, 200, 200, 32, 4),
        # a beam step of 17 ragged sessions, hoisted inside the step
        _case("step_bf16_17q", "step", "bf16", 17, 3, 120, 16, 4096, 32, 5),
        # a serving micro-batch: 128 sessions whose rows were hoisted at their opening
        _case("step_bf16_128q", "step", "bf16", 128, 3, 120, 16, 4096, 32, 6, True),
        _case("step_fp8_128q", "step", "fp8", 128, 3, 120, 16, 4096, 32, 6, True),
        # a later pass of a multi-pass search: memoized feature rows, penalty on
        # known-bad states, selection
        _case("multipass_bf16_17q", "memo", "bf16", 17, 3, 120, 16, 4096, 32, 7),
        # a pre-pass: per-stage costs, the beam, and the stages that the best
        # candidate freezes
        _case("prepass_bf16_5q", "prepass", "bf16", 5, 60, 120, 1000, 4096, 32, 8),
        # the options of 17 sessions before featurization, drawn down to a few
        # percent by their structural hashes
        _case("sample_17q", "sample", "none", 17, 1, 1, 500, 60000, 1, 9),
        # a saturated server: one request of each of 256 sessions, submitted and
        # waited for, beams in host memory
        _case("serve_bf16_256", "serve", "bf16", 256, 3, 120, 16, 4096, 32, 10),
    ]


def draw(rng):
    kind, prec = rng.choice([("score", "fp32"), ("score", "fp32"), ("score", "bf16"), ("score", "fp8"),
                             ("encode", "fp8"), ("step", "bf16"), ("step", "bf16"), ("step", "fp8"),
                             ("memo", "bf16"), ("memo", "fp8"), ("prepass", "bf16"),
                             ("prepass", "fp32"), ("sample", "none"), ("sample", "none"),
                             ("serve", "bf16")])
    sizes = rng.randrange(1 << 30)
    k = rng.choice([1, 8, 17, 32, 32, 64, 200])
    hoisted = rng.random() < 0.5

    def log_uniform(lo, hi):
        return min(hi, int(math.exp(rng.uniform(math.log(lo), math.log(hi + 1)))))

    if kind == "sample":
        nq = log_uniform(1, 64)
        top = log_uniform(20, max(20, min(200000, 1000000 // nq)))
        return _case("", kind, prec, nq, 1, 1, max(1, top // 50), top, 1, sizes)
    if kind == "serve":
        nq = log_uniform(4, 256)
        return _case("", kind, prec, nq, 3, 120, 16, log_uniform(64, 4096), 32, sizes)
    if rng.random() < 0.5:  # one query, of any shape up to 2^21 rows
        S = log_uniform(1, 120)
        N = log_uniform(16, min(65536, (1 << 21) // S))
        return _case("", kind, prec, 1, S, S, N, N, k, sizes, hoisted)
    nq = log_uniform(2, 100)  # a ragged batch
    top = log_uniform(64, 4096)
    return _case("", kind, prec, nq, 3, 120, 16, top, k, sizes, hoisted)


# ------------------------------------------------------------------- inputs

def _shapes(case):
    """[(stages, candidates)] of the case's queries."""
    r = np.random.default_rng(case["sizes"])
    lo, hi, n = case["s_lo"], case["s_hi"], case["nq"]
    S = np.floor(np.exp(r.uniform(math.log(lo), math.log(hi + 1), n))).astype(int)
    N = r.integers(case["n_lo"], case["n_hi"] + 1, n)
    return [(int(min(max(s, lo), hi)), int(c)) for s, c in zip(S, N)]


def _weights(seed):
    r = np.random.default_rng(seed)
    parts, fan_in = [], 1
    for name, shape in PARAM_LAYOUT:
        fan_in = shape[1] if name.startswith("W") else fan_in
        parts.append((r.standard_normal(shape) / math.sqrt(fan_in)).astype(np.float32).ravel())
    return np.concatenate(parts)


class _Inputs:
    """Weights, features and cost terms of a case, on the GPU, from the seed."""

    def __init__(self, case, seed):
        self.shapes = _shapes(case)
        self.params = _weights(seed)
        g = torch.Generator(device="cuda")
        g.manual_seed(seed)
        rows = sum(s * n for s, n in self.shapes)
        stages = sum(s for s, _ in self.shapes)
        self.cands = sum(n for _, n in self.shapes)
        dev = dict(device="cuda")
        self.pipe = torch.poisson(torch.full((stages * 56,), 3.0, **dev), generator=g)
        self.ridx, feature_rows = None, rows
        if case["kind"] == "memo":
            # each stage draws its candidates' rows from its own pool of an
            # eighth as many distinct rows, the first ones of it most often
            feature_rows = max(1, rows // 8)
            pick = torch.empty(rows, **dev).uniform_(generator=g)
            pools, base, at = [], 0, 0
            for s, n in self.shapes:
                m = max(1, n // 8)
                p = (pick[at:at + s * n].square() * m).long().clamp_(max=m - 1).view(s, n)
                p += base + torch.arange(s, **dev).view(s, 1) * m
                pools.append((p % feature_rows).view(-1).to(torch.int32))
                # row numbers of a query start at a multiple of 8
                pools.append(torch.zeros(-(s * n) % 8, dtype=torch.int32, **dev))
                base, at = base + s * m, at + s * n
            self.ridx = torch.cat(pools)
        self.rows = feature_rows
        self.sched = torch.empty(feature_rows * 40, **dev).normal_(4.0, 2.0, generator=g).exp_()
        self.terms = torch.empty(rows * 8, **dev).normal_(6.0, 1.5, generator=g).exp_()
        self.hashes = self.bad = None
        if case["kind"] == "memo":
            r = np.random.default_rng(seed + 1)
            pool = r.integers(0, 2 ** 64, 4096, dtype=np.uint64)
            self.hashes = torch.from_numpy(r.choice(pool, self.cands).view(np.int64)).cuda()
            self.bad = torch.from_numpy(np.sort(pool[:400]).view(np.int64)).cuda()

    def descs(self, with_ridx=False):
        """(stages, candidates, pipe, sched, terms, cost offsets) of each query."""
        out, p, x, t, c = [], 0, 0, 0, 0
        for s, n in self.shapes:
            out.append((s, n, p, x, t, c))
            p, t, c = p + s * 56, t + s * n * 8, c + n
            x += -(-s * n // 8) * 8 if with_ridx else s * n * 40
        return out


def _sample_inputs(case, seed):
    """Per query: the options' structural hashes, in buckets of heavy-tailed
    sizes (many of one option, a few of hundreds), shuffled; and a seed."""
    r = np.random.default_rng(seed)
    parts = []
    for _, n in _shapes(case):
        sizes = np.minimum(r.zipf(1.6, n), n)
        sizes = sizes[:int(np.searchsorted(np.cumsum(sizes), n)) + 1]
        h = np.repeat(r.integers(0, 2 ** 64, sizes.size, dtype=np.uint64), sizes)[:n]
        parts.append(r.permutation(h))
    return parts, r.integers(0, 2 ** 64, len(parts), dtype=np.uint64)


def _stored(sched, prec):
    if prec == "fp32":
        return sched
    return sched.to(torch.bfloat16) if prec == "bf16" else cm.cm_fp8_encode(sched, IN_SCALE)


def prepare(case, seed):
    kind, prec, k = case["kind"], case["prec"], case["k"]
    st = {"case": case}
    if kind == "sample":
        parts, seeds = _sample_inputs(case, seed)
        total, at, descs = sum(p.size for p in parts), 0, []
        for p in parts:
            descs.append((1, p.size, 0, 0, 0, at))
            at += p.size
        z = torch.zeros(16, device="cuda")
        st.update(sampler=cm.cm_sampler_create(len(parts), total), batch=cm.Batch(descs, z, z, z),
                  hashes=torch.from_numpy(np.concatenate(parts).view(np.int64)).cuda(), seeds=seeds,
                  sel=torch.zeros(total, dtype=torch.int32, device="cuda"),
                  count=torch.zeros(len(parts), dtype=torch.int32, device="cuda"))
        return st
    inp = _Inputs(case, seed)
    model = cm.cm_model_create(inp.params)
    if prec == "fp8":
        cm.cm_model_prepare_fp8(model, IN_SCALE, ACT_SCALE)
    nq = len(inp.shapes)
    stages = sum(s for s, _ in inp.shapes)
    st["model"] = model
    if kind == "serve":
        st["sched"], st["terms"] = inp.sched.to(torch.bfloat16), inp.terms
        srv = cm.cm_server_create(model, k=k, arena_bytes=16 << 30, max_slots=3, max_pending=8192,
                                  max_sessions=256, max_stages=128, max_batch_queries=128,
                                  max_batch_cands=1 << 20)
        pipe = inp.pipe.cpu().numpy().reshape(-1, 56)
        xp, tp, sids, at = [], [], [], 0
        for (s, n, _, x, t, _c) in inp.descs():
            sids.append(srv.session_open(pipe[at:at + s]))
            xp.append(st["sched"].data_ptr() + 2 * x)
            tp.append(st["terms"].data_ptr() + 4 * t)
            at += s
        st.update(srv=srv, sids=np.array(sids, np.int32), xp=np.array(xp, np.uint64),
                  tp=np.array(tp, np.uint64), ns=np.array([n for _, n in inp.shapes], np.int32))
        return st
    st["cost"] = torch.zeros(inp.cands, device="cuda")
    st["idx"] = torch.zeros(nq * k, dtype=torch.int32, device="cuda")
    st["val"] = torch.zeros(nq * k, device="cuda")
    if kind == "encode":
        st["raw"] = inp.sched
        st["codes"] = torch.zeros(inp.sched.numel(), dtype=torch.uint8, device="cuda")
        batch = cm.Batch(inp.descs(), inp.pipe, st["codes"], inp.terms)
    else:
        batch = cm.Batch(inp.descs(kind == "memo"), inp.pipe, _stored(inp.sched, prec), inp.terms)
    st["batch"] = batch
    if kind == "step":
        st["step"] = cm.cm_step_create(model, prec, max_queries=nq, max_stages=stages,
                                       max_cands=inp.cands, max_k=k, slots=2)
        st["U"] = None
        if case["hoisted"]:
            st["U"] = torch.empty(stages * 32, device="cuda")
            cm.cm_hoist_stages(model, prec, batch, st["U"])
        return st
    rows = sum(s * n for s, n in inp.shapes)
    st["ws"] = cm.cm_workspace_create(nq, stages, inp.cands, rows, k)
    if kind == "memo":
        st.update(ridx=inp.ridx, rows=inp.rows, hashes=inp.hashes, bad=inp.bad)
    if kind == "prepass":
        st["stage"] = torch.zeros(rows, device="cuda")
        st["frozen"] = torch.zeros(stages, dtype=torch.uint8, device="cuda")
    return st


def run(st):
    c = st["case"]
    kind, prec, k = c["kind"], c["prec"], c["k"]
    if kind == "sample":
        cm.cm_sample_buckets(st["sampler"], st["batch"], st["hashes"], st["seeds"], st["sel"],
                             st["count"])
        return {"sel": st["sel"], "count": st["count"]}
    if kind == "serve":
        tickets = st["srv"].submit_batch(st["sids"], st["ns"], st["xp"], st["tp"], k)
        beams = st["srv"].wait_all_results(tickets)
        return {"idx": np.concatenate([i for i, _ in beams]),
                "val": np.concatenate([v for _, v in beams])}
    batch, cost = st["batch"], st["cost"]
    out = {"cost": cost, "idx": st["idx"], "val": st["val"]}
    if kind == "step":
        cm.cm_step_run(st["step"], batch, st["U"], k, cost, st["idx"], st["val"])
        return out
    if kind == "memo":
        cm.cm_eval_indexed(st["model"], prec, batch, st["ridx"], st["rows"], st["ws"], cost)
        cm.cm_penalize_known_bad(batch, st["hashes"], st["bad"], PENALTY, cost)
    elif kind == "prepass":
        cm.cm_eval_stages(st["model"], prec, batch, st["ws"], cost, st["stage"])
    else:
        if kind == "encode":
            cm.cm_fp8_encode(st["raw"], IN_SCALE, st["codes"])
            out["codes"] = st["codes"]
        cm.cm_eval_batch(st["model"], prec, batch, st["ws"], cost)
    cm.cm_topk_per_query(cost, batch, k, st["ws"], st["idx"], st["val"])
    if kind == "prepass":
        cm.cm_freeze_stages(st["stage"], batch, st["idx"], k, st["frozen"])
        out["stage"], out["frozen"] = st["stage"], st["frozen"]
    return out


# --------------------------------------------------- what a pass cannot avoid

def work(case):
    shapes = _shapes(case)
    cands = sum(n for _, n in shapes)
    if case["kind"] == "sample":
        # hashes read, representatives (about an eighth) and counts written
        return {"bytes": 8.0 * cands + 4.0 * cands / 8 + 4 * len(shapes), "flops": 0.0}
    rows = sum(s * n for s, n in shapes)
    stages = sum(s for s, _ in shapes)
    feature = {"fp32": 160, "bf16": 80, "fp8": 40}[case["prec"]]
    kind = case["kind"]
    # features, 8 terms and the two folded layers of each row; the stage rows;
    # costs and beams
    b = rows * (feature + 32.0) + 4.0 * cands + 8.0 * case["k"] * len(shapes)
    b += stages * (128.0 if case["hoisted"] or kind == "serve" else 224.0)
    if kind == "encode":
        b += rows * 160.0  # the raw features; the codes (counted above) are an output
    if kind == "memo":
        b += rows * 4.0 - rows * feature * 7.0 / 8 + 8.0 * cands
    if kind == "prepass":
        b += rows * 4.0 + stages
    return {"bytes": b, "flops": rows * 2.0 * (40 * 32 + 32 * 8 + 8)}


# ------------------------------------------------------- the same in 64 bits

def _e4m3(v):
    """The nearest e4m3 value (ties to even, saturating at 448) of each double."""
    a = v.abs().clamp(max=448.0)
    quantum = torch.exp2(torch.floor(torch.log2(a.clamp(min=2.0 ** -6))) - 3)
    return torch.copysign(torch.round(a / quantum) * quantum, v).clamp(-448.0, 448.0)


def _pow2_under(amax):
    return 2.0 ** math.floor(math.log2(448.0 / amax))


def exact(case, seed):
    kind, prec, k = case["kind"], case["prec"], case["k"]
    if kind == "sample":
        return None
    inp = _Inputs(case, seed)
    w, at = {}, 0
    for name, shape in PARAM_LAYOUT:
        n = int(np.prod(shape))
        w[name] = torch.from_numpy(inp.params[at:at + n].reshape(shape)).cuda().double()
        at += n
    sched = inp.sched.to(torch.bfloat16) if prec == "bf16" else inp.sched
    wf = w["W_1"][:, 24:] @ w["W_s"]
    sw1, sw2 = _pow2_under(float(wf.abs().max())), _pow2_under(float(w["W_2"].abs().max()))
    costs, stage_costs, vals = [], [], []
    for (s, n, p, x, t, c) in inp.descs(kind == "memo"):
        pipe = inp.pipe[p:p + s * 56].view(s, 56).double()
        hoisted = (torch.log1p(pipe) @ w["W_p"].T + w["b_p"]) @ w["W_1"][:, :24].T + w["b_1"]
        total = torch.zeros(n, dtype=torch.float64, device="cuda")
        for j in range(s):
            if kind == "memo":
                row = inp.ridx[x + j * n:x + (j + 1) * n].long()
                f = sched.view(-1, 40)[row].double()
            else:
                f = sched[x + j * n * 40:x + (j + 1) * n * 40].view(n, 40).double()
            f = torch.log1p(f)
            if prec == "fp8":
                a = (_e4m3(f * IN_SCALE) @ _e4m3(wf * sw1).T) / (sw1 * IN_SCALE)
                a = a + hoisted[j] + w["W_1"][:, 24:] @ w["b_s"]
                h = _e4m3(a.clamp(min=0) * ACT_SCALE)
                co = (h @ _e4m3(w["W_2"] * sw2).T) / (sw2 * ACT_SCALE) + w["b_2"]
            else:
                h = ((f @ w["W_s"].T + w["b_s"]) @ w["W_1"][:, 24:].T + hoisted[j]).clamp(min=0)
                co = h @ w["W_2"].T + w["b_2"]
            terms = inp.terms[t + j * n * 8:t + (j + 1) * n * 8].view(n, 8).double()
            v = (co.clamp(min=0) * terms).sum(1)
            total += v
            if kind == "prepass":
                stage_costs.append(v)
        if kind == "memo":
            total += PENALTY * torch.isin(inp.hashes[c:c + n], inp.bad)
        costs.append(total)
        best = torch.full((k,), math.inf, dtype=torch.float64, device="cuda")
        m = min(k, n)
        best[:m] = torch.sort(total).values[:m]
        vals.append(best)
    val = torch.cat(vals)
    if kind == "serve":
        return {"idx": None, "val": val}
    out = {"cost": torch.cat(costs), "idx": None, "val": val}
    if kind == "encode":
        out["codes"] = None
    if kind == "prepass":
        out["stage"], out["frozen"] = torch.cat(stage_costs), None
    return out
