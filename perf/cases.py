"""The workloads whose time is measured: what a serving engine that compresses its paged KV
cache has this library do, through the Python binding.

Six kinds of pass, each one or two calls as an engine makes them:

  step      the compression step of one layer (actkv.step): score the cache against the action
            queries, keep the best entries of every (request, KV head), move them to fresh pages
  decode    streaming scoring: one decode step's scores added to the running aggregate
  fresh     compression by scores already aggregated over an action: select and move to fresh
            pages (actkv.select_compact)
  inplace   the same with the in-place compaction: actkv.select, then actkv.compact_inplace
  lrfu      eviction by LRFU keep scores carried from step to step, then the compaction
  monitor   the confidence monitor: the token confidence of a decode step's logits and the
            budget update over the requests' traces

Inputs follow the repository's synthetic recipe: N(0, 1) bf16 queries, keys and values, 1% of
the keys leaning towards the mean action query of their head, pages scattered over a pool twice
the pages in use.  Lengths, query counts and budgets belong to the case; the values to the seed.
The block table is laid out anew for every pass from the engine's page lists, as an engine does
for each batch (a pass rewrites it); K and V need no restoring: the pages a pass writes are never
ones that it reads.
"""
import math

import numpy as np
import torch

from paper_2609_31395_amd import actkv

PAGE = 16
DEVICE = "cuda"
TOP_P, DECAY = 0.9, 0.5          # the LRFU settings of the paper
TOP_K, CONF_WINDOW, CONF_STRIDE = 20, 64, 8


def _case(name, kind, reqs, len_lo, len_hi, q_lo, q_hi, q_heads, kv_heads, head_dim, budget,
          amount, window, agg="sum", lse=True, lens=1):
    c = dict(kind=kind, reqs=reqs, len_lo=len_lo, len_hi=len_hi, q_lo=q_lo, q_hi=q_hi,
             q_heads=q_heads, kv_heads=kv_heads, head_dim=head_dim, budget=budget, amount=amount,
             window=window, agg=agg, lse=lse, lens=lens)
    if name:
        c["name"] = name
    return c


def _monitor(name, reqs, vocab, trace_lo, trace_hi, lens=1):
    c = dict(kind="monitor", reqs=reqs, vocab=vocab, trace_lo=trace_lo, trace_hi=trace_hi,
             lens=lens)
    if name:
        c["name"] = name
    return c


def listed():
    return [
        # one short conversation of a small model: launch latency and the host path
        _case("step_short", "step", 1, 2048, 2048, 16, 16, 8, 2, 64, "fixed", 512, 5),
        # one agent trace of a 25-iteration web task, compressed by itself as it ends an action
        _case("step_one_trace", "step", 1, 35000, 35000, 64, 64, 32, 4, 128, "frac", 0.25, 7),
        # a small group of traces in the paper's own form: max over the group and mean over the
        # queries, no pooling, the attention backend hands over no LSE
        _case("step_paper_form", "step", 8, 8000, 33000, 32, 128, 32, 4, 128, "frac", 0.25, 1,
              agg="max_mean", lse=False, lens=1003),
        # a batch of agents at different points of their traces, unequal query counts
        _case("step_ragged", "step", 32, 8000, 40000, 32, 128, 32, 4, 128, "frac", 0.25, 7,
              lens=1003),
        # the headline batch: 32 requests of 35,000 tokens
        _case("step_batch", "step", 32, 35000, 35000, 64, 64, 32, 4, 128, "frac", 0.25, 7,
              lens=1006),
        # one layer of a full-model compression: long traces, budgets unequal across the heads
        _case("step_model_layer", "step", 32, 16000, 64000, 64, 64, 32, 4, 128, "dirichlet", 0.25,
              7, lens=1007),
        # a decode step of four short conversations (block 16, 8 KV heads)
        _case("decode_short", "decode", 4, 2048, 2048, 1, 1, 32, 8, 128, "fixed", 1536, 1),
        # a decode step over the headline batch's cache
        _case("decode_batch", "decode", 32, 35000, 35000, 1, 1, 32, 4, 128, "frac", 0.25, 1,
              lens=1006),
        # the compression of a few short conversations to fresh pages
        _case("fresh_short", "fresh", 4, 2048, 2048, 1, 1, 32, 8, 128, "fixed", 1536, 1),
        # the compression of many conversations within their own pages
        _case("inplace_many", "inplace", 64, 6144, 6144, 1, 1, 32, 8, 128, "fixed", 4096, 1),
        # LRFU eviction of a group of traces, some longer than others
        _case("lrfu_group", "lrfu", 16, 8000, 60000, 1, 1, 32, 4, 128, "frac", 0.25, 7, lens=1005),
        # the monitor over a batch: a 151,936-token vocabulary, traces of up to 35,000 tokens
        _monitor("monitor_batch", 32, 151936, 2000, 35000),
    ]


HEADS = [(8, 2, 64), (32, 4, 128), (32, 8, 128), (64, 8, 64), (16, 8, 128), (16, 2, 128)]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case of the same ranges: requests, lengths, query counts, head shapes, budgets,
    windows and options at random, never more work than the largest listed case."""
    kind = rng.choice(["step", "step", "step", "decode", "fresh", "inplace", "lrfu", "monitor"])
    lens = rng.randrange(1, 1 << 20)
    if kind == "monitor":
        hi = _log(rng, 300, 35000)
        return _monitor(None, _log(rng, 1, 64), _log(rng, 32000, 200000), max(64, hi // 4), hi,
                        lens=lens)
    while True:
        hq, hkv, d = rng.choice(HEADS)
        reqs = _log(rng, 1, 64)
        hi = _log(rng, 512, 64000)
        lo = hi if rng.random() < 0.3 else max(256, int(hi * rng.uniform(0.2, 0.9)))
        q_hi = _log(rng, 4, 128) if kind == "step" else 1
        q_lo = q_hi if rng.random() < 0.5 else max(1, q_hi // 4)
        tokens = reqs * (lo + hi) / 2
        lse = rng.random() < 0.8
        work = tokens * hkv * (hq // hkv) * q_hi * d * 2 * (1 if lse else 2)
        if work <= 4e11 and tokens * hkv * d <= 4.5e8:   # K in use: at most 0.9 GB
            break
    budget = rng.choice(["frac", "dirichlet", "fixed"])
    amount = rng.choice([0.15, 0.25, 0.5]) if budget != "fixed" else max(64, lo // 3)
    return _case(None, kind, reqs, lo, hi, q_lo, q_hi, hq, hkv, d, budget, amount,
                 rng.choice([1, 5, 7]) if kind in ("step", "lrfu") else 1,
                 agg=rng.choice(["sum", "sum", "max_mean"]), lse=lse, lens=lens)


def _shape(case):
    """Lengths, query counts and budgets of a case (the same for every seed)."""
    rng = np.random.default_rng(case["lens"])
    R, H = case["reqs"], case["kv_heads"]
    L = rng.integers(case["len_lo"], case["len_hi"] + 1, size=R).astype(np.int32)
    n = rng.integers(case["q_lo"], case["q_hi"] + 1, size=R).astype(np.int32)
    if case["budget"] == "fixed":
        b = np.full((R, H), int(case["amount"]))
    elif case["budget"] == "frac":
        b = np.repeat(np.floor(case["amount"] * L)[:, None], H, axis=1)
    else:   # a Dirichlet(0.5) split of the request's share over its heads
        w = rng.dirichlet(np.full(H, 0.5), size=R)
        b = np.minimum(np.floor(w * H * case["amount"] * L[:, None]), L[:, None])
    return L, n, b.astype(np.int32).reshape(-1)


def _traces(case):
    rng = np.random.default_rng(case["lens"])
    T = rng.integers(case["trace_lo"], case["trace_hi"] + 1, size=case["reqs"])
    return np.concatenate([[0], np.cumsum(T)]).astype(np.int64)


class State:
    pass


def _row_lse(q, k, n, scale, dtype):
    """Causal log-sum-exp of the rows q [n * G, D] (query-major) over the keys k [L, D]."""
    s = (q.to(dtype) @ k.to(dtype).t().contiguous()).mul_(scale)
    G = q.shape[0] // n
    s[:, -n:].masked_fill_(_hidden(n, G, s.device), -math.inf)
    return torch.logsumexp(s, 1), s


def _hidden(n, G, device):
    """Of the last n keys, those past a query's own position ([n * G, n])."""
    j = torch.arange(n, device=device)
    return (j[None, :] > j[:, None]).repeat_interleave(G, 0)


def _keys(st, r, h):
    L = int(st.L[r])
    pages = st.table[r, :-(-L // PAGE)].long()
    return st.kv[0, pages, :, h].reshape(-1, st.kv.shape[-1])[:L]


def _queries(st, r, h):
    c = st.case
    G = c["q_heads"] // c["kv_heads"]
    q = st.q[int(st.cu[r]):int(st.cu[r + 1]), h * G:(h + 1) * G]
    return q.reshape(-1, q.shape[-1])


def prepare(case, seed):
    gen = torch.Generator(device=DEVICE)
    gen.manual_seed(int(seed))
    st = State()
    st.case = case
    if case["kind"] == "monitor":
        st.offsets = _traces(case)
        st.offsets_d = torch.from_numpy(st.offsets).to(DEVICE)
        st.logits = torch.randn(case["reqs"], case["vocab"], generator=gen, device=DEVICE).mul_(3)
        st.conf = torch.rand(int(st.offsets[-1]), generator=gen, device=DEVICE).mul_(2).add_(8)
        st.budgets = torch.full((case["reqs"],), 2048, dtype=torch.int32, device=DEVICE)
        return st

    R, Hq, Hkv, D = case["reqs"], case["q_heads"], case["kv_heads"], case["head_dim"]
    G = Hq // Hkv
    L, n, budgets = _shape(case)
    st.L, st.n, st.cu = L, n, np.concatenate([[0], np.cumsum(n)])
    Y = -(-L // PAGE)
    used = int(Y.sum())
    P = 2 * used
    perm = torch.randperm(P, generator=gen, device=DEVICE).to(torch.int32)
    table = torch.full((R, int(Y.max())), -1, dtype=torch.int32, device=DEVICE)
    off = 0
    for r in range(R):
        table[r, :int(Y[r])] = perm[off:off + int(Y[r])]
        off += int(Y[r])
    st.table, st.bt = table, torch.empty_like(table)
    st.free = perm[used:].clone()
    st.kv = torch.randn(2, P, PAGE, Hkv, D, generator=gen, device=DEVICE, dtype=torch.bfloat16)
    st.q = torch.randn(int(n.sum()), Hq, D, generator=gen, device=DEVICE, dtype=torch.bfloat16)
    rows = st.kv[0].view(P * PAGE, Hkv, D)
    heads = torch.arange(Hkv, device=DEVICE)[None, :]
    for r in range(R):
        cnt = int(round(0.01 * L[r]))
        if cnt == 0:
            continue
        mean = st.q[int(st.cu[r]):int(st.cu[r + 1])].float().view(-1, Hkv, G, D).mean((0, 2))
        t = torch.randint(0, int(L[r]), (cnt, Hkv), generator=gen, device=DEVICE)
        slot = table[r].long()[t // PAGE] * PAGE + t % PAGE
        rows[slot, heads] = (rows[slot, heads].float() + 3 * mean).to(torch.bfloat16)

    st.scale = float(np.float32(1) / np.sqrt(np.float32(D)))
    st.p = actkv.Problem(seq_lens=L, q_lens=n, budgets=budgets, num_q_heads=Hq, num_kv_heads=Hkv,
                         head_dim=D, num_pages=P, bt_stride=int(Y.max()), sm_scale=st.scale,
                         pool_window=case["window"], agg=case["agg"]).to_device(DEVICE)
    st.planned = st.p.planned()
    st.ws = actkv.workspace(st.p)
    N = int(L.astype(np.int64).sum()) * Hkv
    st.lse = None
    if case["kind"] == "decode" or (case["kind"] == "step" and case["lse"]):
        # the LSE that the attention kernel left behind
        st.lse = torch.empty(int(n.sum()), Hq, device=DEVICE)
        for r in range(R):
            for h in range(Hkv):
                lse, _ = _row_lse(_queries(st, r, h), _keys(st, r, h), int(n[r]), st.scale,
                                  torch.float32)
                st.lse[int(st.cu[r]):int(st.cu[r + 1]), h * G:(h + 1) * G] = lse.view(-1, G)
    if case["kind"] == "step":
        st.scores = torch.empty(N, device=DEVICE)
    else:
        # scores aggregated over the decode steps of an action so far
        s = torch.randn(N, generator=gen, device=DEVICE).mul_(0.4).exp_()
        spike = torch.rand(N, generator=gen, device=DEVICE) < 0.01
        s = torch.where(spike, s * 8, s).mul_(G * 16 / float(L.mean()))
        st.scores = s
        if case["kind"] == "decode":
            st.acc = torch.empty_like(s)
        if case["kind"] == "lrfu":
            st.carried = torch.randn(N, generator=gen, device=DEVICE).mul_(0.5).exp_()
            st.carried.mul_(float(s.mean()))
            st.ks = torch.empty_like(s)
            st.hit = torch.empty(N, dtype=torch.uint8, device=DEVICE)
    return st


def _bits(kv):
    return kv.view(torch.int16)   # rows are moved bit for bit


def run(st):
    case, p = st.case, getattr(st, "p", None)
    kind = case["kind"]
    if kind == "monitor":
        conf = actkv.token_confidence(st.logits, TOP_K)
        b = actkv.budget_update(st.conf, st.offsets, st.budgets, CONF_WINDOW, CONF_STRIDE,
                                offsets_d=st.offsets_d)
        return {"conf": conf, "budgets": b["budgets"], "slopes": b["slopes"],
                "thresholds": b["thresholds"], "retained": b["retained"]}
    if kind == "decode":
        st.acc.copy_(st.scores)   # the aggregate so far, which a pass adds to in place
        acc = actkv.score_accumulate(p, st.q, st.kv, st.table, st.acc, lse=st.lse, ws=st.ws)
        return {"acc": acc}
    st.bt.copy_(st.table)
    if kind == "step":
        o = actkv.step(p, st.q, st.kv, st.bt, st.free, lse=st.lse, scores=st.scores, ws=st.ws)
        return {"scores": st.scores, "freed": o["freed"], "new_lens": o["new_lens"],
                "table": st.bt, "kv": _bits(st.kv)}
    if kind == "fresh":
        o = actkv.select_compact(p, st.scores, st.kv, st.bt, st.free, ws=st.ws)
        return {"freed": o["freed"], "new_lens": o["new_lens"], "table": st.bt,
                "kv": _bits(st.kv)}
    if kind == "inplace":
        kept, _ = actkv.select(p, st.scores, ws=st.ws, want_pooled=False)
        o = actkv.compact_inplace(st.planned, st.kv, st.bt, kept, ws=st.ws)
        return {"kept": kept, "freed": o["freed"], "new_lens": o["new_lens"],
                "order": o["new_order"], "table": st.bt, "kv": _bits(st.kv)}
    st.ks.copy_(st.carried)   # the keep scores carried over, which a pass updates in place
    o = actkv.lrfu_select(p, st.scores, st.ks, TOP_P, DECAY, hit=st.hit, ws=st.ws)
    freed, lens = actkv.compact(st.planned, st.kv, st.bt, o["kept"], st.free, ws=st.ws)
    return {"kept": o["kept"], "ks": st.ks, "ks_kept": o["ks_kept"], "hit": st.hit,
            "freed": freed, "new_lens": lens, "table": st.bt, "kv": _bits(st.kv)}


def work(case):
    if case["kind"] == "monitor":
        tokens = int(_traces(case)[-1])
        R, V = case["reqs"], case["vocab"]
        return {"bytes": 4 * R * V + 4 * tokens + 32 * R, "flops": 4 * R * V}
    L, n, b = _shape(case)
    R, Hq, Hkv, D = case["reqs"], case["q_heads"], case["kv_heads"], case["head_dim"]
    k = np.minimum(b.reshape(R, Hkv).astype(np.int64), L[:, None])
    N, kept = int(L.astype(np.int64).sum()) * Hkv, int(k.sum())
    table = 4 * int((-(-L // PAGE)).sum())
    nbytes, flops = 0, 0
    if case["kind"] in ("step", "decode"):
        nbytes += 2 * N * D + 2 * int(n.sum()) * Hq * D + 4 * N   # K, Q, the scores written
        if case["lse"] or case["kind"] == "decode":
            nbytes += 4 * int(n.sum()) * Hq
        pairs = int((L.astype(np.int64) * n).sum()) * Hq
        flops += 2 * D * pairs * (1 if case["lse"] or case["kind"] == "decode" else 2)
    if case["kind"] == "decode":
        return {"bytes": nbytes + 4 * N + table, "flops": flops}
    if case["kind"] in ("fresh", "inplace", "lrfu"):
        nbytes += 4 * N
    if case["kind"] == "lrfu":
        nbytes += 9 * N + 4 * kept
    nbytes += 3 * table + 4 * kept + 4 * R * Hkv
    moved = kept
    if case["kind"] == "inplace":
        # survivors already in the tail region stay: their share is that of the kept entries
        X = -(-k.max(1) // PAGE)
        start = (-(-L // PAGE) - X) * PAGE
        inside = np.minimum(start[:, None] + k, L[:, None]) - start[:, None]
        moved = int((k * (1 - inside / L[:, None])).sum())
    return {"bytes": nbytes + 8 * D * moved, "flops": flops}


def tolerance(case):
    """Four times the error measured against exact().  Scores: 1.0e-7 to 1.8e-7 with the LSE
    given, 5.2e-7 with the library's (at most 5.4e-7 and 1.0e-6 for a single value).  Two scores
    that close at the edge of a selection may change places, and the rows between them then
    move by one: at most 0.12% of the pool's values when they did.  A selection or keep score
    from given scores, and what is moved by it, has one right answer."""
    kind = case["kind"]
    if kind == "step":
        return {"rel": 2e-6, "max": 4e-6, "differ": 0.005}
    if kind == "decode":
        return {"rel": 1e-6, "max": 4e-6}
    if kind == "monitor":
        return {"rel": 2e-7, "max": 1e-6}
    return "exact"


def exact(case, seed):
    """What run() returns, in 64 bits and plain torch; None for what is moved or chosen."""
    st = prepare(case, seed)
    kind = case["kind"]
    if kind == "monitor":
        x = st.logits.double()
        top = torch.topk(x, min(TOP_K, x.shape[1]), 1).values
        out = {"conf": torch.logsumexp(x, 1) - top.mean(1), "budgets": None, "retained": None}
        conf, off = st.conf.cpu().numpy().astype(np.float64), st.offsets
        slopes, thresholds = [], []
        for r in range(case["reqs"]):
            t = conf[off[r]:off[r + 1]]
            w = np.lib.stride_tricks.sliding_window_view(t, CONF_WINDOW)[::CONF_STRIDE].min(1)
            q = np.percentile(w, 10)
            m = np.nonzero(w <= q)[0].astype(np.float64)
            y = w[w <= q]
            d = m - m.mean()
            slopes.append(float((d * (y - y.mean())).sum() / (d * d).sum()) if len(m) > 1 else 0.0)
            thresholds.append(float(q))
        out["slopes"] = torch.tensor(slopes, dtype=torch.float64)
        out["thresholds"] = torch.tensor(thresholds, dtype=torch.float64)
        return out
    moved = {"freed": None, "new_lens": None, "table": None, "kv": None}
    if kind in ("fresh", "inplace"):
        return None
    R, Hkv = case["reqs"], case["kv_heads"]
    if kind == "lrfu":
        ks = torch.empty(st.scores.numel(), dtype=torch.float64, device=DEVICE)
        off = 0
        w = case["window"]
        for r in range(R):
            for h in range(Hkv):
                seg = slice(off, off + int(st.L[r]))
                off = seg.stop
                s = st.scores[seg].double()
                att = torch.nn.functional.max_pool1d(s[None, None], w, 1, w // 2)[0, 0]
                order = torch.sort(att, descending=True, stable=True).indices
                mass = torch.cumsum(att[order], 0)
                hits = int((mass < float(np.float32(TOP_P)) * float(mass[-1])).sum()) + 1
                ks[seg] = DECAY * st.carried[seg].double()
                ks[seg].index_add_(0, order[:hits], att[order[:hits]])
        return {"kept": None, "ks": ks, "ks_kept": None, "hit": None, **moved}
    parts = []
    G = case["q_heads"] // Hkv
    for r in range(R):
        n = int(st.n[r])
        for h in range(Hkv):
            lse, s = _row_lse(_queries(st, r, h), _keys(st, r, h), n, st.scale, torch.float64)
            if st.lse is not None:
                lse = st.lse[int(st.cu[r]):int(st.cu[r + 1]), h * G:(h + 1) * G].reshape(-1).double()
            pr = s.sub_(lse[:, None]).exp_()
            if case["agg"] == "max_mean":
                pr = pr.view(n, G, -1).amax(1)
                # a decode step adds its maximum; a step takes the mean over its queries
                parts.append(pr.sum(0) if kind == "decode" else pr.mean(0))
            else:
                parts.append(pr.sum(0))
    scores = torch.cat(parts)
    if kind == "decode":
        return {"acc": st.scores.double() + scores}
    return {"scores": scores, **moved}
