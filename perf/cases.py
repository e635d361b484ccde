"""Performance cases of the decode path: what is timed, on which inputs, and what the results must be.

A case is a dict of plain values.  `call` names the entry points one pass goes through:

  step    kvd_step on one layer
  layers  kvd_step_layers over all layers of a decode step
  stages  kvd_score_select, kvd_cache_resolve and kvd_sparse_decode_attn one after another
  token   a whole decoding step of a growing sequence: kvd_step and kvd_append_kv per layer, then kvd_advance
  index   kvd_build_summaries and kvd_build_centroids of one layer, as after a prefill

Sizes: `layers` (over `stored_layers` layers of the host store), `batch` sequences of `context` tokens (with
`ragged` the later ones are shorter, down to half), `q_heads` / `kv_heads` of 128 elements, pages of `page`
tokens, `topk` pages selected per step, a GPU window of `window` pages per unit.  The queries drift
(`rho`) through a cycle of `queries`: a window that holds what the cycle selects is all hits once the cycle
has gone round, a smaller one has the steady stream of misses of a running decode.
"""
import math

import torch

from paper_2605_18071_amd import kvd

DEV = "cuda"
D = 128
ROOM = 4096                      # tokens a "token" case can grow before its sequences are cut back


def _case(name, call, **kw):
    c = dict(name=name, call=call, layers=1, stored_layers=1, batch=1, q_heads=32, kv_heads=8, dtype="bf16", page=16,
             context=32768, ragged=False, topk=128, window=1024, sink=0, recent=0, policy="lru", pool=0, centroids=0,
             rounds=0, queries=8, rho=0.9)
    c.update(kw)
    return c


def listed():
    return [
        # interactive chat with a short context: one sequence, everything resident, launch latency counts
        _case("one_sequence_4k", "step", dtype="f16", context=4096, topk=64, window=256),
        # all layers of a decode step of a small serving batch, several layers per launch
        _case("layers_32k", "layers", layers=8, stored_layers=2, batch=8),
        # the long-context serving batch the framework is quoted on, selected pages resident
        _case("batch16_128k", "step", batch=16, context=131072, topk=256, window=2048),
        # the same contexts with a window that is too small: every step fetches over the host link
        _case("misses_128k", "step", batch=4, context=131072, topk=256, window=1024, queries=64),
        # seven query heads per KV head, pages of 32, a large batch of sequences of different lengths
        _case("gqa7_64k", "step", dtype="f16", q_heads=28, kv_heads=4, batch=32, page=32, context=65536, ragged=True, topk=64,
              window=409, rho=0.95),
        # one sequence of a million tokens, the newest pages always selected
        _case("million_tokens", "step", page=64, context=1048576, topk=128, window=819, recent=64),
        # the finest pages: 32768 of them per sequence
        _case("page4_128k", "step", batch=4, page=4, context=131072, topk=1024, window=8192),
        # a page size that is no multiple of 16, ragged lengths, sink and recent pages
        _case("page24_ragged", "step", dtype="f16", q_heads=28, kv_heads=4, batch=8, page=24, context=50001, ragged=True,
              topk=85, window=400, sink=2, recent=4),
        # hierarchical index with lookahead eviction, missing pages fetched
        _case("clusters_128k", "step", batch=4, context=131072, topk=256, window=1024, centroids=4096, rounds=4,
              policy="lookahead", queries=64),
        # a growing conversation: step, append and advance
        _case("next_token_16k", "token", dtype="f16", layers=4, stored_layers=4, batch=4, context=16001, topk=128, window=640,
              sink=1, recent=4),
        # the index of a freshly prefilled sequence
        _case("build_index_128k", "index", context=131072, topk=256, window=256, centroids=4096, rounds=4),
        # a caller that goes through the stages one by one, small pages, a finite look-ahead pool
        _case("stages_page8_32k", "stages", batch=8, page=8, topk=256, window=1024, policy="lookahead", pool=320),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One case of the ranges above: 1 to 128 units, contexts of 2k to 1M tokens, budgets of 512 to 4096 tokens."""
    while True:
        c = _draw(rng)
        units = c["batch"] * c["kv_heads"]
        store = c["stored_layers"] * units * _pages(c) * c["page"] * 4 * D
        # no more than the listed cases take: 4 GiB of host store, 2 GiB of window, the traffic of the largest
        if store <= 1 << 32 and c["layers"] * units * c["window"] * c["page"] * 4 * D <= 1 << 31 and \
                work(c)["bytes"] <= (3e8 if c["call"] == "index" else 5e8) and work(c)["flops"] <= 2.5e11:
            return c


def _draw(rng):
    call = rng.choice(["step", "step", "step", "step", "layers", "stages", "token", "index"])
    page = rng.choice([4, 8, 16, 16, 16, 32, 64, rng.choice([6, 12, 20, 24, 40])])
    kv_heads = rng.choice([2, 4, 8])
    context = _log(rng, 2048, 300000 if page < 32 else 1048576)
    layers = {"layers": rng.randint(2, 8), "token": rng.randint(1, 6)}.get(call, 1)
    stored = layers if call == "token" else min(layers, 2)
    units = max(kv_heads, min(128, (1 << 23) // (context * stored), (1 << 20) // (layers * (context // page + 1))))
    batch = _log(rng, 1, max(1, units // kv_heads))
    hierarchical = call == "index" or (call in ("step", "stages") and rng.random() < 0.25)
    if hierarchical and context // page >= 16384:
        page = 16 if context < 262144 else 64
    pages = -(-context // page)
    topk = max(1, min(2048, pages, _log(rng, 512, 4096) // page))
    window = min(pages, max(topk, int(topk * rng.uniform(2.0, 8.0))))
    centroids = max(1, min(8192, pages // rng.choice([2, 3, 4, 8]))) if hierarchical else 0
    policy = rng.choice(["lru", "lookahead"])
    forced = 0 if centroids else rng.choice([0, 0, topk // 16])
    return _case("", call, layers=layers, stored_layers=stored, batch=batch, q_heads=kv_heads * rng.choice([1, 2, 4, 4, 5, 7, 8]),
                 kv_heads=kv_heads, dtype=rng.choice(["f16", "bf16"]), page=page, context=context, ragged=rng.random() < 0.5,
                 topk=topk, window=window, sink=forced, recent=forced, policy=policy,
                 pool=int(topk * 1.25) if policy == "lookahead" and rng.random() < 0.3 else 0, centroids=centroids,
                 rounds=rng.randint(2, 5) if centroids else 0, queries=rng.choice([8, 8, 48]), rho=rng.choice([0.9, 0.95]))


# ---- inputs --------------------------------------------------------------------------------------

def _dtype(c):
    return torch.float16 if c["dtype"] == "f16" else torch.bfloat16


def _lens(c):
    """Tokens of every sequence at the first pass."""
    n = c["context"]
    return [max(1, n - (b * n) // (2 * c["batch"]) - 3 * b) if c["ragged"] else n for b in range(c["batch"])]


def _pages(c):
    return -(-(c["context"] + (ROOM if c["call"] == "token" else 0)) // c["page"])


def _gen(seed, *stream):
    g = torch.Generator(device=DEV)
    n = int(seed)
    for s in stream:
        n = (n * 1000003 + s + 1) % (1 << 62)
    g.manual_seed(n)
    return g


def _queries(c, seed):
    """[queries][layers][batch][q_heads][D]: N(0, 1), drifting from one to the next."""
    g = _gen(seed, 0)
    shape = (c["layers"], c["batch"], c["q_heads"], D)
    q, got = torch.randn(shape, generator=g, device=DEV), []
    for _ in range(c["queries"]):
        got.append(q.to(_dtype(c)))
        q = c["rho"] * q + (1.0 - c["rho"]) * torch.randn(shape, generator=g, device=DEV)
    return torch.stack(got)


def _kv(c, seed, q0, layer, b):
    """[kv_heads][pages][2][page][D] of one sequence: N(0, 1), the keys of a page of importance rank r shifted along the
    first query's direction by 6 r^-1.1."""
    g, H, NP = _gen(seed, 1, layer, b), c["kv_heads"], _pages(c)
    kv = torch.randn((H, NP, 2, c["page"], D), generator=g, device=DEV, dtype=_dtype(c))
    u = q0[layer, b].float().reshape(H, -1, D).mean(1)
    u = u / u.norm(dim=-1, keepdim=True)
    rank = torch.argsort(torch.rand((H, NP), generator=g, device=DEV), dim=-1) + 1
    kv[:, :, 0] += (6.0 * rank.float().pow(-1.1)[:, :, None, None] * u[:, None, None, :]).to(kv.dtype)
    return kv


def _new_token(c, seed):
    """Keys and values of the appended tokens, [2][queries][layers][batch][kv_heads][D]."""
    return torch.randn((2, c["queries"], c["layers"], c["batch"], c["kv_heads"], D), generator=_gen(seed, 2), device=DEV, dtype=_dtype(c))


def prepare(case, seed):
    c, dt, NP, U = case, _dtype(case), _pages(case), case["batch"] * case["kv_heads"]
    L, B, H, P, k = c["layers"], c["batch"], c["kv_heads"], c["page"], c["topk"]
    q = _queries(c, seed)
    store = torch.empty((c["stored_layers"], B, H, NP, 2, P, D), dtype=dt, pin_memory=True)
    for l in range(c["stored_layers"]):
        for b in range(B):
            store[l, b].copy_(_kv(c, seed, q[0], l, b))
    s = dict(case=c, q=q, store=store, t=0, grown=0)
    s["summaries"] = torch.zeros((L, B, H, NP, D), dtype=dt, device=DEV)
    s["slots"] = torch.zeros((L, B, H, c["window"], 2, P, D), dtype=dt, device=DEV)
    s["out"] = torch.empty((L, B, c["q_heads"], D), dtype=torch.float32, device=DEV)
    s["lse"] = torch.empty((L, B, c["q_heads"]), dtype=torch.float32, device=DEV)
    x = kvd.Kvd(n_layers=L, batch=B, n_q_heads=c["q_heads"], n_kv_heads=H, page_size=P, max_pages=NP, topk_pages=k,
                capacity_max=c["window"], kv_dtype=dt, sink_pages=c["sink"], recent_pages=c["recent"], policy=c["policy"],
                lookahead_pool=c["pool"], index_centroids=c["centroids"], physical_layers=c["stored_layers"])
    s["kvd"] = x
    x.bind_summaries(s["summaries"])
    x.bind_host_store(store)
    x.bind_slot_pool(s["slots"])
    x.set_seq_lens(_lens(c))
    if c["centroids"]:
        s["centroids"] = torch.zeros((L, B, H, c["centroids"], D), dtype=dt, device=DEV)
        s["cluster_start"] = torch.zeros((L, U, c["centroids"] + 1), dtype=torch.int32, device=DEV)
        s["cluster_pages"] = torch.zeros((L, U, NP), dtype=torch.int32, device=DEV)
        x.bind_centroids(s["centroids"], s["cluster_start"], s["cluster_pages"])
    if c["call"] == "index":
        return s
    for l in range(L):
        x.build_summaries(l)
        if c["centroids"]:
            x.build_centroids(l, c["rounds"])
    if c["call"] == "stages":
        i32 = dict(dtype=torch.int32, device=DEV)
        s["sel_pages"], s["sel_slots"], s["hit_mask"] = (torch.empty((U, k), **i32) for _ in range(3))
        s["counts"] = torch.empty((U, 3), **i32)
        s["scores"] = torch.zeros((U, NP), dtype=torch.float32, device=DEV)
    if c["call"] == "token":
        s["new"] = _new_token(c, seed)
    # the decode that ran before: the window holds what the last queries selected
    for t in range(c["queries"]):
        for l in range(L):
            x.step(l, t, q[t, l], s["out"][l], s["lse"][l])
    s["t"] = c["queries"]
    torch.cuda.synchronize()
    return s


def run(s):
    c, x, t = s["case"], s["kvd"], s["t"]
    i = t % c["queries"]
    q, out, lse = s["q"][i], s["out"], s["lse"]
    s["t"] = t + 1
    if c["call"] == "step":
        x.step(0, t, q[0], out, lse)
        return {"out": out, "lse": lse}
    if c["call"] == "layers":
        x.step_layers(0, c["layers"], t, q, out, lse)
        return {"out": out, "lse": lse}
    if c["call"] == "stages":
        x.score_select(0, q[0], s["sel_pages"], s["scores"])
        x.cache_resolve(0, t, s["sel_pages"], s["sel_slots"], s["hit_mask"], counts=s["counts"])
        x.sparse_decode_attn(0, q[0], s["sel_pages"], s["sel_slots"], out, lse)
        return {"scores": s["scores"], "sel_pages": s["sel_pages"], "hit_mask": s["hit_mask"], "counts": s["counts"], "out": out, "lse": lse}
    if c["call"] == "token":
        for l in range(c["layers"]):
            x.step(l, t, q[l], out[l], lse[l])
            x.append_kv(l, s["new"][0, i, l], s["new"][1, i, l])
        x.advance()
        s["grown"] += 1
        if s["grown"] == ROOM:                      # the sequences are full: the next turn starts from the prompt again
            s["grown"] = 0
            x.set_seq_lens(_lens(c))
        return {"out": out, "lse": lse, "summaries": s["summaries"]}
    x.build_summaries(0)
    x.build_centroids(0, c["rounds"])
    return {"summaries": s["summaries"], "centroids": s["centroids"], "cluster_start": s["cluster_start"], "cluster_pages": s["cluster_pages"]}


def work(case):
    c, G = case, case["q_heads"] // case["kv_heads"]
    rows = selected = 0
    for n in _lens(c):
        valid = -(-n // c["page"])
        rows += c["kv_heads"] * (c["centroids"] or valid)
        selected += c["kv_heads"] * min(c["topk"], valid)
    row = 2 * D
    if c["call"] == "index":
        tokens = c["kv_heads"] * sum(_lens(c))
        valid = sum(-(-n // c["page"]) for n in _lens(c))
        return {"bytes": row * (tokens + 2 * c["kv_heads"] * valid + rows),
                "flops": 2 * D * c["rounds"] * c["kv_heads"] * valid * c["centroids"] + D * tokens}
    tokens = selected * c["page"]
    heads = c["batch"] * c["q_heads"]
    per_layer = row * (rows + 2 * tokens) + heads * D * 6
    flops = 2 * D * rows + 4 * D * G * tokens
    if c["call"] == "token":
        per_layer += 4 * c["batch"] * c["kv_heads"] * row
    return {"bytes": c["layers"] * per_layer, "flops": c["layers"] * flops}


def tolerance(case):
    """About four times the distance from the same in 64 bits: scores, logits and sums are fp32, the probabilities that
    multiply V keep 11 bits with fp16 pages (1.4e-4 seen in the output) and 16 bits or more with bf16 pages (1.8e-6).  An
    index is computed in 64 bits and rounded once.  `differ`: ties of scores or distances."""
    if case["call"] == "index":
        return {"rel": 1e-6, "max": 1e-3, "differ": 1e-5}
    t = {"rel": 6e-4, "max": 5e-3} if case["dtype"] == "f16" else {"rel": 1e-5, "max": 2e-4}
    if case["call"] == "stages":
        t["differ"] = 1e-3
    return t


# ---- the same in 64 bits -------------------------------------------------------------------------

def _round(x, dt):
    """float64 -> dt with one rounding: to fp32 by truncation with a sticky last bit, then to nearest even."""
    f = x.float()
    f = torch.where(f.double().abs() > x.abs(), torch.nextafter(f, torch.zeros_like(f)), f)
    bits = f.view(torch.int32)
    return torch.where(f.double() != x, bits | 1, bits).view(torch.float32).to(dt)


def _summaries(c, keys, n):
    """[H][pages][D] mean keys over the valid tokens, rounded to the KV type; zero for pages beyond the end."""
    H, NP, P = keys.shape[:3]
    tok = torch.arange(NP * P, device=DEV).reshape(NP, P, 1)
    live = (tok < n).double()
    total = torch.stack([(keys[h].double() * live).sum(1) for h in range(H)])
    return _round(total / live.sum(1).clamp(min=1.0), _dtype(c))


def _clusters(c, summ, valid):
    """Lloyd's k-means of one unit: (centroids in 64 bits, assignment)."""
    x, Nc = summ[:valid].double(), c["centroids"]
    at = ((torch.arange(Nc, dtype=torch.float64, device=DEV) + 0.5) * valid / Nc).floor().long()
    cent, assign = x[at].clone(), None
    for _ in range(c["rounds"]):
        assign = (cent.square().sum(1)[None, :] - 2.0 * (x @ cent.T)).argmin(1)
        total = torch.zeros_like(cent).index_add_(0, assign, x)
        size = torch.bincount(assign, minlength=Nc).double()[:, None]
        cent = torch.where(size > 0, total / size.clamp(min=1.0), cent)
    return cent, assign


def _select(c, score, assign, valid):
    """Selected pages of one unit, ascending."""
    k = min(c["topk"], valid)
    if assign is not None:
        rank = torch.empty_like(score, dtype=torch.long)
        rank[torch.sort(score, descending=True, stable=True).indices] = torch.arange(score.numel(), device=DEV)
        key = rank[assign] * valid + torch.arange(valid, device=DEV)
        return key.topk(k, largest=False).indices.sort().values
    s = score[:valid].clone()
    s[: c["sink"]] = math.inf
    s[max(0, valid - c["recent"]):] = math.inf
    return s.topk(k).indices.sort().values


def exact(case, seed):
    c, P = case, case["page"]
    G, H, scale = c["q_heads"] // c["kv_heads"], c["kv_heads"], 1.0 / math.sqrt(D)
    q_all = _queries(c, seed)
    q0, NP = q_all[0], _pages(c)
    L, B = c["layers"], c["batch"]
    out = torch.zeros((L, B, c["q_heads"], D), dtype=torch.float64, device=DEV)
    lse = torch.zeros((L, B, c["q_heads"]), dtype=torch.float64, device=DEV)
    summaries = torch.zeros((L, B, H, NP, D), dtype=torch.float64, device=DEV)
    scores = torch.zeros((B * H, NP), dtype=torch.float64, device=DEV)
    centroids = torch.zeros((L, B, H, c["centroids"], D), dtype=torch.float64, device=DEV)
    for b, n in enumerate(_lens(c)):
        valid = -(-n // P)
        for sl in range(c["stored_layers"]):
            kv = _kv(c, seed, q0, sl, b)
            summ = _summaries(c, kv[:, :, 0], n)
            for l in range(sl, L, c["stored_layers"]):
                summaries[l, b] = summ
                for h in range(H):
                    rows, assign = summ[h].double(), None
                    if c["centroids"]:
                        cent, assign = _clusters(c, summ[h], valid)
                        rows = _round(cent, _dtype(c)).double()
                        centroids[l, b, h] = rows
                    if c["call"] == "index":
                        continue
                    qg = q0[l, b, h * G:(h + 1) * G].double()
                    score = scale * (rows @ qg.mean(0))
                    if not c["centroids"]:
                        scores[b * H + h] = score
                    else:
                        scores.view(-1)[(b * H + h) * c["centroids"]:(b * H + h + 1) * c["centroids"]] = score
                    sel = _select(c, score, assign, valid)
                    tok = (sel[:, None] * P + torch.arange(P, device=DEV)).reshape(-1)
                    keys, vals = kv[h, sel, 0].reshape(-1, D).double(), kv[h, sel, 1].reshape(-1, D).double()
                    logits = torch.where(tok < n, scale * (qg @ keys.T), -math.inf)
                    out[l, b, h * G:(h + 1) * G] = torch.softmax(logits, -1) @ vals
                    lse[l, b, h * G:(h + 1) * G] = torch.logsumexp(logits, -1)
            if c["call"] == "token":
                # the pass has also appended a token to every sequence
                kv[:, n // P, 0, n % P] = _new_token(c, seed)[0, 0, sl, b]
                summaries[sl, b] = _summaries(c, kv[:, :, 0], n + 1)
    if c["call"] == "index":
        return {"summaries": summaries, "centroids": centroids, "cluster_start": None, "cluster_pages": None}
    if c["call"] == "stages":
        return {"scores": scores, "sel_pages": None, "hit_mask": None, "counts": None, "out": out, "lse": lse}
    if c["call"] == "token":
        # built over the sequence as it was prefilled: pages beyond its end are zero there and here
        return {"out": out, "lse": lse, "summaries": summaries}
    return {"out": out, "lse": lse}
