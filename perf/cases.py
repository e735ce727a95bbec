"""Timed cases of the eviction-step library: what its users have it do, through the public entry points.

A case is a dict of plain values; `path` names the call sequence:
  step        epicache_evict_step: score, top-M, in-place compaction of one batch of caches
  overlapped  epicache_evict_step_overlapped, the library choosing its chunks (what bench.py times)
  ragged      epicache_evict_step_ragged_overlapped: lengths and budgets in device memory, budgets from
              epicache_layer_budgets, selection per head or pooled over the heads of an item
  attn        epicache_evict_step_attn: the patch's own attention output with the step behind it
  snapkv      epicache_evict_step_snapkv: the block's last tokens as the scoring window
  keydiff     epicache_score_keydiff, epicache_topk, epicache_compact: the attention-free scorer
  episodes    epicache_episode_medoids and epicache_match_queries: the geometry of a conversation's segments

A batch item is one episode's cache of one layer; `layers` > 1 folds the layers into the batch, as a caller does that
evicts once per block, after the forward pass; `layers` = 1 is a caller that evicts layer by layer inside it.

The calls compact K and V in place.  Rows behind the kept ones stay as they were, so a further pass on the same state
is the next step of a prefill whose new block holds the same rows again.  The queries change from step to step, as the
patch's hidden states do: a state holds kTurns + n_batch - 1 sets of patch queries and step t takes sets
[t, t + n_batch).  Every step then drops rows all over the cache and takes in new ones, instead of settling on rows
that never move.
"""
import math
import random

import torch

from paper_2509_17396_amd import binding as ep

kTurns = 64   # steps until the queries repeat
kTopics = 8   # subjects of the cached conversation
kSinks = 4    # leading rows that draw attention from every query


def _cache_case(name, path, dtype, d, q_heads, kv_heads, layers, episodes, budget, block, patch, reduce, **more):
    case = {"name": name, "path": path, "dtype": dtype, "head_dim": d, "q_heads": q_heads, "kv_heads": kv_heads,
            "layers": layers, "episodes": episodes, "budget": budget, "block": block, "patch": patch, "reduce": reduce}
    case.update(more)
    return case


def listed():
    return [
        # the smallest call: one layer and one episode in fp32, the configuration of a first integration
        _cache_case("tiny_f32", "step", "f32", 64, 8, 2, 1, 1, 256, 128, 32, "max"),
        # a 3B-class model that evicts layer by layer inside its forward pass, four episodes
        _cache_case("layer_3b", "step", "bf16", 128, 24, 8, 1, 4, 2048, 2048, 64, "max"),
        # the SnapKV baseline on one layer of an 8B-class model, sizes that are no multiples of anything
        _cache_case("layer_snapkv", "snapkv", "bf16", 128, 32, 8, 1, 3, 3000, 1337, 64, "sum"),
        # one layer of a multi-head model whose head dimension is neither 64 nor 128
        _cache_case("layer_d96", "step", "bf16", 96, 32, 32, 1, 2, 1024, 1000, 64, "sum"),
        # the patch's forward pass with the step behind it on one layer of a small model (head_dim 64)
        _cache_case("layer_attn_d64", "attn", "bf16", 64, 32, 8, 1, 4, 2000, 1000, 50, "max", causal=1),
        # the same on four layers of an 8B-class model
        _cache_case("attn_8b", "attn", "bf16", 128, 32, 8, 4, 4, 4096, 4096, 128, "max", causal=1),
        # whole models, all layers in one call
        _cache_case("folded_3b", "overlapped", "bf16", 128, 24, 8, 28, 4, 2048, 2048, 64, "sum"),
        _cache_case("folded_8b", "overlapped", "bf16", 128, 32, 8, 32, 4, 4096, 4096, 128, "max"),
        # layers with budgets of their own and heads of uneven lengths, retention pooled over the heads of a layer
        _cache_case("ragged_7b", "ragged", "bf16", 128, 28, 4, 28, 8, 6000, 2048, 64, "sum", select="pooled"),
        # long contexts, many episodes, long patches: eight layers (a pipeline stage) of the largest configuration
        _cache_case("long_context", "overlapped", "bf16", 128, 32, 8, 8, 16, 16384, 8192, 256, "sum"),
        # the attention-free baseline over all layers of a 3B-class model
        _cache_case("keydiff_3b", "keydiff", "bf16", 128, 24, 8, 28, 4, 2048, 2048, 1, "sum"),
        # a long conversation's segments: clusters' centroids and medoids, then a batch of queries matched to them
        {"name": "episodes", "path": "episodes", "segments": 1873, "dim": 1024, "episodes": 10, "queries": 256},
    ]


def _log_int(rng, lo, hi):
    """An integer spread evenly over the logarithm of [lo, hi]."""
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi + 0.49)))))))


def _flops(case):
    """One Q.K^T over the whole batch."""
    heads = case["layers"] * case["episodes"] * case["q_heads"]
    return 2.0 * heads * case["patch"] * (case["budget"] + case["block"]) * case["head_dim"]


def _kv_bytes(case):
    elem = 4 if case["dtype"] == "f32" else 2
    return 2.0 * case["layers"] * case["episodes"] * case["kv_heads"] * (case["budget"] + case["block"]) * case["head_dim"] * elem


def draw(rng):
    path = rng.choice(["step", "step", "step", "overlapped", "overlapped", "ragged", "attn", "attn", "snapkv", "keydiff", "episodes"])
    if path == "episodes":
        return {"path": path, "segments": _log_int(rng, 40, 4000), "dim": rng.choice([100, 384, 768, 1024, 1536]),
                "episodes": rng.randint(2, 24), "queries": _log_int(rng, 1, 1000)}
    while True:
        dtype, d = "bf16", rng.choice([128, 128, 128, 64])
        if path == "step":
            dtype, d = rng.choice([("bf16", 128), ("bf16", 128), ("bf16", 64), ("bf16", rng.choice([80, 96, 256])),
                                   ("f32", rng.choice([64, 128]))])
        kv_heads = rng.choice([2, 4, 8, 8])
        group = rng.choice([1, 3, 4, 4, 7])
        # layer by layer, or all layers of a model (or of a pipeline stage) at once
        layers = rng.randint(4, 32) if path in ("overlapped", "ragged", "keydiff") else rng.choice([1, 1, 1, rng.randint(2, 8)])
        case = {"path": path, "dtype": dtype, "head_dim": d, "q_heads": kv_heads * group, "kv_heads": kv_heads,
                "layers": layers, "episodes": _log_int(rng, 1, 16), "budget": _log_int(rng, 256, 16384),
                "block": _log_int(rng, 128, 8192), "patch": rng.choice([32, 64, 64, 128, 256, rng.randint(20, 256)]),
                "reduce": rng.choice(["max", "sum"])}
        if path == "attn":
            case["causal"] = rng.choice([0, 1, 1])
        if path == "snapkv":
            case["patch"] = rng.choice([32, 64, 64, rng.randint(16, 128)])
        if path == "keydiff":
            case["patch"] = 1
        if path == "ragged":
            case["select"] = rng.choice(["per_head", "pooled", "pooled"])
        # no larger than the largest listed case; one layer in fp32, another head dimension or the attention at head
        # dimension 64 is no larger than what one call over a layer is
        most = 5e12 if dtype == "bf16" and d in (64, 128) else 6e9
        if path == "attn":
            most = 1.2e11 if d == 128 else 6e9
        if _flops(case) <= most and _kv_bytes(case) <= 12.5e9:
            return case


# The second stream of the overlapped calls: a program creates it once and keeps it.
_aux = None


def _aux_stream():
    global _aux
    if _aux is None:
        _aux = torch.cuda.Stream()
    return _aux


def _bits(t):
    """The cache's bits as whole numbers: the compaction copies rows, it computes nothing."""
    return t.view(torch.int32 if t.dtype == torch.float32 else torch.int16)


def _prepare_episodes(case, seed):
    g = torch.Generator(device="cuda").manual_seed(seed)
    n, dim, e, nq = case["segments"], case["dim"], case["episodes"], case["queries"]
    # what a sentence encoder returns: unit vectors, a topic's segments around the topic's direction
    topics = torch.randn(e, dim, device="cuda", generator=g)
    assign = torch.randint(0, e, (n,), device="cuda", generator=g, dtype=torch.int32)
    emb = torch.nn.functional.normalize(topics[assign.long()] + 1.2 * torch.randn(n, dim, device="cuda", generator=g), dim=1)
    about = torch.randint(0, e, (nq,), device="cuda", generator=g)
    queries = torch.nn.functional.normalize(topics[about] + 1.5 * torch.randn(nq, dim, device="cuda", generator=g), dim=1)
    out = {"centroids": torch.empty(e, dim, device="cuda"), "medoid": torch.empty(e, dtype=torch.int32, device="cuda"),
           "episode": torch.empty(nq, dtype=torch.int32, device="cuda"), "cosine": torch.empty(nq, device="cuda")}
    return {"path": "episodes", "emb": emb, "assign": assign, "n": e, "queries": queries, "out": out}


def _randn(g, *shape):
    return torch.randn(*shape, device="cuda", generator=g)


def _make_inputs(case, seed, rows):
    """The queries of every turn and K, V with the layers folded into the batch axis; K and V hold `rows` rows per head.

    Keys: runs of rows about one of a few topics, channels of unequal magnitude, leading rows that every query attends
    to.  Queries: one direction for a set's patch, the patch tokens scattered around it."""
    g = torch.Generator(device="cuda").manual_seed(seed)
    heads, d, p = case["kv_heads"], case["head_dim"], case["patch"]
    group, nb = case["q_heads"] // heads, case["layers"] * case["episodes"]
    dtype = torch.float32 if case["dtype"] == "f32" else torch.bfloat16
    sink = torch.nn.functional.normalize(_randn(g, 1, heads, 1, d), dim=-1)
    channel = torch.exp(0.3 * _randn(g, 1, heads, 1, d))
    sets = nb + kTurns - 1
    q = torch.empty(sets, heads * group, p, d, dtype=dtype, device="cuda")
    step = max(1, int(1e8 / (heads * group * p * d)))
    for i in range(0, sets, step):
        n = min(step, sets - i)
        x = 0.75 * _randn(g, n, heads, 1, 1, d) + 1.5 * _randn(g, n, heads, group, p, d) + 6.0 * sink.unsqueeze(2)
        q[i:i + n] = x.reshape(n, heads * group, p, d)
    k = torch.empty(nb, heads, rows, d, dtype=dtype, device="cuda")
    v = torch.empty_like(k)
    step = max(1, int(1e8 / (heads * rows * d)))
    for i in range(0, nb, step):
        n = min(step, nb - i)
        topic = 0.5 * _randn(g, kTopics, d)
        runs = torch.randint(0, kTopics, (rows // 96 + 1,), device="cuda", generator=g)
        x = topic[runs.repeat_interleave(96)[:rows]] + _randn(g, n, heads, rows, d)
        x *= channel
        x[:, :, :kSinks] += math.sqrt(d) * sink
        k[i:i + n] = x
        v[i:i + n] = _randn(g, n, heads, rows, d)
    return q, k, v


def prepare(case, seed):
    path = case["path"]
    if path == "episodes":
        return _prepare_episodes(case, seed)
    reduce = ep.REDUCE_MAX if case["reduce"] == "max" else ep.REDUCE_SUM
    nb, heads = case["layers"] * case["episodes"], case["kv_heads"]
    n_cached, budget, causal = case["budget"], case["budget"], case.get("causal", 0)
    if path == "ragged":
        # budgets that follow the layers' sensitivities; after earlier pooled steps a head holds more or less than that
        host = random.Random(case["layers"])  # the model's own, whatever it reads
        per_layer = ep.epicache_layer_budgets([host.uniform(0.35, 0.65) for _ in range(case["layers"])], 1.0, budget)
        budget = max(per_layer)
        n_cached = int(1.25 * budget)
        host = random.Random(seed)
        held = [[int(m * host.uniform(0.7, 1.25)) for _ in range(heads)] for m in per_layer for _ in range(case["episodes"])]
    n = n_cached + case["block"]
    q, k, v = _make_inputs(case, seed, n + (case["patch"] if causal else 0))
    turns = [q[t:t + nb] for t in range(kTurns)]
    prm = ep.make_params(turns[0], k, n_cached, case["block"], budget, reduce=reduce, causal_patch=causal)
    out = {"k": _bits(k), "v": _bits(v)}
    s = {"path": path, "prm": prm, "turns": turns, "turn": 0, "k": k, "v": v, "out": out}
    n_keep = min(budget, n)
    if path == "overlapped":
        s["aux"] = _aux_stream()
        ws = ep.epicache_overlapped_workspace_size(prm, 0)[0]
    elif path == "ragged":
        s["aux"] = _aux_stream()
        s["select"] = ep.SELECT_POOLED if case["select"] == "pooled" else ep.SELECT_PER_HEAD
        ws, n_keep, _ = ep.epicache_ragged_overlapped_workspace_size(prm, s["select"], 0)
        s["n_ctx"] = torch.tensor(held, dtype=torch.int32, device="cuda") + case["block"]
        s["budgets"] = torch.tensor([m for m in per_layer for _ in range(case["episodes"])], dtype=torch.int32, device="cuda")
        s["n_kept"] = out["n_kept"] = torch.zeros(nb, heads, dtype=torch.int32, device="cuda")
    elif path == "snapkv":
        ws = ep.epicache_snapkv_workspace_size(prm)
    else:
        ws = ep.epicache_workspace_size(prm)
    if path == "keydiff":
        s["scores"] = torch.empty(nb, heads, n, dtype=torch.float32, device="cuda")
    if path == "attn":
        s["attn"] = out["attn"] = torch.empty(nb, case["q_heads"], case["patch"], case["head_dim"], dtype=q.dtype, device="cuda")
    s["ws"] = torch.empty(max(ws, 256), dtype=torch.uint8, device="cuda")
    s["keep"] = out["keep"] = torch.full((nb, heads, n_keep), -1, dtype=torch.int32, device="cuda")
    return s


def run(s):
    path = s["path"]
    if path not in ("keydiff", "episodes"):
        q = s["turns"][s["turn"]]
        s["turn"] = (s["turn"] + 1) % kTurns
    if path == "step":
        ep.epicache_evict_step(s["prm"], q, s["k"], s["v"], s["ws"], keep_idx=s["keep"])
    elif path == "overlapped":
        ep.epicache_evict_step_overlapped(s["prm"], q, s["k"], s["v"], s["ws"], s["aux"], 0, keep_idx=s["keep"])
    elif path == "ragged":
        ep.epicache_evict_step_ragged_overlapped(s["prm"], s["select"], q, s["k"], s["v"], s["n_ctx"], s["budgets"],
                                                 s["n_kept"], s["ws"], s["aux"], 0, keep_idx=s["keep"])
    elif path == "attn":
        ep.epicache_evict_step_attn(s["prm"], q, s["k"], s["v"], s["attn"], s["ws"], keep_idx=s["keep"])
    elif path == "snapkv":
        ep.epicache_evict_step_snapkv(s["prm"], q, s["k"], s["v"], s["ws"], keep_idx=s["keep"])
    elif path == "keydiff":
        ep.epicache_score_keydiff(s["prm"], s["k"], s["scores"], s["ws"])
        ep.epicache_topk(s["prm"], s["scores"], s["keep"], s["ws"])
        ep.epicache_compact(s["prm"], s["keep"], s["k"], s["v"], s["ws"])
    else:
        out = s["out"]
        ep.epicache_episode_medoids(s["emb"], s["assign"], s["n"], out["centroids"], out["medoid"])
        ep.epicache_match_queries(s["queries"], out["centroids"], 0.2, out["episode"], out["cosine"])
    return s["out"]


def work(case):
    if case["path"] == "episodes":
        n, dim, e, nq = case["segments"], case["dim"], case["episodes"], case["queries"]
        return {"bytes": 4.0 * (n * dim + n + nq * dim + e * dim + e + 2 * nq),
                "flops": 5.0 * n * dim + 2.0 * nq * e * dim + 2.0 * (nq + e) * dim}
    elem = 4 if case["dtype"] == "f32" else 2
    d, budget, n = case["head_dim"], case["budget"], case["budget"] + case["block"]
    heads = case["layers"] * case["episodes"] * case["kv_heads"]
    rows = case["q_heads"] // case["kv_heads"] * case["patch"]
    keys = n + (case["patch"] / 2 if case.get("causal") else 0)
    # K is read whole and its kept rows are written; V's kept rows are read and written; kept indices
    per_head = d * elem * (n + budget + 2 * budget) + 4 * budget
    flops = 2.0 * rows * keys * d
    if case["path"] == "keydiff":
        flops = 5.0 * n * d
    else:
        per_head += rows * d * elem
    if case["path"] == "attn":
        # the attention reads V whole and writes its output
        per_head += d * elem * (n - budget + (2 * case["patch"] if case.get("causal") else 0)) + rows * d * elem
        flops *= 2
    return {"bytes": float(heads * per_head), "flops": float(heads * flops)}


def tolerance(case):
    if case["path"] == "episodes":
        return {"rel": 1e-5, "differ": 0.005}
    # Scores are 32-bit sums of exponentials and stay inside the step.  A row whose score lies within their rounding of
    # the last kept one may take its place, which moves the kept rows between the two by one.
    if case["path"] == "attn":
        return {"rel": 1e-2, "differ": 0.01}  # the attention's output is bf16
    return {"rel": 0.0, "differ": 0.01}
