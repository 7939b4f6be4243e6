"""Timed cases of the RNNLM scoring step: what a search has the library do, through its Python entry points.

A case is one of six kinds of pass:

  grouped  rnnlm_step_dedup: N raw queries, `unique` of them with distinct histories, full softmax
  rows     rnnlm_step: `rows` distinct histories the caller has told apart itself, N queries mapped to them
  cached   an utterance of `steps` steps through the cache kept between steps (reset, then rnnlm_step_cached)
  hs       rnnlm_hs_step: rows the caller has told apart, hierarchical (Huffman-tree) output layer
  hsgroup  rnnlm_step_dedup on a model with that output layer
  index    an index table: reset, N contexts interned by content, the same contexts fetched again

Sizes are those of workloads/configs.py where the comment says so, and generic otherwise.
"""
import math

import numpy as np
import torch

import paper_2007_11794_amd as rn

DEV = "cuda:0"


def listed():
    return [
        # The smallest call in earnest: a handful of hypotheses on a toy vocabulary; launches and host work are all of it
        # (workload 1).
        dict(name="tiny_f32", kind="grouped", V=1000, H=64, N=8, unique=8, K=4, dtype="f32", sigma=0.1, zipf=0.0),
        # A WSJ-sized vocabulary in fp32, one frame's new hypotheses (workload 2).
        dict(name="wsj_f32", kind="grouped", V=20000, H=256, N=256, unique=256, K=16, dtype="f32", sigma=0.05, zipf=1.1),
        # The headline step: large vocabulary, bf16 weights, all histories distinct (workload 3).
        dict(name="large_vocab_bf16", kind="grouped", V=65536, H=512, N=1024, unique=1024, K=32, dtype="bf16", sigma=0.03,
             zipf=1.1),
        # The same model kept in fp32 by a user who does not want rounded weights.
        dict(name="large_vocab_f32", kind="grouped", V=65536, H=512, N=1024, unique=1024, K=32, dtype="f32", sigma=0.03,
             zipf=1.1),
        # A step of a decode in which histories repeat: thousands of raw queries, 30 % distinct (workload 4).
        dict(name="decode_trace_bf16", kind="grouped", V=65536, H=512, N=4096, unique=1229, K=8, dtype="bf16", sigma=0.03,
             zipf=1.1),
        # The same search through the cache kept between steps, at the redundancy the paper reports (a tenth of the raw
        # queries distinct, nine tenths of them known from the step before): an utterance of eight steps.
        dict(name="cached_trace_bf16", kind="cached", V=65536, H=512, N=4096, unique=410, K=8, dtype="bf16", sigma=0.03,
             zipf=1.1, carry=0.9, steps=8, capacity=100000),
        # The largest: wide hidden layer, 200000 words, many words asked per history (workload 5).
        dict(name="stress_bf16", kind="grouped", V=200000, H=1024, N=2048, unique=2048, K=64, dtype="bf16", sigma=0.02,
             zipf=1.0),
        # A million words, the few histories a frame leaves behind a cache: bound by reading the weights (workload 6).
        dict(name="million_words_bf16", kind="rows", V=1000000, H=128, N=64, rows=64, K=32, dtype="bf16", sigma=0.05,
             zipf=1.1),
        # Sizes as they come: odd vocabulary, hidden layer of 650 units, odd batch, more queries than rows, and output
        # weights as large as training makes them, so that the log-sum-exp needs its running maximum.
        dict(name="ragged_bf16", kind="rows", V=30011, H=650, N=511, rows=317, K=11, dtype="bf16", sigma=0.2, zipf=1.1),
        # The paper's own output layer on the headline shape: paths through a Huffman tree.
        dict(name="tree_large_vocab_bf16", kind="hs", V=65536, H=512, N=1024, rows=1024, K=32, dtype="bf16", sigma=0.03,
             zipf=1.1),
        # The paper's regime: that output layer on a million words, few rows (workload 6).
        dict(name="tree_million_words_bf16", kind="hs", V=1000000, H=128, N=64, rows=64, K=32, dtype="bf16", sigma=0.05,
             zipf=1.1),
        # Contexts handed back and forth by index instead of by value: a step's contexts interned and fetched.
        dict(name="index_table", kind="index", H=512, N=4096, unique=1229, zipf=1.1, V=65536),
    ]


def _log_uniform(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def _hidden_size(rng, lo, hi):
    h = _log_uniform(rng, lo, hi)
    return h if rng.random() < 0.4 else max(lo, min(hi, (h + 32) // 64 * 64))


def draw(rng):
    kind = rng.choice(["grouped", "grouped", "grouped", "rows", "rows", "cached", "hs", "hsgroup", "index"])
    frac = rng.choice([1.0, 1.0, 0.3, 0.1])
    zipf = rng.choice([1.0, 1.1])
    if kind == "index":
        n = _log_uniform(rng, 64, 16384)
        return dict(kind=kind, H=_hidden_size(rng, 64, 1024), N=n, unique=max(1, int(frac * n)), zipf=zipf, V=65536)
    if kind in ("hs", "hsgroup"):
        v, n = _log_uniform(rng, 5000, 1000000), _log_uniform(rng, 16, 4096)
        c = dict(kind=kind, V=v, H=_hidden_size(rng, 64, 128 if v > 200000 else 512), N=n, K=_log_uniform(rng, 1, 32),
                 dtype=rng.choice(["bf16", "bf16", "f32"]), sigma=0.05, zipf=zipf)
        c["rows" if kind == "hs" else "unique"] = max(1, int(frac * n))
        return c
    dtype = rng.choice(["bf16", "bf16", "f32"])
    v = _log_uniform(rng, 1000, 1000000 if kind == "rows" else 200000)
    h = _hidden_size(rng, 64, 128 if v > 200000 else 1024)
    n = _log_uniform(rng, 256, 4096) if kind == "cached" else _log_uniform(rng, 1, 4096)
    c = dict(kind=kind, V=v, H=h, N=n, K=_log_uniform(rng, 1, 64), dtype=dtype, sigma=rng.choice([0.02, 0.05, 0.05, 0.2]),
             zipf=zipf)
    if kind == "cached":
        c.update(unique=max(1, int(rng.choice([0.3, 0.1]) * n)), carry=rng.choice([0.5, 0.9]), steps=8, capacity=100000)
    else:
        c["rows" if kind == "rows" else "unique"] = max(1, int(frac * n))
    # nothing beyond the largest listed case: weights of no more bytes, and fewer queries where the whole would be more work (an fp32 product is six
    # bf16 ones on the matrix cores; half the listed limit, for shapes that reach less of the card's rate)
    c["V"] = min(v, int(4.1e8) // (h * (2 if dtype == "bf16" else 4)))
    limit = 0.4e12 / (6 if dtype == "f32" else 1)
    while _flops(c) > limit:
        c["N"] = max(1, c["N"] // 2)
        key = "rows" if kind == "rows" else "unique"
        c[key] = max(1, c[key] // 2)
    return c


# ---- inputs

def _generator(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(1000003 * 7 + int(seed))
    return g


def _weights(g, shape, case):
    """Weights as the loader takes them: float32, or bfloat16 bit patterns, in host memory (pinned: it is copied from)."""
    w = torch.randn(shape, generator=g, device=DEV).mul_(case["sigma"])
    bf16 = case["dtype"] == "bf16"
    if bf16:
        w = w.to(torch.bfloat16).view(torch.int16)
    host = torch.empty(shape, dtype=w.dtype, pin_memory=True).copy_(w).numpy()
    return host.view(np.uint16) if bf16 else host


def _words(g, case, shape):
    """Word ids with p(rank r) ~ r^-zipf; 0: uniform."""
    u = torch.rand(shape, generator=g, device=DEV, dtype=torch.float64)
    if not case["zipf"]:
        return (u * case["V"]).to(torch.int32).clamp_(max=case["V"] - 1)
    mass = torch.arange(1, case["V"] + 1, device=DEV, dtype=torch.float64).pow_(-case["zipf"]).cumsum(0)
    return torch.searchsorted(mass / mass[-1], u, right=True).clamp_(max=case["V"] - 1).to(torch.int32)


def _hidden(g, rows, H):
    return torch.sigmoid(torch.randn((rows, H), generator=g, device=DEV))


def _model(g, case, max_b):
    V, H = case["V"], case["H"]
    kind = rn.RNNLM_BF16 if case["dtype"] == "bf16" else rn.RNNLM_F32
    U, W = _weights(g, (V, H), case), _weights(g, (H, H), case)
    if case["kind"] in ("hs", "hsgroup"):
        theta = _weights(g, (V - 1, H), case)
        off, entry = rn.rnnlm_huffman_build(np.arange(1, V + 1, dtype=np.float64) ** -case["zipf"])
        return rn.rnnlm_hs_load(V, H, kind, U, W, theta, off, entry, max_b)
    O = _weights(g, (H, V), case)
    bias = (torch.randn(V, generator=g, device=DEV) * case["sigma"]).cpu().numpy()
    return rn.rnnlm_load(V, H, kind, U, W, O, bias, max_b)


def _copies(g, n, unique):
    """Which of `unique` histories each of n raw queries carries: every one at least once, in random order."""
    src = torch.cat([torch.arange(unique, device=DEV),
                     torch.randint(0, unique, (n - unique,), generator=g, device=DEV)])
    return src[torch.randperm(n, generator=g, device=DEV)]


def _carried(case):
    return int(round(case["carry"] * case["unique"]))


def prepare(case, seed):
    g = _generator(seed)
    kind, H, N = case["kind"], case["H"], case["N"]
    i32 = dict(dtype=torch.int32, device=DEV)
    s = {"kind": kind}
    if kind == "index":
        src = _copies(g, N, case["unique"])
        s["word"], s["h"] = _words(g, case, (case["unique"],))[src].contiguous(), _hidden(g, case["unique"], H)[src].contiguous()
        s["table"] = rn.rnnlm_index_create(H, 4 * N, N)
        s["index"], s["word_out"], s["h_out"] = torch.zeros(N, **i32), torch.zeros(N, **i32), torch.zeros((N, H), device=DEV)
        return s
    K = case["K"]
    s["model"] = _model(g, case, N)
    if kind in ("rows", "hs"):
        B = case["rows"]
        s["prev"], s["h_in"] = _words(g, case, (B,)), _hidden(g, B, H)
        s["row"] = None if B == N else _copies(g, N, B).to(torch.int32)
        s["query"] = _words(g, case, (N, K))
        s["h_out"], s["logprob"] = torch.zeros((B, H), device=DEV), torch.zeros((N, K), device=DEV)
        return s
    # raw queries with 64-bit history ids: a context counter in the high half, as the search packs them
    T, U = case.get("steps", 1), case["unique"]
    s["steps"], ids, prev, h, fresh = [], None, None, None, 0
    for _ in range(T):
        new_ids = (torch.arange(fresh, fresh + U, device=DEV) << 32) | torch.randint(0, 1 << 31, (U,), generator=g, device=DEV)
        new_prev, new_h = _words(g, case, (U,)), _hidden(g, U, H)
        fresh += U
        if ids is not None:                       # these histories are still there from the step before
            keep = torch.randperm(U, generator=g, device=DEV)[:_carried(case)]
            new_ids[keep], new_prev[keep], new_h[keep] = ids[keep], prev[keep], h[keep]
        ids, prev, h = new_ids, new_prev, new_h
        src = _copies(g, N, U)
        s["steps"].append((ids[src].contiguous(), prev[src].contiguous(), h[src].contiguous(), _words(g, case, (N, K))))
    s["rep"], s["inverse"] = torch.zeros((T, N), **i32), torch.zeros((T, N), **i32)
    s["n_unique"] = torch.zeros((T, 1), **i32)
    s["h_out"], s["logprob"] = torch.zeros((T, N, H), device=DEV), torch.zeros((T, N, K), device=DEV)
    s["workspace"] = torch.empty(rn.rnnlm_dedup_workspace_bytes(N), dtype=torch.uint8, device=DEV)
    if kind == "cached":
        s["cache"] = rn.rnnlm_cache_create(s["model"], case["capacity"])
        s["stats"] = torch.zeros((T, 4), **i32)
    s["out"] = [tuple(s[k][t] for k in ("rep", "inverse", "n_unique", "h_out", "logprob")) for t in range(T)]
    return s


def run(s):
    kind = s["kind"]
    if kind == "index":
        s["table"].reset()
        rn.rnnlm_index_intern(s["table"], s["word"], s["h"], s["index"])
        rn.rnnlm_index_fetch(s["table"], s["index"], s["word_out"], s["h_out"])
        return s["index"], s["word_out"], s["h_out"]
    if kind == "rows":
        rn.rnnlm_step(s["model"], s["prev"], s["h_in"], s["query"], s["h_out"], s["logprob"], row_of_query=s["row"])
        return s["h_out"], s["logprob"]
    if kind == "hs":
        rn.rnnlm_hs_step(s["model"], s["prev"], s["h_in"], s["query"], s["h_out"], s["logprob"], row_of_query=s["row"])
        return s["h_out"], s["logprob"]
    if kind == "cached":
        s["cache"].reset()
        for t, (x, out) in enumerate(zip(s["steps"], s["out"])):
            rn.rnnlm_step_cached(s["model"], s["cache"], *x, *out, s["workspace"], step_stats=s["stats"][t])
        return s["rep"], s["inverse"], s["n_unique"], s["h_out"], s["logprob"], s["stats"]
    rn.rnnlm_step_dedup(s["model"], *s["steps"][0], *s["out"][0], s["workspace"])
    return s["rep"], s["inverse"], s["n_unique"], s["h_out"], s["logprob"]


# ---- the work of one pass

def _distinct_words(case, n):
    """Expected number of different words among n draws."""
    V = case["V"]
    if not case["zipf"]:
        return V * -math.expm1(n * math.log1p(-1.0 / V))
    p = np.arange(1, V + 1, dtype=np.float64) ** -case["zipf"]
    p /= p.sum()
    return float(-np.expm1(n * np.log1p(-p)).sum())


def _rows(case):
    """Histories computed in one pass, one number a step."""
    if case["kind"] in ("rows", "hs"):
        return [case["rows"]]
    if case["kind"] == "cached":
        return [case["unique"]] + [case["unique"] - _carried(case)] * (case["steps"] - 1)
    return [case["unique"]]


def _flops(case):
    if case["kind"] == "index":
        return 0.0
    V, H, N, K = case["V"], case["H"], case["N"], case["K"]
    total = 0.0
    for rows in _rows(case):
        total += 2.0 * rows * H * H + 2.0 * N * K * H
        if case["kind"] not in ("hs", "hsgroup"):
            total += 2.0 * rows * H * V
    return total


def work(case):
    kind, H, N = case["kind"], case["H"], case["N"]
    if kind == "index":
        # read: words and vectors of all contexts; written: the index of each, the distinct ones into the store, and
        # the contexts handed back
        return {"bytes": 8.0 * N * (1 + H) + 4.0 * N + 4.0 * case["unique"] * (1 + H), "flops": 0.0}
    V, K, es = case["V"], case["K"], 2 if case["dtype"] == "bf16" else 4
    total = 0.0
    for rows in _rows(case):
        total += es * H * H + rows * (4 + 8 * H) + es * H * _distinct_words(case, rows)      # W, prev, h, h', U rows
        total += 8.0 * N * K                                                                # words asked and answers
        if kind in ("hs", "hsgroup"):
            total += es * H * (_distinct_words(case, N * K) - 1)    # a tree's paths to n leaves pass n - 1 nodes at least
        else:
            total += es * H * V + 4.0 * V
        if kind in ("grouped", "hsgroup", "cached"):
            total += 12.0 * N + 4.0 * rows                                                  # ids, groups
        elif rows != N:
            total += 4.0 * N
    if kind == "cached":
        total += 4.0 * H * sum(case["unique"] - r for r in _rows(case))                     # stored vectors handed out
    return {"bytes": total, "flops": _flops(case)}


def tolerance(case):
    """Four times and more what the outputs differ by from the same computation in float64, seen over the ranges above:
    fp32 sums (rel up to 6e-7); on top of them, with bf16 weights and the full softmax, the hidden vectors rounded to
    bf16 in front of the matrix cores (rel 2e-7 to 2.5e-6 at weights of 0.05 and below, 3e-5 at weights of 0.2)."""
    if case["kind"] == "index":
        return "exact"
    if case["dtype"] == "bf16" and case["kind"] not in ("hs", "hsgroup"):
        return {"rel": 1e-5, "max": 4e-5} if case["sigma"] <= 0.05 else {"rel": 1e-4, "max": 4e-4}
    return {"rel": 2e-6, "max": 2e-5}
