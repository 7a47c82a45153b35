"""The work that users of this library have it do, as cases that can be timed and compared.

A case is a dict of plain values.  Four kinds:

  session    one session of one attention layer: `append` new tokens behind `cached` retained ones (data
             plane), then `query` tokens against the grown cache (query plane), then the appended tokens
             are dropped again (host metadata only), so that every pass sees the same lengths
  batch      one ragged step over many sessions: a third of them append, the others are queried
  questions  a batch of registered questions with a shared prefix against one session
  top2       greedy token, runner-up and logit gap of logit rows

Sizes are those of the benchmark's workloads, the latency curves and the tests.  Inputs are i.i.d. N(0,1)
(what projected, position-encoded activations are stood in by throughout this repository), drawn on the GPU from
the seed alone.
"""
import math

import numpy as np
import torch

import paper_2605_13784_amd as sk

DEVICE = "cuda:0"

# layer shapes: (dtype, query heads, KV heads, head_dim)
SHAPES = [("bf16", 32, 8, 128), ("bf16", 64, 8, 128), ("bf16", 28, 4, 128), ("bf16", 12, 4, 128), ("bf16", 32, 8, 64),
          ("bf16", 14, 2, 64), ("f32", 4, 4, 64), ("f32", 8, 2, 128)]


def _session(name, shape, cached, append, query, own_kv=False, block=16, out="f32", frozen=0, evicted=0, shuffled=True):
    dtype, hq, hkv, d = shape
    return {"name": name, "kind": "session", "dtype": dtype, "hq": hq, "hkv": hkv, "dim": d, "cached": cached, "append": append,
            "query": query, "own_kv": own_kv, "block": block, "out": out, "frozen": frozen, "evicted": evicted, "shuffled": shuffled}


def listed():
    layer = ("bf16", 32, 8, 128)
    return [
        # one token of an answer decoded against a short session (the shortest context of the latency curves):
        # what a caller waits for per generated token, nearly all of it launches and fixed latency
        _session("decode_1_at_2600", layer, 2600, 0, 1, own_kv=True),
        # a question of odd length with its own K/V at the longer context of the same curves, bf16 results, 64-token blocks
        _session("query_23_at_14800", layer, 14800, 0, 23, own_kv=True, block=64, out="bf16"),
        # the benchmark's query plane: 32 tokens against 32,768 cached ones
        _session("query_32_at_32k", layer, 32768, 0, 32),
        # the benchmark's headline step: 256 new tokens, then the query
        _session("step_256_32_at_32k", layer, 32512, 256, 32),
        # a ragged update of a sliding window (frozen head, evicted tokens behind it, seven query heads per KV head,
        # bf16 results) and a short question with its own K/V
        _session("step_77_5_window_9001", ("bf16", 28, 4, 128), 9001, 77, 5, own_kv=True, block=64, out="bf16", frozen=500, evicted=1000),
        # a session is opened: its whole header in one append, then the first question
        _session("open_2600_16", layer, 0, 2600, 16, own_kv=True),
        # the long-context workload's step: 512 new tokens and a 16-token query at 131,072
        _session("step_512_16_at_128k", layer, 130560, 512, 16),
        # a head_dim 64 layer at the headline's length
        _session("step_256_16_d64_32k", ("bf16", 32, 8, 64), 32512, 256, 16),
        # the fp32 path at its workload's size
        _session("step_64_16_f32_1k", ("f32", 4, 4, 64), 960, 64, 16),
        # multi-tenant step: 48 sessions of 2K-64K cached tokens, 16 append 128-1024 tokens, 32 are queried with 8-64
        {"name": "batch_48_sessions", "kind": "batch", "dtype": "bf16", "hq": 32, "hkv": 8, "dim": 128, "block": 16, "sessions": 48,
         "shortest": 2048, "longest": 65536, "mix": 4},
        # 64 registered questions, 16 shared and 8 own tokens each, on the 70B-shaped layer at 65,536 cached tokens
        {"name": "questions_64_at_64k", "kind": "questions", "dtype": "bf16", "hq": 64, "hkv": 8, "dim": 128, "block": 16,
         "cached": 65536, "prefix": 16, "questions": 64, "suffix": 8},
        # the answers of that batch: 64 logit rows of a 128,256-entry vocabulary
        {"name": "top2_64_rows", "kind": "top2", "rows": 64, "vocab": 128256},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _draw_once(rng):
    kind = rng.choices(["query", "append", "step", "f32", "batch", "questions", "top2"], [4, 3, 4, 2, 2, 2, 2])[0]
    block = rng.choice([16, 16, 16, 64, 256])
    if kind in ("query", "append", "step"):
        shape = rng.choice([s for s in SHAPES if s[0] == "bf16"] + [("bf16", 32, 8, 128)] * 4)
        append = 0 if kind == "query" else _log_int(rng, 1, 2600)
        query = 0 if kind == "append" else _log_int(rng, 1, 128)
        opening = kind != "query" and rng.random() < 0.15
        cached = 0 if opening else _log_int(rng, 1024, 131072)
        window = not opening and rng.random() < 0.2
        c = _session("", shape, cached, append, query, own_kv=rng.random() < 0.5, block=block, out=rng.choice(["f32", "f32", "bf16"]),
                     frozen=min(500, cached) if window else 0, evicted=_log_int(rng, 10, 2000) if window else 0, shuffled=rng.random() < 0.7)
    elif kind == "f32":
        shape = rng.choice([s for s in SHAPES if s[0] == "f32"])
        c = _session("", shape, _log_int(rng, 128, 8192), rng.choice([0, _log_int(rng, 1, 256)]), _log_int(rng, 1, 64),
                     own_kv=rng.random() < 0.5, block=block, shuffled=rng.random() < 0.7)
    elif kind == "batch":
        c = {"kind": "batch", "dtype": "bf16", "hq": 32, "hkv": 8, "dim": 128, "block": block, "sessions": rng.randint(3, 48),
             "shortest": _log_int(rng, 256, 2048), "longest": _log_int(rng, 4096, 65536), "mix": rng.randrange(1 << 16)}
    elif kind == "questions":
        _, hq, hkv, d = rng.choice([("bf16", 64, 8, 128), ("bf16", 64, 8, 128), ("bf16", 32, 8, 128), ("bf16", 28, 4, 128), ("bf16", 32, 8, 64)])
        c = {"kind": "questions", "dtype": "bf16", "hq": hq, "hkv": hkv, "dim": d, "block": block, "cached": _log_int(rng, 2048, 65536),
             "prefix": rng.randint(0, 64), "questions": _log_int(rng, 2, 64), "suffix": rng.randint(1, 32)}
    else:
        c = {"kind": "top2", "rows": _log_int(rng, 1, 1024), "vocab": _log_int(rng, 1000, 131072)}
    c.pop("name", None)
    return c


def _cost(case):
    w = work(case)
    return max(w["bytes"] * 100, w["flops"])


def draw(rng):
    dearest = _cost(listed()[-3])          # the multi-tenant step
    while True:
        c = _draw_once(rng)
        if _cost(c) <= dearest:
            return c


# ---- what a case comes down to ----------------------------------------------------------------------

def _batch_items(case):
    """Lengths, operations and token counts of a multi-tenant step: (cached, op, tokens) per session."""
    r = np.random.RandomState(case["mix"])
    n = case["sessions"]
    ratio = max(1.0, case["longest"] / case["shortest"])
    lengths = [int(case["shortest"] * ratio ** u) for u in r.uniform(size=n)]
    n_app = max(1, n // 3)
    ops = [sk.SK_OP_APPEND] * n_app + [sk.SK_OP_QUERY_A if i % 4 == 3 else sk.SK_OP_QUERY_B for i in range(n - n_app)]
    counts = [int(x) for x in r.randint(128, 1025, size=n_app)] + [int(x) for x in r.randint(8, 65, size=n - n_app)]
    return list(zip(lengths, ops, counts))


def _attend(case, n, T, causal):
    """Bytes and operations of T tokens attending over n cached ones (and, causal, over each other)."""
    el = 2 if case["dtype"] == "bf16" else 4
    out = 2 if case.get("out") == "bf16" else 4
    kv = 2 * case["hkv"] * case["dim"] * el
    pairs = T * (n + (T + 1) / 2.0) if causal else T * n
    nbytes = n * kv + (T * kv if causal else 0) + T * case["hq"] * (case["dim"] * (el + out) + 4)
    return nbytes, 4.0 * case["dim"] * case["hq"] * pairs


def work(case):
    """Each input of each call read once, each result written once."""
    if case["kind"] == "top2":
        return {"bytes": case["rows"] * (case["vocab"] * 4.0 + 20), "flops": 0.0}
    nbytes = flops = 0.0

    def add(n, T, causal, committed=False):
        nonlocal nbytes, flops
        b, f = _attend(case, n, T, causal)
        nbytes += b + (T * 2 * case["hkv"] * case["dim"] * (2 if case["dtype"] == "bf16" else 4) if committed else 0)
        flops += f

    if case["kind"] == "session":
        if case["append"]:
            add(case["cached"], case["append"], True, committed=True)
        if case["query"]:
            add(case["cached"] + case["append"], case["query"], case["own_kv"])
    elif case["kind"] == "batch":
        for n, op, T in _batch_items(case):
            add(n, T, op != sk.SK_OP_QUERY_A, committed=op == sk.SK_OP_APPEND)
    else:                                   # questions: the cache once, the prefix's rows once, every suffix
        n, P, NQ, S = case["cached"], case["prefix"], case["questions"], case["suffix"]
        add(n, P, True)
        add(0, NQ * S, False)
        flops += 4.0 * case["dim"] * case["hq"] * NQ * S * (n + P + (S + 1) / 2.0)
        nbytes += NQ * S * 2 * case["hkv"] * case["dim"] * 2
    return {"bytes": nbytes, "flops": flops}


def tolerance(case):
    if case["kind"] == "top2":
        return "exact"                      # indices and copied logits; the gap is one fp32 subtraction
    if case["dtype"] == "f32":
        # against attention in 64 bits: 3.4e-7 of the norm at 1,024 keys, growing with the root of the length
        return {"rel": 5e-6, "max": 5e-5}
    # bf16 softmax weights: against attention in 64 bits 1.3e-3 to 1.7e-3 of the norm whatever the length, 2.3e-3 with
    # bf16 results; single values up to 0.016 of the rms, 0.038 where rows see only a few keys
    return {"rel": 9e-3, "max": 0.15}


# ---- inputs, and one pass ---------------------------------------------------------------------------

def _generator(seed):
    return torch.Generator(device=DEVICE).manual_seed(int(seed) & 0x7FFFFFFF)


def _normal(gen, shape, dtype):
    return torch.randn(shape, generator=gen, device=DEVICE, dtype=torch.float32).to(torch.bfloat16 if dtype == "bf16" else torch.float32)


def _qkv(gen, case, T):
    return (_normal(gen, (T, case["hq"], case["dim"]), case["dtype"]),) + tuple(
        _normal(gen, (T, case["hkv"], case["dim"]), case["dtype"]) for _ in range(2))


def _outputs(case, T):
    dt = torch.bfloat16 if case.get("out") == "bf16" else torch.float32
    return (torch.empty((T, case["hq"], case["dim"]), dtype=dt, device=DEVICE),
            torch.empty((T, case["hq"]), dtype=torch.float32, device=DEVICE))


def _pool(case, tokens, sessions, max_batch_tokens, seed, shuffled):
    """A pool for sessions of `tokens` tokens (a list), with room for one step's appends twice over."""
    B = case["block"]
    n_blocks = sum(-(-t // B) + 2 for t in tokens) + 2 * (-(-max_batch_tokens // B)) + 8
    pool = sk.Pool(case["dtype"], case["hq"], case["hkv"], case["dim"], B, n_blocks, max_sessions=sessions,
                   max_batch_tokens=max_batch_tokens)
    if shuffled:                            # a pool in service hands out blocks in no order
        pool.sk_pool_set_alloc_order(np.random.RandomState(seed & 0x7FFFFFFF).permutation(n_blocks))
    return pool


def _grow(pool, case, gen, sid, tokens, piece=1024):
    for t in range(0, tokens, piece):
        L = min(piece, tokens - t)
        k, v = (_normal(gen, (L, case["hkv"], case["dim"]), case["dtype"]) for _ in range(2))
        pool.sk_session_append(sid, None, k, v)


def prepare(case, seed):
    gen = _generator(seed)
    s = {"case": case}
    if case["kind"] == "top2":
        stride = -(-case["vocab"] // 4) * 4
        s["logits"] = (2.5 * torch.randn((case["rows"], stride), generator=gen, device=DEVICE))[:, :case["vocab"]]
        s["workspace"] = torch.empty(max(16, sk.lib().sk_top2_workspace_bytes(case["rows"], case["vocab"])), dtype=torch.uint8, device=DEVICE)
        s["outputs"] = sk.top2_outputs(case["rows"], DEVICE)
    elif case["kind"] == "session":
        held = case["cached"] + case["evicted"]
        pool = s["pool"] = _pool(case, [held + case["append"]], 1, max(1024, case["append"], case["query"]), seed, case["shuffled"])
        sid = s["sid"] = pool.sk_session_create()
        _grow(pool, case, gen, sid, held)
        if case["frozen"]:
            pool.sk_session_freeze(sid, case["frozen"])
        if case["evicted"]:
            pool.sk_session_evict_oldest(sid, case["evicted"])
        if case["append"]:
            s["append"] = _qkv(gen, case, case["append"])
            s["append_out"] = _outputs(case, case["append"])
        if case["query"]:
            q, k, v = _qkv(gen, case, case["query"])
            s["query"] = (q, k, v) if case["own_kv"] else (q, None, None)
            s["query_out"] = _outputs(case, case["query"])
    elif case["kind"] == "batch":
        items = _batch_items(case)
        total = sum(T for _, _, T in items)
        pool = s["pool"] = _pool(case, [n for n, _, _ in items], len(items), max(1024, total), seed, True)
        s["sids"] = [pool.sk_session_create() for _ in items]
        longest = max(n for n, _, _ in items)
        for t in range(0, longest, 1024):   # sessions grow in turn, so their blocks interleave
            for sid, (n, _, _) in zip(s["sids"], items):
                if n > t:
                    _grow(pool, case, gen, sid, min(1024, n - t))
        s["ops"] = [op for _, op, _ in items]
        s["cu"] = [int(x) for x in np.concatenate([[0], np.cumsum([T for _, _, T in items])])]
        s["qkv"] = _qkv(gen, case, total)
        s["out"] = _outputs(case, total)
        s["grown"] = [(sid, n) for sid, (n, op, _) in zip(s["sids"], items) if op == sk.SK_OP_APPEND]
    else:
        n, P, NQ, S = case["cached"], case["prefix"], case["questions"], case["suffix"]
        pool = s["pool"] = _pool(case, [n], 1, max(1024, P + NQ * S), seed, True)
        s["sid"] = pool.sk_session_create()
        _grow(pool, case, gen, s["sid"], n)
        s["prefix"] = _qkv(gen, case, P) if P else (None, None, None)
        s["suffix"] = tuple(x.view(NQ, S, x.shape[1], case["dim"]) for x in _qkv(gen, case, NQ * S))
    return s


def run(s):
    case = s["case"]
    if case["kind"] == "top2":
        return sk.sk_top2(s["logits"], workspace=s["workspace"], outputs=s["outputs"])
    pool = s["pool"]
    if case["kind"] == "batch":
        out, lse = s["out"]
        pool.sk_batch_step(s["sids"], s["ops"], s["cu"], *s["qkv"], out=out, lse=lse)
        for sid, n in s["grown"]:
            pool.sk_session_truncate(sid, n)
        return out, lse
    if case["kind"] == "questions":
        return pool.sk_session_query_shared_prefix(s["sid"], *s["prefix"], *s["suffix"])
    sid, got = s["sid"], []
    if case["append"]:
        out, lse = s["append_out"]
        pool.sk_session_append(sid, *s["append"], out=out, lse=lse, out_dtype=case["out"])
        got += [out, lse]
    if case["query"]:
        out, lse = s["query_out"]
        pool.sk_session_query(sid, *s["query"], out=out, lse=lse, out_dtype=case["out"])
        got += [out, lse]
    if case["append"]:
        pool.sk_session_truncate(sid, case["cached"])
    return got
