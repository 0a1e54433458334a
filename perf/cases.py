"""Performance cases: the layer call of prefix-cached prefill attention, from one
short request to whole waves of the 13B-class geometry, and the host control
plane that forms the waves.

A case is a dict of plain values.  ``prepare`` builds what a serving program
holds before the call (tensors, page pools, block table, plan, workspace),
``run`` makes one pass through the public entry points, ``work`` counts the
bytes and operations one pass cannot do without.  ``listed`` names the fixed
cases; ``draw`` gives further ones from the same ranges.
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_2605_08581_amd import binding as B
from paper_2605_08581_amd import replay as R
from paper_2605_08581_amd import trace as T
from paper_2605_08581_amd import workload as W

# Head geometries (query heads, kv heads, head dim) of the configurations and tests.
MHA13B, GQA4B = (40, 40, 128), (32, 8, 128)
GEOMETRIES = (MHA13B, GQA4B, (8, 2, 128), (32, 8, 64), (4, 4, 64), (8, 1, 64))

# What one drawn pass may cost at most: operations as in the full-recompute wave
# listed below, bytes as in the wave that runs through forty layers.
MAX_FLOPS, MAX_BYTES = 3.0e12, 1.0e10


def _heads(g):
    return {"hq": g[0], "hkv": g[1], "d": g[2]}


def listed():
    return [
        # The smallest configuration: four short requests, head dim 64.  Launches and host time.
        {"name": "tiny", "kind": "config", "index": 0, **_heads((4, 4, 64))},
        # One user's turn in a conversation: one request, a cached prefix that ends inside a page.
        {"name": "one-request", "kind": "wave", **_heads(GQA4B), "batch": 1, "p_lo": 1003, "p_hi": 1003,
         "s_lo": 37, "s_hi": 37, "align": False, "wave_seed": 1},
        # A decode step of a small batch: one new token each over ragged cached lengths, grouped heads.
        {"name": "decode-gqa-16", "kind": "wave", **_heads(GQA4B), "batch": 16, "p_lo": 300, "p_hi": 4100,
         "s_lo": 1, "s_hi": 1, "align": False, "wave_seed": 2},
        # A decode step of a full batch of the 13B-class model: all K/V of 64 x 4096 tokens is read.
        {"name": "decode-mha-64", "kind": "wave", **_heads(MHA13B), "batch": 64, "p_lo": 4096, "p_hi": 4096,
         "s_lo": 1, "s_hi": 1, "align": True, "wave_seed": 3},
        # The 4B-class wave: grouped heads, 16 requests, Zipf-shared prefixes.
        {"name": "4b-gqa", "kind": "config", "index": 1, **_heads(GQA4B)},
        # The 13B-class wave (the benchmark's headline): 32 requests, long shared prefixes, short suffixes.
        {"name": "13b-mha", "kind": "config", "index": 2, **_heads(MHA13B)},
        # The hit-rate sweep's ends: no cached prefix at all, and nine tenths cached.
        {"name": "full-recompute", "kind": "hit", "hit": 0.0, "batch": 32, **_heads(MHA13B), "wave_seed": 4},
        {"name": "hit-0.9", "kind": "hit", "hit": 0.9, "batch": 32, **_heads(MHA13B), "wave_seed": 5},
        # Long-context retrieval: 8 requests of 16k to 32k cached tokens, permuted pages, split keys.
        {"name": "long-rag", "kind": "config", "index": 4, **_heads(GQA4B)},
        # Chunked prefill at head dim 64: chunks of a few hundred tokens on odd boundaries; the
        # append and the attention called one after the other.
        {"name": "chunked-d64", "kind": "wave", **_heads((32, 8, 64)), "batch": 12, "p_lo": 130, "p_hi": 3000,
         "s_lo": 200, "s_hi": 512, "align": False, "entry": "separate", "wave_seed": 6},
        # One wave of the serving replay through a whole model: a plan made for the wave (as every
        # wave needs), the block table sent over, then one call per layer.
        {"name": "serve-wave-40-layers", "kind": "wave", **_heads(MHA13B), "batch": 7, "p_lo": 0, "p_hi": 300,
         "s_lo": 500, "s_hi": 700, "align": True, "layers": 40, "plan_each_pass": True, "wave_seed": 7},
        # The control plane alone: scheduler rounds and radix-tree admissions of a Poisson trace.
        {"name": "control-plane", "kind": "replay", "requests": 640, "qps": 60.0, "policy": "dart", "budget": 16,
         "pages": 6144},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    if rng.random() < 0.08:
        return {"kind": "replay", "requests": _log_int(rng, 48, 512), "qps": round(rng.uniform(30.0, 80.0), 1),
                "policy": rng.choice(["dart", "lru_active", "lru", "lfu"]), "budget": rng.choice([8, 16, 24]),
                "pages": _log_int(rng, 2500, 12000)}
    while True:
        g = rng.choice(GEOMETRIES)
        decode = rng.random() < 0.25
        p_hi = _log_int(rng, 16, 32768)
        s_hi = 1 if decode else _log_int(rng, 4, 4096)
        c = {"kind": "wave", **_heads(g), "batch": _log_int(rng, 1, 64),
             "p_lo": int(p_hi * rng.choice([0.0, 0.25, 0.75, 1.0])), "p_hi": p_hi,
             "s_lo": max(1, int(s_hi * rng.choice([0.1, 0.5, 1.0]))), "s_hi": s_hi,
             "align": rng.random() < 0.6, "entry": rng.choice(["prefill", "prefill", "prefill", "separate"]),
             "wave_seed": rng.randrange(1 << 20)}
        if rng.random() < 0.15:
            c["layers"], c["plan_each_pass"] = rng.choice([8, 24, 40]), True
        w = work(c)
        if w["flops"] <= MAX_FLOPS and w["bytes"] <= MAX_BYTES:
            return c


def _wave(case):
    """Request lengths, page sharing and block table of a case (host integers only)."""
    if case["kind"] == "config":
        return W.make_config(case["index"])
    geom = W.Geometry(case["hq"], case["hkv"], case["d"])
    if case["kind"] == "hit":
        return W.make_hit_rate_batch(case["hit"], seed=case["wave_seed"], batch=case["batch"], geom=geom)
    rng = np.random.default_rng(case["wave_seed"])
    prefix = rng.integers(case["p_lo"], case["p_hi"] + 1, size=case["batch"])
    if case["align"]:                               # hits end on a page boundary, as the radix tree gives them
        prefix = prefix // W.PAGE_SIZE * W.PAGE_SIZE
    suffix = rng.integers(case["s_lo"], case["s_hi"] + 1, size=case["batch"])
    # aligned waves share cached prefixes in pairs now and then; the others are requests of their own
    groups = [int(x) if case["align"] else -1 for x in rng.integers(0, max(1, case["batch"]) * 2, size=case["batch"])]
    return W.make_custom_batch("wave", geom, prefix.tolist(), suffix.tolist(), case["wave_seed"], share_groups=groups)


def work(case):
    if case["kind"] == "replay":
        # every prompt token read once (system prompt, five passages, a suffix of 60 to 160), its page id written
        tokens = case["requests"] * (20 + 5 * 128 + 110)
        return {"bytes": 4.0 * tokens + 4.0 * tokens / 16, "flops": 0.0}
    b = _wave(case)
    g, p = b.geom, b.geom.page_size
    P, S = b.prefix_len.astype(np.int64), b.suffix_len.astype(np.int64)
    cached = set()                                  # pages that hold cached tokens, each read once
    for r in range(b.batch):
        cached.update(int(x) for x in b.block_table[r, :-(-int(P[r]) // p)])
    row = 2 * g.head_dim                            # bytes of one head's row
    kv_read = len(cached) * p * 2 * g.num_kv_heads * row
    new = int(S.sum())
    append = 2 * 2 * new * g.num_kv_heads * row     # new K and V rows read, and written to the pool
    q_out = 2 * new * g.num_q_heads * row
    table = 4 * int((-(-(P + S) // p)).sum())
    flops = 4 * g.head_dim * g.num_q_heads * int((S * P + S * (S + 1) // 2).sum())
    n = case.get("layers", 1)
    return {"bytes": float(n * (kv_read + append + q_out + table)), "flops": float(n * flops)}


def tolerance(case):
    # bf16 inputs and outputs, probabilities rounded to bf16 for the second product; decisions of the
    # control plane are whole numbers
    return "exact" if case["kind"] == "replay" else {"rel": 1e-2}


def prepare(case, seed):
    if case["kind"] == "replay":
        trace = T.make_trace(case["requests"], case["qps"], seed=seed)
        cfg = R.ReplayConfig(policy=case["policy"], dispatch_budget=case["budget"], num_pages=case["pages"])
        return {"case": case, "trace": trace, "cfg": cfg}
    b = _wave(case)
    g = b.geom
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)

    def normal(*shape):                             # unit variance: what normalised projections give
        return torch.empty(shape, dtype=torch.bfloat16, device="cuda").normal_(generator=gen)

    layers, new = case.get("layers", 1), b.total_suffix
    shape = B.shape_of(b)
    state = {
        "case": case, "batch": b, "shape": shape, "layers": layers,
        "q": normal(new, g.num_q_heads, g.head_dim),
        "k": normal(new, g.num_kv_heads, g.head_dim), "v": normal(new, g.num_kv_heads, g.head_dim),
        # one pool per layer
        "k_pool": normal(layers, b.num_pages, g.num_kv_heads, g.page_size, g.head_dim),
        "v_pool": normal(layers, b.num_pages, g.num_kv_heads, g.page_size, g.head_dim),
        "out": torch.empty(new, g.num_q_heads, g.head_dim, dtype=torch.bfloat16, device="cuda"),
    }
    plan = B.Plan(shape, b.prefix_len, b.suffix_len, block_table=b.block_table)
    state["workspace"] = torch.empty(max(256, plan.prism_plan_workspace_bytes()), dtype=torch.uint8, device="cuda")
    if case.get("plan_each_pass"):
        plan.close()
        state["pinned_table"] = torch.from_numpy(b.block_table).pin_memory()
        state["table"] = torch.empty(b.block_table.shape, dtype=torch.int32, device="cuda")
    else:
        state["plan"] = plan
        state["table"] = torch.from_numpy(b.block_table).cuda()
    return state


def _run_replay(state):
    waves = []

    def on_wave(rec):
        waves.append((rec.requests, rec.hit_tokens, rec.prompt_tokens, rec.rows))

    res = R.replay(state["trace"], state["cfg"], on_wave)
    n = len(state["trace"].requests)
    # per request, in dispatch order: its id, wave, hit and prompt length; and its block-table row (at most 64 pages)
    per_request = np.full((n, 4), -1, dtype=np.int64)
    rows = np.full((n, 64), -1, dtype=np.int64)
    i = 0
    for w, (ids, hits, prompts, pages) in enumerate(waves):
        for j in range(len(ids)):
            per_request[i] = ids[j], w, hits[j], prompts[j]
            rows[i, :len(pages[j])] = pages[j]
            i += 1
    counts = np.asarray([res["waves"], res["hit_tokens"], res["prompt_tokens"], res["evicted_pages"],
                         res["evicted_nodes"], res["memory_stalls"]], dtype=np.int64)
    return {"per_request": per_request, "rows": rows, "counts": counts}


def run(state):
    if state["case"]["kind"] == "replay":
        return _run_replay(state)
    b, table = state["batch"], state["table"]
    each = bool(state["case"].get("plan_each_pass"))
    if each:
        plan = B.Plan(state["shape"], b.prefix_len, b.suffix_len, block_table=b.block_table)
        table.copy_(state["pinned_table"], non_blocking=True)
    else:
        plan = state["plan"]
    q, k, v, out, ws = state["q"], state["k"], state["v"], state["out"], state["workspace"]
    separate = state["case"].get("entry") == "separate"
    for layer in range(state["layers"]):
        k_pool, v_pool = state["k_pool"][layer], state["v_pool"][layer]
        if separate:
            plan.prism_kv_append(k, v, k_pool, v_pool, table)
            plan.prism_prefix_attention(q, k_pool, v_pool, table, out, ws)
        else:
            plan.prism_prefix_prefill(q, k, v, k_pool, v_pool, table, out, ws)
    if each:
        plan.close()
    return {"out": out, "k_pool": state["k_pool"], "v_pool": state["v_pool"]}
