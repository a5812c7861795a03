"""The work a scorer has this library do, as cases that can be timed and compared.

A case is one pass (or one episode of passes) of one attention layer while responses
stream in: appending the chunk to the persistent cache and attending to it, in 16 and in
8 bits, the prefill of prompts, and the layer's projection and rotation in front of it.
Head shapes, batch sizes, chunk sizes and length distributions are those of the five
workloads in paper_2509_25762_amd/workload.py and of the ranges around them.

All lengths of a case follow from its values; `seed` only makes the tensors: N(0, 1)
queries, keys, values and hidden rows and N(0, 1 / hidden) weights, in bf16.
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_2509_25762_amd import binding as ob

THETA = 500000.0

# One pass, `kind`:
#   step      oppo_chunk_step: append + attention of the chunk, 16-bit cache
#   step8     oppo_kv_append_fp8 + oppo_chunk_prefill_attn_fp8: the same over the 8-bit cache
#   episode   every pass of a batch from its first response chunk to its last one
#   prompt    oppo_kv_append + oppo_chunk_prefill_attn of whole prompts into empty slabs
#   proj      oppo_qkv_proj_rope_append: projection, rotation and cache write of the chunk
#   layer     proj, then oppo_chunk_prefill_attn
#   epilogue  oppo_qkv_rope_append behind a projection made elsewhere
# batch sequences hold ctx_lo .. ctx_hi tokens; of them a share `idle` has ended or sits the
# pass out, a share `short` ends within the pass (1 .. chunk rows), the others bring chunk rows.


def listed():
    llama = dict(q_heads=32, kv_heads=8, head_dim=128)
    return [
        # the smallest call: four short sequences, head size 64, no grouping
        dict(name="step tiny", kind="step", batch=4, q_heads=4, kv_heads=4, head_dim=64, chunk=32, ctx_lo=32, ctx_hi=64,
             short=0.0, idle=0.0, lengths=1),
        # token by token: the scorer follows the actor with no chunking at all
        dict(name="step c1", kind="step", batch=64, **llama, chunk=1, ctx_lo=2048, ctx_hi=8192, short=0.0, idle=0.0, lengths=2),
        # small chunks over many sequences (bound by reading the cache)
        dict(name="step c64", kind="step", batch=256, **llama, chunk=64, ctx_lo=513, ctx_hi=2500, short=0.25, idle=0.1,
             lengths=3),
        # the usual chunk, full batch, early in the response
        dict(name="step c256", kind="step", batch=64, **llama, chunk=256, ctx_lo=262, ctx_hi=1017, short=0.15, idle=0.0,
             lengths=4),
        # the end of a long-tailed batch: a few stragglers far into their responses
        dict(name="step stragglers c512", kind="step", batch=32, **llama, chunk=512, ctx_lo=4096, ctx_hi=9999, short=0.05,
             idle=0.88, lengths=5),
        # a wide layer with long contexts and large chunks: the largest pass
        dict(name="step wide c1024", kind="step", batch=16, q_heads=64, kv_heads=8, head_dim=128, chunk=1024, ctx_lo=1237,
             ctx_hi=8192, short=0.2, idle=0.0, lengths=6),
        # a batch of responses from first chunk to last, the thin passes at its end among them
        dict(name="episode c256", kind="episode", batch=64, **llama, chunk=256, ctx_lo=256, ctx_hi=1024, median=512, sigma=0.8,
             resp_lo=16, resp_hi=4096, lengths=7),
        # new sequences enter: their prompts are prefilled
        dict(name="prompt", kind="prompt", batch=32, **llama, ctx_lo=512, ctx_hi=2048, lengths=8),
        # the layer's projection for a full batch's chunk
        dict(name="proj c256", kind="proj", batch=64, **llama, hidden=4096, chunk=256, ctx_lo=262, ctx_hi=1017, short=0.15,
             idle=0.0, lengths=9),
        # projection and attention of a thin pass
        dict(name="layer thin c256", kind="layer", batch=6, **llama, hidden=4096, chunk=256, ctx_lo=600, ctx_hi=3000,
             short=0.35, idle=0.0, lengths=10),
        # rotation and cache write behind a library projection, small chunks
        dict(name="epilogue c64", kind="epilogue", batch=256, **llama, chunk=64, ctx_lo=513, ctx_hi=2500, short=0.25, idle=0.1,
             lengths=11),
        # small chunks through the 8-bit cache
        dict(name="step8 c64", kind="step8", batch=256, **llama, chunk=64, ctx_lo=513, ctx_hi=2500, short=0.25, idle=0.1,
             lengths=12),
    ]


def draw(rng):
    most = max(_cost(c) for c in listed())
    while True:
        kind = rng.choice(["step", "step", "step", "step8", "step8", "episode", "prompt", "proj", "layer", "epilogue"])
        q_heads, kv_heads, head_dim = rng.choice([(32, 8, 128), (32, 8, 128), (64, 8, 128), (8, 2, 128), (16, 4, 64), (4, 4, 64)])
        c = dict(kind=kind, batch=_log_int(rng, 1, 256), q_heads=q_heads, kv_heads=kv_heads, head_dim=head_dim)
        c["ctx_lo"] = _log_int(rng, 16, 6000)
        c["ctx_hi"] = min(12288, int(c["ctx_lo"] * rng.uniform(1.0, 3.0)))
        if kind != "prompt":
            c["chunk"] = _log_int(rng, 1, 1024)
        if kind == "episode":
            c["chunk"] = _log_int(rng, 32, 1024)
            c.update(median=_log_int(rng, 64, 2048), sigma=round(rng.uniform(0.5, 1.0), 2), resp_lo=8)
            c["resp_hi"] = min(8 * c["median"], 40 * c["chunk"])
        elif kind != "prompt":
            c.update(short=round(rng.uniform(0.0, 0.5), 2), idle=round(rng.choice([0.0, rng.uniform(0.0, 0.9)]), 2))
        if kind in ("proj", "layer"):
            c["hidden"] = 64 * _log_int(rng, 4, 128)
        c["lengths"] = rng.randrange(1 << 20)
        if kind in ("proj", "layer", "epilogue") and c["batch"] * c["chunk"] > 40000:
            continue
        if _cost(c) <= most:
            return c


def prepare(case, seed):
    dev = torch.device("cuda")
    gen = torch.Generator(device=dev)
    gen.manual_seed(seed)
    Hq, Hkv, D, kind = case["q_heads"], case["kv_heads"], case["head_dim"], case["kind"]
    ctx, rows = _lengths(case)
    batch, total, most_rows = len(ctx), int(rows.sum()), int(rows.max())

    def randn(*shape, scale=1.0):
        return torch.randn(shape, generator=gen, device=dev, dtype=torch.bfloat16).mul_(scale)

    desc = ob.make_desc(Hq, Hkv, D, 1.0 / math.sqrt(D))
    # slabs with a little room, on multiples of 64 slots (what the 8-bit cache asks for)
    slot_begin = np.concatenate([[0], np.cumsum((ctx + rows + 63) // 64 * 64)])
    slots = int(slot_begin[-1])
    s = dict(kind=kind, desc=desc, ctx=ctx.astype(np.int32), cu=np.concatenate([[0], np.cumsum(rows)]).astype(np.int32))
    if kind == "step8":
        scale = 6.0 / 448.0   # N(0, 1) values stay below 6
        codes = [torch.zeros(slots * Hkv * D, device=dev, dtype=torch.uint8) for _ in range(2)]
        s["cache"] = ob.KVCacheFp8(codes[0], codes[1], slot_begin, scale, scale)
        held = np.concatenate([[0], np.cumsum(ctx)])
        ob.oppo_kv_append_fp8(desc, s["cache"], held, randn(int(held[-1]), Hkv, D), randn(int(held[-1]), Hkv, D))
    else:
        s["cache"] = ob.KVCache(randn(slots, Hkv, D), randn(slots, Hkv, D), slot_begin, ctx)
    if kind == "episode":
        s.update(resp=rows.astype(np.int32), chunk=case["chunk"])
        per_pass = [np.clip(rows - t * case["chunk"], 0, case["chunk"]) for t in range(-(-most_rows // case["chunk"]))]
        first = np.concatenate([[0], np.cumsum([p.sum() for p in per_pass])])
        s["pass_rows"] = [slice(int(a), int(b)) for a, b in zip(first[:-1], first[1:])]
        ws_rows = max(int(p.sum()) for p in per_pass)
    else:
        ws_rows = total
    if kind in ("proj", "layer"):
        s["x"] = randn(total, case["hidden"])
        s["w"] = randn((Hq + 2 * Hkv) * D, case["hidden"], scale=1.0 / math.sqrt(case["hidden"]))
        s["proj_ws"] = torch.empty(ob.oppo_qkv_proj_workspace_bytes(desc, total), device=dev, dtype=torch.uint8)
        s["hidden"] = case["hidden"]
    elif kind == "epilogue":
        s["qkv"] = randn(total, Hq + 2 * Hkv, D)
    else:
        s["k"], s["v"] = randn(total, Hkv, D), randn(total, Hkv, D)
    if kind in ("proj", "layer", "epilogue"):
        s["q"] = torch.zeros((total, Hq, D), device=dev, dtype=torch.bfloat16)
    else:
        s["q"] = randn(total, Hq, D)
    if kind not in ("proj", "epilogue"):
        s["out"] = torch.zeros((total, Hq, D), device=dev, dtype=torch.bfloat16)
        s["ws"] = torch.empty(max(256, ob.oppo_workspace_bytes(desc, batch, ws_rows)), device=dev, dtype=torch.uint8)
    return s


def run(s):
    cache = s["cache"]
    cache.kv_len[:] = s["ctx"]   # the pass starts from the same prefix each time
    return _RUN[s["kind"]](s, s["desc"], cache)


def _run_step(s, desc, cache):
    ob.oppo_chunk_step(desc, cache, s["cu"], s["q"], s["k"], s["v"], s["out"], s["ws"])
    return s["out"], cache.k, cache.v


def _run_step8(s, desc, cache):
    ob.oppo_kv_append_fp8(desc, cache, s["cu"], s["k"], s["v"])
    ob.oppo_chunk_prefill_attn_fp8(desc, cache, s["cu"], s["q"], s["out"], s["ws"])
    return s["out"], cache.k, cache.v


def _run_episode(s, desc, cache):
    for t, r in enumerate(s["pass_rows"]):
        _, _, cu = ob.oppo_chunk_schedule(s["ctx"], s["resp"], s["chunk"], t)
        ob.oppo_chunk_step(desc, cache, cu, s["q"][r], s["k"][r], s["v"][r], s["out"][r], s["ws"])
    return s["out"], cache.k, cache.v


def _run_prompt(s, desc, cache):
    ob.oppo_kv_append(desc, cache, s["cu"], s["k"], s["v"])
    ob.oppo_chunk_prefill_attn(desc, cache, s["cu"], s["q"], s["out"], s["ws"])
    return s["out"], cache.k, cache.v


def _run_proj(s, desc, cache):
    ob.oppo_qkv_proj_rope_append(desc, cache, s["cu"], s["x"], s["hidden"], s["w"], s["q"], s["proj_ws"], THETA)
    return s["q"], cache.k, cache.v


def _run_layer(s, desc, cache):
    ob.oppo_qkv_proj_rope_append(desc, cache, s["cu"], s["x"], s["hidden"], s["w"], s["q"], s["proj_ws"], THETA)
    ob.oppo_chunk_prefill_attn(desc, cache, s["cu"], s["q"], s["out"], s["ws"])
    return s["q"], s["out"], cache.k, cache.v


def _run_epilogue(s, desc, cache):
    ob.oppo_qkv_rope_append(desc, cache, s["cu"], s["qkv"], s["q"], THETA)
    return s["q"], cache.k, cache.v


_RUN = dict(step=_run_step, step8=_run_step8, episode=_run_episode, prompt=_run_prompt, proj=_run_proj, layer=_run_layer,
            epilogue=_run_epilogue)


def work(case):
    """What a pass cannot do without: visible (query, key) pairs, two products of 2 D operations
    each per query head; cached keys and values of the sequences that take part read once, the
    chunk's rows read and written once."""
    Hq, Hkv, D, kind = case["q_heads"], case["kv_heads"], case["head_dim"], case["kind"]
    ctx, rows = _lengths(case)
    if kind == "episode":
        chunks = [(ctx + np.minimum(rows, t * case["chunk"]), np.clip(rows - t * case["chunk"], 0, case["chunk"]))
                  for t in range(-(-int(rows.max()) // case["chunk"]))]
    else:
        chunks = [(ctx, rows)]
    flops = nbytes = 0.0
    for before, new in chunks:
        n = float(new.sum())
        q_row, kv_row, cached = 2.0 * Hq * D, 4.0 * Hkv * D, float(before[new > 0].sum())   # bytes of a row in bf16
        if kind in ("proj", "layer"):
            n_out = (Hq + 2 * Hkv) * D
            flops += 2.0 * n * case["hidden"] * n_out
            nbytes += 2.0 * (n + n_out) * case["hidden"]
        elif kind == "epilogue":
            flops += 3.0 * n * (Hq + Hkv) * D
            nbytes += n * (q_row + kv_row)
        else:
            nbytes += n * (q_row + kv_row)   # queries, keys and values of the chunk
        if kind == "step8":
            nbytes += (n + cached) * kv_row / 2
        else:
            nbytes += n * kv_row + (cached * kv_row if kind not in ("proj", "epilogue") else 0.0)
        nbytes += n * q_row   # out, or the projection's queries
        if kind not in ("proj", "epilogue"):
            flops += 4.0 * D * Hq * float((new * before + new * (new + 1) / 2.0).sum())
    return {"bytes": nbytes, "flops": flops}


def tolerance(case):
    if case["kind"] in ("proj", "epilogue"):
        return {"rel": 7e-3}   # one bf16 rounding of fp32 sums: 1.7e-3 against float64
    if case["kind"] != "step8":
        return {"rel": 1e-2}   # bf16 softmax weights and results, fp32 sums: 2.2e-3 .. 2.4e-3 against float64
    # queries and softmax weights are rounded to 3 mantissa bits on the way: 3.8e-2 against float64 over the
    # stored values, 1.5e-2 between two ways of cutting the key ranges (another reference for the weights)
    return {"rel": 8e-2}


def _lengths(case):
    """(tokens held before the pass, new rows) per sequence."""
    r = np.random.default_rng(case["lengths"])
    B = case["batch"]
    held = r.integers(case["ctx_lo"], case["ctx_hi"], size=B, endpoint=True)
    if case["kind"] == "prompt":
        return np.zeros(B, dtype=np.int64), held
    if case["kind"] == "episode":
        n = np.rint(np.exp(math.log(case["median"]) + case["sigma"] * r.standard_normal(B)))
        return held, np.clip(n, case["resp_lo"], case["resp_hi"]).astype(np.int64)
    C = case["chunk"]
    rows = np.full(B, C, dtype=np.int64)
    u = r.random(B)
    ends = u < case["short"]
    rows[ends] = r.integers(1, C, size=int(ends.sum()), endpoint=True)
    rows[u >= 1.0 - case["idle"]] = 0
    if rows.sum() == 0:
        rows[0] = C
    return held, rows


def _cost(case):
    w = work(case)
    return max(w["bytes"] / 4e12, w["flops"] / 1e15)


def _log_int(rng, lo, hi):
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi + 0.5)))))))
