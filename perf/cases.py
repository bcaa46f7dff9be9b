"""Workloads the TreeKV library is timed on: what a program around it calls, at the sizes it calls it with.

A case is a dict of plain values; its "path" says which entry points a pass goes through:

  decode    one generated token for every sequence of a batch through all layers of a model: treekv_decode_step once
            per layer, each layer its own full cache
  chunk     one prompt chunk into the full caches of a few layers: treekv_prefill_chunk once per layer
  sequence  a new prompt from its first token: treekv_reset, then treekv_prefill_chunk until it is in, the last chunk
            shorter; the caches fill during the first chunks and evict afterwards
  prompt    the paper's own prefilling stage: treekv_prefill_prompt, a whole prompt in one shot
  wavelet   the Haar analysis of a set of heads: treekv_wavelet_components

Inputs are drawn on the device from the seed with the recipe of paper_2501_04987_amd.inputs: N(0,1) plus a per-head
rank-8 part, so that a few slots carry most of the attention, as in a trained model (fp32 storage: plain N(0,1), as
the fp32 configuration has it).
"""
from __future__ import annotations

import math

import torch

from paper_2501_04987_amd import binding, inputs

CHUNK = 512        # tokens per prefill chunk of the configurations


def listed():
    return [
        # The tiny fp32 configuration: one layer, 2 heads x 64, 64 slots.  A step is all latency.
        dict(name="decode_tiny_f32", path="decode", layers=1, batch=1, kv_heads=2, group=1, head_dim=64, budget=64,
             dtype="f32", rerank=False),
        # Interactive generation, one sequence through the 32 layers of a Llama-7B-shaped model, 1024 slots.
        dict(name="decode_batch1", path="decode", layers=32, batch=1, kv_heads=32, group=1, head_dim=128, budget=1024,
             dtype="bf16", rerank=False),
        # The headline shape (batch 8, 2048 slots), 8 of its layers: more rows than any cache of the chip holds.
        dict(name="decode_batch8", path="decode", layers=8, batch=8, kv_heads=32, group=1, head_dim=128, budget=2048,
             dtype="bf16", rerank=False),
        # The same with positions re-assigned to cache ranks, which is how the paper runs its models.
        dict(name="decode_batch8_rerank", path="decode", layers=8, batch=8, kv_heads=32, group=1, head_dim=128,
             budget=2048, dtype="bf16", rerank=True),
        # Batched serving with grouped queries: 16 sequences, 32 query heads on 8 KV heads, 4096 slots.
        dict(name="decode_gqa", path="decode", layers=4, batch=16, kv_heads=8, group=4, head_dim=128, budget=4096,
             dtype="bf16", rerank=False),
        # Chunked prefill at steady state: 512 tokens into full 2048-slot caches of four layers.
        dict(name="chunk_512", path="chunk", layers=4, batch=1, kv_heads=32, group=1, head_dim=128, budget=2048,
             dtype="bf16", rerank=False, length=512),
        # The same with positions re-assigned.
        dict(name="chunk_512_rerank", path="chunk", layers=4, batch=1, kv_heads=32, group=1, head_dim=128, budget=2048,
             dtype="bf16", rerank=True, length=512),
        # A chunk with fp32 storage, ragged length.
        dict(name="chunk_f32", path="chunk", layers=1, batch=1, kv_heads=8, group=1, head_dim=64, budget=512,
             dtype="f32", rerank=False, length=200),
        # Two new requests of 6000 tokens each on a model with grouped queries and 64-wide heads: the caches fill,
        # then evict; the last chunk has 368 tokens.
        dict(name="sequence_gqa", path="sequence", batch=2, kv_heads=8, group=4, head_dim=64, budget=4096,
             dtype="bf16", rerank=False, length=6000),
        # A 32768-token prompt compressed in one shot into 2048 slots, blocks of 64.
        dict(name="prompt_32k", path="prompt", batch=1, kv_heads=32, group=1, head_dim=128, budget=2048, dtype="bf16",
             rerank=False, length=32768, block=64),
        # Two shorter prompts with grouped queries, positions re-assigned, blocks of 32.
        dict(name="prompt_gqa_rerank", path="prompt", batch=2, kv_heads=8, group=4, head_dim=128, budget=2048,
             dtype="bf16", rerank=True, length=12000, block=32),
        # The motivation's figure: 5 levels at step 512, 32 layers x 32 heads x 8 samples.
        dict(name="wavelet", path="wavelet", heads=8192, length=512, head_dim=128, levels=5, dtype="bf16"),
    ]


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    """One more case of the listed ranges: sizes over their logarithm, whatever number comes out."""
    path = rng.choice(["decode", "decode", "decode", "chunk", "chunk", "sequence", "prompt", "wavelet"])
    ref = [dict(c) for c in listed() if c["path"] == path]
    if path == "wavelet":
        levels = rng.randint(1, 5)
        c = dict(path=path, heads=_log_int(rng, 64, 8192), length=_log_int(rng, 2, 4096 >> levels) << levels,
                 head_dim=rng.choice([64, 128]), levels=levels, dtype=rng.choice(["bf16", "bf16", "f32"]))
        shrink = ["heads"]
    else:
        group = rng.choice([1, 1, 2, 4, 8])
        c = dict(path=path, batch=_log_int(rng, 1, 16), kv_heads=rng.choice([2, 4, 8, 16, 32]), group=group,
                 head_dim=rng.choice([64, 128, 128]), budget=_log_int(rng, 64, 4096), dtype="bf16",
                 rerank=rng.random() < 0.25)
        shrink = ["batch", "kv_heads"]
        if path in ("decode", "chunk"):
            c["layers"] = _log_int(rng, 1, 32 if path == "decode" else 4)
            c["dtype"] = rng.choice(["bf16"] * 4 + ["f32"])
            shrink.insert(0, "layers")
        if path == "chunk":
            c["length"] = _log_int(rng, 1, CHUNK)
            if c["dtype"] == "f32":                    # the fp32 chunk's own range
                c["budget"], c["length"] = _log_int(rng, 64, 1024), _log_int(rng, 1, 256)
        if path == "sequence":
            c["length"] = _log_int(rng, 100, 8192)
        if path == "prompt":
            c["block"] = rng.choice([b for b in (8, 16, 32, 64, 128) if b * group <= 128])
            c["budget"] = c["block"] * max(16, c["budget"] // c["block"])
            c["length"] = c["block"] * (_log_int(rng, 1024, 32768) // c["block"])
    # no dearer than the largest listed case of the path (for chunks, of the storage type: fp32 has a range of its own)
    if path == "chunk":
        ref = [r for r in ref if r["dtype"] == c["dtype"]]
    cap = {n: max(work(r)[n] for r in ref) for n in ("bytes", "flops")}
    for name in shrink:
        while c[name] > 1 and any(work(c)[n] > cap[n] for n in ("bytes", "flops")):
            c[name] = (c[name] + 1) // 2
    while any(work(c)[n] > cap[n] for n in ("bytes", "flops")):
        c["length"] = c["length"] // 2 // c.get("block", 1) * c.get("block", 1)
    return c


# ---------------------------------------------------------------------------------------------------------------
# what a program has in hand before the call
# ---------------------------------------------------------------------------------------------------------------
def _context(case, **kw):
    flags = binding.TREEKV_POSITION_RERANK if case["rerank"] else 0
    return binding.TreeKV(case["budget"], case["kv_heads"] * case["group"], case["head_dim"],
                          kv_heads=case["kv_heads"], batch=case["batch"], dtype=case["dtype"], flags=flags, **kw)


def _tokens(case, seed, n):
    """q [B, n, H, d], k and v [B, n, Hkv, d] of n consecutive tokens."""
    x = inputs.device_lowrank(seed, n, case["batch"], case["kv_heads"], case["group"], case["head_dim"],
                              beta=4.0 if case["dtype"] == "bf16" else 0.0, dtype=case["dtype"])
    return [t.transpose(0, 1).contiguous() for t in x]


def _filled(case, seed):
    """A context whose cache is full: as many tokens as it has slots, fed as chunks."""
    kv = _context(case, max_chunk=CHUNK)
    for at in range(0, case["budget"], CHUNK):
        n = min(CHUNK, case["budget"] - at)
        q, k, v = _tokens(case, seed + at, n)
        out, ret, nret, ev = kv.new_outputs(n)
        kv.prefill_chunk(q, k, v, n, out, ret, nret, ev)
    return kv


def prepare(case, seed):
    path, seed = case["path"], 1_000_003 * (int(seed) + 1)
    s = dict(path=path, t=0)
    if path == "wavelet":
        g = torch.Generator(device="cuda").manual_seed(seed)
        h, t, d = case["heads"], case["length"], case["head_dim"]
        s["a"] = torch.softmax(3.0 * torch.randn(h, t, device="cuda", generator=g), dim=-1).contiguous()
        v = torch.empty(h, t, d, dtype={"bf16": torch.bfloat16, "f32": torch.float32}[case["dtype"]], device="cuda")
        for lo in range(0, h, 1024):
            v[lo:lo + 1024] = torch.randn(min(1024, h - lo), t, d, device="cuda", generator=g)
        s["V"], s["levels"] = v, case["levels"]
        s["per_head"] = torch.empty(h, case["levels"], t, device="cuda")
        s["mean"] = torch.empty(case["levels"], t, device="cuda")
        return s
    if path == "prompt":
        q, k, v = _tokens(case, seed, case["length"])
        s["kv"] = _context(case, max_prompt=case["length"])
        s["qw"], s["k"], s["v"] = q[:, -case["block"]:].contiguous(), k, v
        s["length"], s["block"] = case["length"], case["block"]
        shape = (case["batch"], case["kv_heads"])
        s["ret"] = torch.empty(*shape, case["budget"], dtype=torch.int32, device="cuda")
        s["nret"] = torch.empty(*shape, dtype=torch.int32, device="cuda")
        s["ev"] = torch.empty(*shape, case["length"] // case["block"], dtype=torch.int32, device="cuda")
        s["tok"] = torch.empty(*shape, case["length"], device="cuda")
        return s
    if path == "sequence":
        s["kv"] = _context(case, max_chunk=CHUNK)
        s["chunks"] = []
        for at in range(0, case["length"], CHUNK):
            n = min(CHUNK, case["length"] - at)
            s["chunks"].append((*_tokens(case, seed + at, n), n, *s["kv"].new_outputs(n)))
        return s
    # decode and chunk: full caches, and a few tokens (chunks) to feed in turn
    s["layers"] = [_filled(case, seed + 10_007 * l) for l in range(case["layers"])]
    if path == "decode":
        s["out"] = [torch.stack([x] * case["layers"]) for x in s["layers"][0].new_outputs()]   # one tensor for all layers
        s["outs"] = [[x[l] for x in s["out"]] for l in range(case["layers"])]
        steps = [_tokens(case, seed + 10_007 * l + 9_001, 16) for l in range(case["layers"])]
        s["in"] = [[[x[:, t].contiguous() for x in layer] for layer in steps] for t in range(16)]
    else:
        s["length"] = case["length"]
        s["outs"] = [kv.new_outputs(case["length"]) for kv in s["layers"]]
        s["in"] = [[_tokens(case, seed + 10_007 * l + 9_001 + i, case["length"]) for l in range(case["layers"])]
                   for i in range(3)]
    return s


def run(s):
    path = s["path"]
    if path == "wavelet":
        return binding.wavelet_components(s["a"], s["V"], s["levels"], s["per_head"], s["mean"])
    if path == "prompt":
        s["kv"].prefill_prompt(s["qw"], s["k"], s["v"], s["length"], s["block"], s["ret"], s["nret"], s["ev"], s["tok"])
        return s["ret"], s["nret"], s["ev"], s["tok"]
    if path == "sequence":
        kv = s["kv"]
        kv.reset()
        for q, k, v, n, out, ret, nret, ev in s["chunks"]:
            kv.prefill_chunk(q, k, v, n, out, ret, nret, ev)
        return [c[4:] for c in s["chunks"]]
    x = s["in"][s["t"] % len(s["in"])]
    s["t"] += 1
    if path == "decode":
        for kv, (q, k, v), o in zip(s["layers"], x, s["outs"]):
            kv.decode_step(q, k, v, *o)
        return s["out"]
    n = s["length"]
    for kv, (q, k, v), o in zip(s["layers"], x, s["outs"]):
        kv.prefill_chunk(q, k, v, n, *o)
    return s["outs"]


# ---------------------------------------------------------------------------------------------------------------
# what a pass cannot do without, and how close two correct implementations come
# ---------------------------------------------------------------------------------------------------------------
def _chunk_work(case, n, L):
    """One chunk of L tokens into a cache that holds n: (bytes, flops) of one layer."""
    e, d, G, c = 2 if case["dtype"] == "bf16" else 4, case["head_dim"], case["group"], case["budget"]
    after = min(c, n + L)
    per_unit = (2 * n * d * e + 2 * L * d * e        # cached rows and the chunk's own, read
                + 2 * min(L, c) * d * e              # the chunk's rows that stay, written
                + L * G * d * (e + 4)                # queries read, outputs written
                + 4 * (n + after)                    # scores
                + 4 * n + 4 * c + 4 * L)             # positions read; retained and evicted lists written
    units = case["batch"] * case["kv_heads"]
    return units * per_unit, units * G * 4 * d * L * (n + (L + 1) / 2)


def work(case):
    path = case["path"]
    if path == "wavelet":
        e = 2 if case["dtype"] == "bf16" else 4
        h, t, d, lv = case["heads"], case["length"], case["head_dim"], case["levels"]
        return {"bytes": h * t * (d * e + 4) + h * lv * t * 4 + lv * t * 4, "flops": h * t * d * 4}
    e, d, G, c = 2 if case["dtype"] == "bf16" else 4, case["head_dim"], case["group"], case["budget"]
    units = case["batch"] * case["kv_heads"]
    if path == "decode":
        # rows; scores read and written; positions read; retained list; query and output; the new rows
        per_unit = 2 * (c + 1) * d * e + 8 * (c + 1) + 4 * (c + 1) + 4 * c + G * d * (e + 4) + 2 * d * e
        return {"bytes": case["layers"] * units * per_unit, "flops": case["layers"] * units * 4 * G * d * (c + 1)}
    if path == "chunk":
        b, f = _chunk_work(case, c, case["length"])
        return {"bytes": case["layers"] * b, "flops": case["layers"] * f}
    if path == "sequence":
        total = [_chunk_work(case, min(c, at), min(CHUNK, case["length"] - at)) for at in range(0, case["length"], CHUNK)]
        return {"bytes": sum(x[0] for x in total), "flops": sum(x[1] for x in total)}
    T, b = case["length"], case["block"]
    kept = min(T, c)
    # every key; the window's queries; token scores; the kept rows read (their keys have been) and written; the lists
    per_unit = T * d * e + b * G * d * e + T * 4 + 3 * kept * d * e + 8 * c + 4 * (T // b)
    return {"bytes": units * per_unit, "flops": units * 2 * G * b * d * (T - b / 2)}


def tolerance(case):
    """About four times what was measured: each path against itself in 64 bits, and, where a pass follows others on the
    same caches, against itself with the scores perturbed by more than rounding would (which turns a near-tie)."""
    path = case["path"]
    if path == "wavelet":                      # measured 4e-8 (rel) and 2e-7 (max): products and short sums in fp32
        return {"rel": 2e-7, "max": 8e-7}
    if case["dtype"] == "f32":                 # measured 2e-7 and 2e-6
        return {"rel": 1e-6, "max": 1e-5, "differ": 0.004}
    if path == "prompt":                       # token scores: measured 7e-7 and 8e-6; with turned, split keys 3e-6 and 4e-5
        return {"rel": 1e-5, "max": 2e-4, "differ": 0.004} if case["rerank"] else {"rel": 3e-6, "max": 3e-5, "differ": 0.004}
    # One pass: decode 7e-7, chunk 2e-6, turned and split chunk 7e-6 (rel).  Two of a scope's averaged scores that agree
    # to the last bits may be told apart either way, and in the calls that follow the cache then holds one other row of
    # one unit: measured 1e-4 (rel) and 0.08 (max) for a tie turned that way.
    return {"rel": 4e-4, "max": 0.3, "differ": 0.004}
