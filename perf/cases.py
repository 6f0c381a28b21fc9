"""The workloads this library's speed is judged on: hybrid-batch attention as a serving loop calls it.

A case is one batch shape: ``n_prefill`` chunks of ``q_lo..q_hi`` new tokens over ``past_lo..past_hi``
cached ones, ``n_decode`` single-token requests at contexts of ``ctx_lo..ctx_hi``, the head layout, the
16-bit type and the cache layout.  The lengths themselves are draws from ``lens_seed``, so that a case
fixes its shape and a seed fixes only the values.  One pass is one ``HybridAttention.forward`` call, which is one
layer of a model; the plan, its workspace and the output buffer are what a program keeps for the batch.
"""
import math
import random

import torch

from paper_2410_18038_amd import pod
from paper_2410_18038_amd import workloads as wl

DTYPES = {"fp16": wl.F16, "bf16": wl.BF16}


def _case(name, *, heads, dtype="bf16", block=16, head_major=False, n_prefill=0, q=(1, 1), past=(0, 0),
          n_decode=0, ctx=(1, 1), lens_seed=1):
    hq, hkv, d = heads
    return {"name": name, "hq": hq, "hkv": hkv, "d": d, "dtype": dtype, "block": block, "head_major": head_major,
            "n_prefill": n_prefill, "q_lo": q[0], "q_hi": q[1], "past_lo": past[0], "past_hi": past[1],
            "n_decode": n_decode, "ctx_lo": ctx[0], "ctx_hi": ctx[1], "lens_seed": lens_seed}


def listed():
    return [
        # The smallest call: a short chunk beside eight short conversations, four heads of 64 channels.
        # Launches and the length of one work item are what it costs.
        _case("tiny_hybrid", heads=(4, 4, 64), dtype="fp16", block=0, n_prefill=1, q=(128, 128), past=(384, 384),
              n_decode=8, ctx=(64, 512)),
        # One user's reply being generated: a single decode at a medium, odd context.
        _case("decode_single", heads=(32, 8, 128), n_decode=1, ctx=(6007, 6007)),
        # A lightly loaded server: eight conversations of very different lengths, one K/V head per query head.
        _case("decode_few", heads=(32, 32, 128), dtype="fp16", block=0, n_decode=8, ctx=(512, 4096)),
        # A loaded server between two prompts: nothing but decodes, all streaming.
        _case("decode_many", heads=(32, 8, 128), n_decode=128, ctx=(2048, 16384)),
        # Short prompts that arrive together, processed whole (no cached prefix, causal from key 0).
        _case("prompts_short", heads=(32, 8, 128), n_prefill=4, q=(100, 700)),
        # One long document processed in a single chunk: the causal triangle, work items of all lengths.
        _case("prompt_long", heads=(32, 8, 128), n_prefill=1, q=(8192, 8192)),
        # A chunk beside few decodes: both operations are short and neither hides the other.
        _case("hybrid_light", heads=(32, 8, 128), n_prefill=1, q=(512, 512), past=(3584, 3584),
              n_decode=16, ctx=(4096, 16384)),
        # A chunk beside 64 decodes, one K/V head per query head, contiguous fp16 cache: byte-bound.
        _case("hybrid_mha", heads=(32, 32, 128), dtype="fp16", block=0, n_prefill=1, q=(1024, 1024),
              past=(3072, 3072), n_decode=64, ctx=(4096, 4096)),
        # A chunk of a long document beside long decodes: bound by the matrix units.
        _case("hybrid_long", heads=(32, 4, 128), n_prefill=1, q=(2048, 2048), past=(30720, 30720),
              n_decode=32, ctx=(32768, 32768)),
        # 64 channels per head, three chunks of odd lengths, larger cache blocks in head-major order.
        _case("hybrid_d64", heads=(32, 8, 64), dtype="fp16", block=64, head_major=True, n_prefill=3, q=(150, 900),
              past=(0, 3000), n_decode=48, ctx=(300, 8000)),
        # 256 channels per head.
        _case("hybrid_d256", heads=(16, 8, 256), n_prefill=1, q=(1024, 1024), past=(3072, 3072),
              n_decode=64, ctx=(2048, 8192)),
        # Head counts that are no power of two (a tensor-parallel shard) and cache blocks of 24 tokens:
        # the general address path.
        _case("hybrid_odd", heads=(15, 5, 128), block=24, n_prefill=2, q=(200, 600), past=(100, 2500),
              n_decode=40, ctx=(500, 7000)),
    ]


# (query heads, K/V heads, channels)
_HEADS = [(32, 32, 128), (32, 8, 128), (32, 4, 128), (16, 8, 128), (10, 5, 128), (9, 3, 128), (8, 1, 128),
          (32, 8, 64), (16, 1, 64), (9, 3, 64), (4, 4, 64), (16, 8, 256), (8, 2, 256)]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case: decode only, prompts only, or a hybrid batch, any size up to the largest listed one."""
    limit = _cost(next(c for c in listed() if c["name"] == "hybrid_long"))
    while True:
        kind = rng.choice(["decode", "prefill", "hybrid", "hybrid"])
        n_prefill = n_decode = 0
        q = past = (0, 0)
        ctx = (1, 1)
        if kind != "decode":
            n_prefill = rng.choice([1, 1, 2, 3, 6])
            q_hi = _log_int(rng, 17, 8192 // n_prefill)
            q = (max(1, q_hi // rng.choice([1, 2, 5])), q_hi)
            past_hi = rng.choice([0, _log_int(rng, 64, 30720)])
            past = (past_hi // rng.choice([1, 3]), past_hi)
        if kind != "prefill":
            n_decode = _log_int(rng, 1, 160)
            ctx_hi = _log_int(rng, 64, 32768)
            ctx = (max(1, ctx_hi // rng.choice([1, 4, 8])), ctx_hi)
        case = _case("", heads=rng.choice(_HEADS), dtype=rng.choice(["fp16", "bf16"]),
                     block=rng.choice([0, 16, 16, 16, 64, 24]), head_major=rng.random() < 0.2, n_prefill=n_prefill,
                     q=q, past=past, n_decode=n_decode, ctx=ctx, lens_seed=rng.randrange(1, 1 << 30))
        if _cost(case) <= limit:
            del case["name"]
            return case


def _lengths(case):
    """((new tokens, visible tokens) per chunk, context per decode)."""
    rng = random.Random(case["lens_seed"])
    prefill = []
    for _ in range(case["n_prefill"]):
        q = rng.randint(case["q_lo"], case["q_hi"])
        prefill.append((q, q + rng.randint(case["past_lo"], case["past_hi"])))
    return prefill, [rng.randint(case["ctx_lo"], case["ctx_hi"]) for _ in range(case["n_decode"])]


def prepare(case, seed):
    prefill, decode = _lengths(case)
    batch = wl.make_batch("case", prefill=prefill, decode_kv_lens=decode, n_q_heads=case["hq"], n_kv_heads=case["hkv"],
                          head_dim=case["d"], dtype=DTYPES[case["dtype"]], seed=seed, block_size=case["block"],
                          device="cuda:0")
    if case["head_major"]:
        batch = wl.to_head_major(batch)
    out = torch.empty((batch.n_rows, batch.n_q_heads, batch.head_dim), dtype=batch.torch_dtype, device="cuda:0")
    return {"batch": batch, "attn": pod.HybridAttention(batch), "out": out}


def run(state):
    return state["attn"].forward(state["batch"], out=state["out"])


def work(case):
    """Q and the visible K/V read once, the output written once; 4*d operations per visible (row, key) pair."""
    prefill, decode = _lengths(case)
    pairs = sum(q * (kv - q) + q * (q + 1) // 2 for q, kv in prefill) + sum(decode)
    rows = sum(q for q, _ in prefill) + len(decode)
    tokens = sum(kv for _, kv in prefill) + sum(decode)
    row_bytes = 2 * case["d"]
    return {"bytes": row_bytes * (2 * rows * case["hq"] + 2 * tokens * case["hkv"]),
            "flops": 4 * case["d"] * case["hq"] * pairs}


def _cost(case):
    w = work(case)
    return w["bytes"] / 6e12 + w["flops"] / 8e14


def tolerance(case):
    # Two 16-bit roundings count, of the softmax weights before the second product and of the result.  Against
    # fp64 and against other cuts of the key range the results differ by up to 2.5e-3 and 2.1e-2 (bf16), 3.6e-4 and
    # 2.2e-3 (fp16); these are four times that.
    return {"rel": 1e-2, "max": 8e-2} if case["dtype"] == "bf16" else {"rel": 1.5e-3, "max": 1e-2}
