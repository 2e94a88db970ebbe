"""The attention work of a serving engine on one GPU's head shard, as measurable cases.

Every case is one engine step on a paged KV cache: `prepare` makes the cache with its cached prefixes, the block table,
the step's new tokens and a workspace; `run` passes the step through the library's public calls.  The lengths of a case
follow from the case alone, so its work is known beforehand; the values and the page placement follow from the seed."""
import math
import random

import numpy as np
import torch

import paper_2507_11830_amd as sp

PAGE = 16

# Head shards: (query heads, KV heads, head_dim).
TINY = (2, 1, 64)  # smallest GQA group
SHARD70 = (8, 1, 128)  # a 70B model over eight GPUs
FULL8B = (32, 8, 128)  # an 8B model on one GPU
WIDE64 = (16, 2, 64)  # head_dim 64
SHARDS = (SHARD70, SHARD70, FULL8B, FULL8B, WIDE64, TINY, (16, 2, 128), (32, 4, 128), (12, 3, 64))

MAX_BYTES = 4.7e9  # no drawn case goes beyond the largest listed ones
MAX_FLOPS = 2.19e12


def case(kind, heads, call, **shape):
    hq, hkv, d = heads
    return dict(kind=kind, hq=hq, hkv=hkv, d=d, call=call, **shape)


def listed():
    return [
        # One user, a short chat on a small shard: nothing but latency and launches.
        dict(case("decode", TINY, "step", batch=1, lo=137, hi=137, lengths=1), name="decode-1-short"),
        # The ordinary decode step of continuous batching on a 70B shard: 64 users, mixed contexts.
        dict(case("decode", SHARD70, "step", batch=64, lo=512, hi=8192, lengths=3), name="decode-64"),
        # A big batch of long contexts on an 8B model, several GB of KV: the largest decode (the rows are appended by an
        # earlier call of the same step).
        dict(case("decode", FULL8B, "attend", batch=128, lo=1024, hi=16384, lengths=6), name="decode-8b-128"),
        # One user deep in a long document, after a long prefill on the same cache.
        dict(case("decode", SHARD70, "step", batch=1, lo=32900, hi=32900, lengths=5), name="decode-1-long"),
        # Verification of speculated tokens: 4 query tokens per user.
        dict(case("verify", SHARD70, "step", batch=64, lo=512, hi=8192, chunk=4, lengths=7), name="verify-64x4"),
        # A short prompt alone.
        dict(case("prefill", TINY, "step", batch=1, lo=128, hi=128, lengths=1), name="prefill-1x128"),
        # A few ordinary prompts at once.
        dict(case("prefill", SHARD70, "step", batch=4, lo=2048, hi=2048, lengths=2), name="prefill-4x2048"),
        # A long document in one prefill, appended and attended by separate calls.
        dict(case("prefill", SHARD70, "two", batch=1, lo=32768, hi=32768, lengths=5), name="prefill-1x32768"),
        # Prompts of an 8B model, all its heads on one GPU.
        dict(case("prefill", FULL8B, "step", batch=4, lo=8192, hi=8192, lengths=8), name="prefill-8b-4x8192"),
        # head_dim 64 over the same range.
        dict(case("prefill", WIDE64, "step", batch=2, lo=9001, hi=16384, lengths=9), name="prefill-d64-2x16k"),
        # Chunked prefill of a batch with half of every prompt cached.
        dict(case("chunked", SHARD70, "step", batch=32, median=1500, chunk=512, lengths=4), name="chunked-32x512"),
        # One step that mixes decoding users with a new user's prompt chunk.
        dict(case("mixed", SHARD70, "step", batch=64, lo=512, hi=8192, chunk=2048, lengths=10), name="mixed-63+2048"),
    ]


def log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw_any(rng):
    kind = rng.choice(("decode", "decode", "decode", "verify", "prefill", "prefill", "prefill", "chunked", "mixed"))
    heads = rng.choice(SHARDS)
    seed = rng.randrange(1 << 30)
    if kind == "decode":
        hi = log_int(rng, 130, 33000)
        lo = max(64, int(hi * rng.uniform(0.06, 1.0)))
        return case(kind, heads, rng.choice(("step", "step", "attend", "two")), batch=log_int(rng, 1, 128), lo=min(lo, hi), hi=hi, lengths=seed)
    if kind == "verify":
        hi = log_int(rng, 200, 16384)
        return case(kind, heads, rng.choice(("step", "attend")), batch=log_int(rng, 1, 64), lo=max(32, hi // 16), hi=hi, chunk=rng.randint(2, 8), lengths=seed)
    if kind == "prefill":
        hi = log_int(rng, 100, 32768)
        lo = int(hi * rng.uniform(0.3, 1.0))
        return case(kind, heads, rng.choice(("step", "two", "attend")), batch=log_int(rng, 1, 8), lo=max(1, lo), hi=hi, lengths=seed)
    if kind == "chunked":
        return case(kind, heads, rng.choice(("step", "two")), batch=log_int(rng, 2, 48), median=log_int(rng, 400, 6000), chunk=log_int(rng, 128, 2048), lengths=seed)
    hi = log_int(rng, 500, 12000)
    return case(kind, heads, rng.choice(("step", "attend")), batch=log_int(rng, 8, 96), lo=max(32, hi // 16), hi=hi, chunk=log_int(rng, 100, 4096), lengths=seed)


def draw(rng):
    while True:
        c = draw_any(rng)
        w = work(c)
        if w["bytes"] <= MAX_BYTES and w["flops"] <= MAX_FLOPS:
            return c


def lengths(c):
    """(cached tokens, new tokens) of every sequence."""
    rng = random.Random(c["lengths"])
    n = c["batch"]
    if c["kind"] == "decode":
        total = [rng.randint(c["lo"], c["hi"]) for _ in range(n)]
        return [t - 1 for t in total], [1] * n
    if c["kind"] == "verify":
        total = [max(rng.randint(c["lo"], c["hi"]), c["chunk"]) for _ in range(n)]
        return [t - c["chunk"] for t in total], [c["chunk"]] * n
    if c["kind"] == "prefill":
        return [0] * n, [rng.randint(c["lo"], c["hi"]) for _ in range(n)]
    if c["kind"] == "chunked":
        total = [min(max(round(rng.lognormvariate(math.log(c["median"]), 1.0)), 64), 16384) for _ in range(n)]
        cached = [t // 2 for t in total]
        return cached, [min(c["chunk"], t - p) for t, p in zip(total, cached)]
    total = [rng.randint(c["lo"], c["hi"]) for _ in range(n - 1)]  # mixed: the new prompt's place in the batch is any
    cached, new, at = [t - 1 for t in total], [1] * (n - 1), rng.randrange(n)
    cached.insert(at, 0)
    new.insert(at, c["chunk"])
    return cached, new


def device_ints(values):
    return torch.tensor(values, dtype=torch.int32).cuda()


def prepare(c, seed):
    hq, hkv, d = c["hq"], c["hkv"], c["d"]
    cached, new = lengths(c)
    total = [a + b for a, b in zip(cached, new)]
    gen = torch.Generator(device="cuda").manual_seed(seed)

    def normal(*shape):
        out = torch.empty(shape, dtype=torch.bfloat16, device="cuda")
        flat, step = out.view(-1), 1 << 28
        for a in range(0, flat.numel(), step):
            part = flat[a:a + step]
            part.copy_(torch.randn(part.numel(), generator=gen, device="cuda"))
        return out

    # a pool a quarter larger than needed, its pages dealt out in shuffled order
    pages = [-(-t // PAGE) for t in total]
    num_pages = max(1, math.ceil(1.25 * sum(pages)))
    order = np.random.default_rng(seed).permutation(num_pages).astype(np.int32)
    table = np.full((len(total), max(pages)), -1, np.int32)
    at = 0
    for s, n in enumerate(pages):
        table[s, :n] = order[at:at + n]
        at += n
    tokens = sum(new)
    s = dict(
        call=c["call"], decode=c["kind"] == "decode", scale=1.0 / math.sqrt(d),
        cache=sp.KVCache(normal(num_pages, hkv, PAGE, d), normal(num_pages, hkv, PAGE, d)),
        table=torch.from_numpy(table).cuda(), cu=device_ints(np.concatenate([[0], np.cumsum(new)])),
        ctx=device_ints(cached), total=device_ints(total), max_new=max(new), max_total=max(total),
        q=normal(tokens, hq, d), k=normal(tokens, hkv, d), v=normal(tokens, hkv, d))
    s["out"] = torch.empty_like(s["q"])
    if s["decode"]:
        size = sp.sp_attn_decode_workspace_size(len(total), s["max_total"], hq, d)
    else:
        size = sp.sp_attn_prefill_workspace_size(len(total), tokens, s["max_new"], s["max_total"], hq, hkv, d)
    s["workspace"] = torch.empty(size, dtype=torch.uint8, device="cuda") if size else None
    s["result"] = [s["out"]]
    if c["call"] == "attend":  # the new rows are in the cache already
        sp.sp_kv_append(s["cache"], s["k"], s["v"], s["cu"], s["ctx"], s["table"])
    else:  # the updated cache is a result too, bit for bit
        s["result"] += [s["cache"].k_pages.view(torch.int16), s["cache"].v_pages.view(torch.int16)]
    return s


def run(s):
    cache, table, out = s["cache"], s["table"], s["out"]
    if s["call"] == "two":
        sp.sp_kv_append(cache, s["k"], s["v"], s["cu"], s["ctx"], table)
    if s["decode"]:
        if s["call"] == "step":
            sp.sp_decode_step(cache, s["k"], s["v"], s["q"], out, s["total"], table, s["max_total"], s["scale"], s["workspace"])
        else:
            sp.sp_attn_decode(cache, s["q"], out, s["total"], table, s["max_total"], s["scale"], s["workspace"])
    elif s["call"] == "step":
        sp.sp_chunk_step(cache, s["k"], s["v"], s["q"], out, s["cu"], s["ctx"], table, s["max_new"], s["max_total"], s["scale"], workspace=s["workspace"])
    else:
        sp.sp_attn_prefill(cache, s["q"], out, s["cu"], s["ctx"], table, s["max_new"], s["max_total"], s["scale"], workspace=s["workspace"])
    return s["result"]


def work(c):
    """Queries and new rows read, outputs and new rows written, cached keys and values and their page ids read, each
    once; 4 * head_dim operations per visible (query, key) pair and head."""
    hq, hkv, d = c["hq"], c["hkv"], c["d"]
    cached, new = lengths(c)
    tokens = sum(new)
    total = [a + b for a, b in zip(cached, new)]
    rows = sum(cached) if c["call"] != "attend" else sum(total)  # K/V rows read from the cache
    fresh = 2 * tokens if c["call"] != "attend" else 0  # read from the step's inputs, and written to the cache
    size = 2 * d * (2 * hq * tokens + 2 * hkv * (rows + fresh)) + 4 * sum(-(-t // PAGE) for t in total)
    pairs = sum(n * p + n * (n + 1) // 2 for p, n in zip(cached, new))
    return {"bytes": size, "flops": 4 * d * hq * pairs}


def tolerance(c):
    """bf16 products with fp32 sums; the weights and the result are rounded to bf16.  Against the same sums in 64 bits
    the results are off by rel 0.0024 and max 0.022 at most over the listed cases; cache rows are the same bits."""
    return {"rel": 0.01, "max": 0.08}
