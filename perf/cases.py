"""The workloads that performance is measured on: what a serving program has this library do.

A case is one pass of one attention path through the public entry points, over `layers` layers that
each keep a KV pool of their own, as in a model.  The sizes are those of the repository's named
workloads (``workloads/__init__.py``: 40 query heads of 128 dims over 8 or 40 KV heads, 64 dims in the
small one) and generic ones between and beyond them.  K, V and q are N(0, 1) rounded to fp16; in the
long-context cases 1 % of the key rows are 20 times that.  Context and chunk lengths are spread
evenly over the case's range and dealt to the sequences by the seed; physical blocks are a random
permutation of the pool.

Operations (`op`):
  step         one fused decode step per layer (write of the new token + attention), its schedule
               derived in every launch: paged_gqa_decode_step
  scheduled    the same with the schedule prepared once for the layers: decode_schedule_prepare,
               then paged_gqa_decode_scheduled per layer
  write_decode the write and the attention as separate calls: kv_cache_write_*, paged_gqa_decode
  partitioned  kv_cache_write_*, paged_gqa_decode_partitioned (512 tokens each), paged_gqa_reduce
  prefill      kv_cache_write_* of a chunk per sequence, then paged_gqa_prefill_chunk_ws
  fill         kv_cache_write_* of whole contexts alone (importing a prompt's K and V)
  gather       gather_cached_kv of every sequence's context (handing a cache on)
"""
import math

import torch

import paper_2602_09323_amd as coopt

BLOCK = 16
PARTITION = 512
_DTYPE = {"e4m3": coopt.COOPT_KV_E4M3, "e5m2": coopt.COOPT_KV_E5M2, "fp16": coopt.COOPT_KV_FP16}


def _case(name, op, cache, seqs, q_heads, kv_heads, dim, ctx_lo, ctx_hi, chunk_lo=0, chunk_hi=0, layers=1,
          outliers=False):
    """ctx_*: tokens in the cache when the pass attends (decode: the new token included; prefill: the
    history before the chunk); chunk_*: new rows per sequence (prefill only)."""
    return {"name": name, "op": op, "cache": cache, "seqs": seqs, "q_heads": q_heads,
            "kv_heads": kv_heads, "dim": dim, "ctx_lo": ctx_lo, "ctx_hi": ctx_hi, "chunk_lo": chunk_lo,
            "chunk_hi": chunk_hi, "layers": layers, "outliers": outliers}


def listed():
    return [
        # the smallest call: one short sequence of a small model, where latency and launches count
        _case("tiny_step", "step", "e4m3", 1, 4, 2, 64, 256, 256),
        # one user chatting with a 13B model: one sequence, an odd length, four layers
        _case("single_user_step", "step", "e4m3", 1, 40, 8, 128, 1789, 1789, layers=4),
        # the headline decode batch: 32 sequences of 512 to 2048 tokens, eight layers of one step
        _case("batch32_gqa_fp8", "scheduled", "e4m3", 32, 40, 8, 128, 512, 2048, layers=8),
        # the same batch with an uncompressed cache and one KV head per query head
        _case("batch32_mha_fp16", "write_decode", "fp16", 32, 40, 40, 128, 512, 2048),
        # many short and ragged sequences of a 64-dim model with the other one-byte code
        _case("ragged96_d64_e5m2", "scheduled", "e5m2", 96, 32, 8, 64, 1, 4001, layers=2),
        # long contexts with outlier keys, fused and balanced
        _case("long_context_step", "step", "e4m3", 4, 40, 8, 128, 16384, 32768, layers=2, outliers=True),
        # long contexts through fixed partitions and a reduce
        _case("long_context_partitioned", "partitioned", "e4m3", 4, 40, 8, 128, 16384, 32768, layers=2,
              outliers=True),
        # chunked prefill: 512 new rows behind 8192 tokens of history, 8 sequences
        _case("chunked_prefill", "prefill", "e4m3", 8, 40, 8, 128, 8192, 8192, 512, 512),
        # fresh prompts of ragged lengths: no history, the causal triangle is all there is
        _case("fresh_prompts", "prefill", "e4m3", 3, 40, 8, 128, 0, 0, 301, 1777),
        # one prompt's next chunk over an uncompressed cache, one KV head per query head
        _case("mha_fp16_prefill", "prefill", "fp16", 1, 40, 40, 128, 4096, 4096, 333, 333),
        # a cache fill of 65 536 tokens in ragged sequences
        _case("cache_fill", "fill", "e4m3", 32, 40, 8, 128, 1024, 3072),
        # dequantising gather of long contexts
        _case("gather_long", "gather", "e4m3", 4, 40, 8, 128, 16384, 32768),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case of the same ranges.  Its bytes and operations stay below the largest listed."""
    while True:
        op = rng.choice(["step", "scheduled", "write_decode", "partitioned", "prefill", "prefill", "fill",
                         "gather"])
        cache = rng.choice(["e4m3", "e4m3", "e4m3", "e5m2", "fp16"])
        q_heads, kv_heads, dim = rng.choice([(40, 8, 128), (40, 8, 128), (40, 40, 128), (32, 8, 64), (4, 2, 64)])
        seqs = _log_int(rng, 1, 96)
        ctx_hi = _log_int(rng, 16, 32768)
        ctx_lo = max(1, int(ctx_hi * rng.uniform(0.02, 1.0)))
        chunk_lo = chunk_hi = 0
        layers = _log_int(rng, 1, 8)
        if op == "prefill":
            chunk_hi = _log_int(rng, 16, 2048)
            chunk_lo = max(1, int(chunk_hi * rng.uniform(0.1, 1.0)))
            if rng.random() < 0.3:
                ctx_lo = ctx_hi = 0
        if op in ("prefill", "fill", "gather"):
            layers = 1
        if op == "partitioned":
            ctx_hi, ctx_lo = max(ctx_hi, 2048), max(ctx_lo, 1024)
        if op == "gather":
            seqs = min(seqs, 8)
        case = _case("", op, cache, seqs, q_heads, kv_heads, dim, ctx_lo, ctx_hi, chunk_lo, chunk_hi, layers,
                     outliers=ctx_hi > 8192)
        del case["name"]
        w = work(case)
        if w["bytes"] <= 0.6e9 and w["flops"] <= 2.5e11:
            return case


def _spread(lo, hi, n):
    return [lo + ((hi - lo) * i) // (n - 1) if n > 1 else (lo + hi) // 2 for i in range(n)]


def _lengths(case):
    """Per sequence (before the seed deals them out): tokens visible at the end, new rows.  The
    longest chunks sit on the shortest histories."""
    n = case["seqs"]
    ctx = _spread(case["ctx_lo"], case["ctx_hi"], n)
    if case["op"] == "prefill":
        new = _spread(case["chunk_lo"], case["chunk_hi"], n)[::-1]
        return [c + r for c, r in zip(ctx, new)], new
    if case["op"] == "fill":
        return ctx, ctx
    if case["op"] == "gather":
        return ctx, [0] * n
    return ctx, [1] * n


def work(case):
    total, new = _lengths(case)
    hq, hk, d = case["q_heads"], case["kv_heads"], case["dim"]
    per_token = hk * (4 * d if case["cache"] == "fp16" else 2 * d + 8)      # one token's K and V in the cache
    rows = sum(new)
    write = rows * (hk * 4 * d + per_token + 8)                             # fp16 rows and slots in, cache out
    if case["op"] == "fill":
        return {"bytes": write, "flops": 0}
    tables = sum((t + BLOCK - 1) // BLOCK for t in total) * 4 + 4 * len(total)
    if case["op"] == "gather":
        return {"bytes": sum(total) * (per_token + hk * 4 * d) + tables, "flops": 0}
    attn = sum(total) * per_token + 2 * rows * hq * d * 2 + tables
    pairs = sum(r * (t - r) + r * (r + 1) // 2 for t, r in zip(total, new))
    layers = case["layers"]
    return {"bytes": layers * (attn + write), "flops": layers * 4 * d * hq * pairs}


def tolerance(case):
    """Cache bytes, scales and gathered rows: the same bits (codes and gathered rows are rounded once
    from exact values).  Attention rows are fp16.  Against attention in 64 bits over the same cache the
    listed decode cases differ by at most 2.1e-4 of the norm and 4.9e-4 of a value (that is fp16's own
    rounding), the prefill cases, whose weights enter the second product as fp16, by 3.1e-4 and
    7.3e-3 (the first rows of a fresh prompt): four times that is stated."""
    if case["op"] in ("fill", "gather"):
        return "exact"
    if case["op"] == "prefill":
        return {"rel": 1.2e-3, "max": 3e-2}
    return {"rel": 8e-4, "max": 2e-3}


def prepare(case, seed):
    dev = torch.device("cuda")
    gen = torch.Generator(device=dev)
    gen.manual_seed(seed)
    host = torch.Generator()
    host.manual_seed(seed)
    n, hq, hk, d, layers = case["seqs"], case["q_heads"], case["kv_heads"], case["dim"], case["layers"]
    # (a gather's rows come out one tensor per sequence: there the lengths keep their order)
    order = list(range(n)) if case["op"] == "gather" else torch.randperm(n, generator=host).tolist()
    total, new = _lengths(case)
    total, new = [total[i] for i in order], [new[i] for i in order]
    blocks = [(t + BLOCK - 1) // BLOCK for t in total]
    pool = sum(blocks) + sum(blocks) // 8 + 8
    width = max(blocks)
    perm = torch.randperm(pool, generator=host).to(torch.int32)
    table = torch.full((n, width), -1, dtype=torch.int32)
    at = 0
    for s, b in enumerate(blocks):
        table[s, :b] = perm[at:at + b]
        at += b

    def slots_of(first, last):             # of tokens first[s] .. last[s]-1 of every sequence
        parts = []
        for s in range(n):
            j = torch.arange(first[s], last[s], dtype=torch.int64)
            parts.append(table[s].to(torch.int64)[j // BLOCK] * BLOCK + j % BLOCK)
        return torch.cat(parts).to(dev)

    def normal(*size):
        return torch.randn(*size, generator=gen, device=dev, dtype=torch.float32).to(torch.float16)

    kv = _DTYPE[case["cache"]]
    scaled = kv != coopt.COOPT_KV_FP16
    shape = coopt.Shape(n, hq, hk, d, BLOCK, pool, width, kv, 1.0 / math.sqrt(d))
    st = {"case": case, "shape": shape, "table": table.to(dev),
          "lens": torch.tensor(total, dtype=torch.int32, device=dev), "layers": []}
    old = [t - r for t, r in zip(total, new)]
    history, fresh = slots_of([0] * n, old), slots_of(old, total)
    st["slots"] = fresh
    rows = sum(new)
    code = 1 if scaled else 2
    for _ in range(layers):
        layer = {"cache": [torch.zeros(pool, hk, BLOCK * d * code, dtype=torch.uint8, device=dev) for _ in range(2)]}
        layer["scale"] = [torch.zeros(pool, hk, BLOCK, device=dev) for _ in range(2)] if scaled else [None, None]
        if len(history):
            k, v = normal(len(history), hk, d), normal(len(history), hk, d)
            if case["outliers"]:
                hit = torch.rand(len(history), generator=gen, device=dev) < 0.01
                k[hit] *= 20.0
            _write(k, v, history, layer, shape)
        layer["k"], layer["v"] = normal(rows, hk, d), normal(rows, hk, d)
        if case["op"] not in ("fill", "gather"):
            layer["q"] = normal(rows, hq, d)
            layer["out"] = torch.empty(rows, hq, d, dtype=torch.float16, device=dev)
        st["layers"].append(layer)

    def buffer(nbytes):
        return torch.empty(max(nbytes, 16), dtype=torch.uint8, device=dev)

    if case["op"] in ("step", "scheduled", "write_decode"):
        st["workspace"] = buffer(coopt.decode_workspace_bytes(shape))
    if case["op"] == "scheduled":
        st["schedule"] = buffer(coopt.decode_schedule_bytes(shape))
    if case["op"] == "partitioned":
        parts = (width * BLOCK + PARTITION - 1) // PARTITION
        st["parts"] = parts
        st["tmp"] = torch.empty(n, hq, parts, d, device=dev)
        st["max"] = torch.empty(n, hq, parts, device=dev)
        st["sum"] = torch.empty(n, hq, parts, device=dev)
    if case["op"] == "prefill":
        starts = [0]
        for r in new:
            starts.append(starts[-1] + r)
        st["starts"] = torch.tensor(starts, dtype=torch.int32, device=dev)
        st["rows"], st["longest"] = rows, max(new)
        need = coopt.prefill_workspace_bytes(shape, st["longest"])
        st["workspace"] = buffer(need) if need else None
    if case["op"] == "gather":
        st["total"] = total
        st["gathered"] = [[torch.empty(t, hk, d, dtype=torch.float16, device=dev) for _ in range(2)] for t in total]
    return st


def _write(k, v, slots, layer, shape):
    if shape.kv_dtype == coopt.COOPT_KV_FP16:
        coopt.kv_cache_write_fp16(k, v, slots, *layer["cache"], shape)
    else:
        coopt.kv_cache_write_fp8(k, v, slots, *layer["cache"], *layer["scale"], shape)


def run(st):
    op, shape, table, lens, slots = st["case"]["op"], st["shape"], st["table"], st["lens"], st["slots"]
    results = []
    if op == "scheduled":
        coopt.decode_schedule_prepare(table, lens, slots, st["schedule"], shape)
    for layer in st["layers"]:
        cache, scale, k, v = layer["cache"], layer["scale"], layer["k"], layer["v"]
        if op == "gather":
            for s, (ko, vo) in enumerate(st["gathered"]):
                coopt.gather_cached_kv(*cache, *scale, table, s, 0, st["total"][s], ko, vo, shape)
                results += [ko, vo]
            continue
        if op == "fill":
            _write(k, v, slots, layer, shape)
            results += [*cache, *[x for x in scale if x is not None]]
            continue
        q, out = layer["q"], layer["out"]
        if op == "step":
            coopt.paged_gqa_decode_step(k, v, slots, q, *cache, *scale, table, lens, out, st["workspace"], shape)
        elif op == "scheduled":
            coopt.paged_gqa_decode_scheduled(k, v, slots, q, *cache, *scale, lens, out, st["workspace"],
                                             st["schedule"], shape)
        else:
            _write(k, v, slots, layer, shape)
            if op == "write_decode":
                coopt.paged_gqa_decode(q, *cache, *scale, table, lens, out, st["workspace"], shape)
            elif op == "partitioned":
                coopt.paged_gqa_decode_partitioned(q, *cache, *scale, table, lens, PARTITION, st["tmp"], st["max"],
                                                   st["sum"], st["parts"], shape)
                coopt.paged_gqa_reduce(st["tmp"], st["max"], st["sum"], lens, PARTITION, st["parts"], out, shape)
            else:
                coopt.paged_gqa_prefill_chunk_ws(q, *cache, *scale, table, lens, st["starts"], st["rows"],
                                                 st["longest"], out, st["workspace"], shape)
        results += [out, *cache, *[x for x in scale if x is not None]]
    return results
