"""Cases that time the library the way a serving program uses it.

A case is one pass through the public entry points of ``paper_2508_15212_amd``: pruning a key cache at prefill,
one decode step over a packed cache, or both.  Shapes are the five benchmark configurations of ``workloads`` (or
cut-down ones of the same form), ragged batches and odd lengths.

    op         what a pass does
    --------   -------------------------------------------------------------------------------------------------
    step       prune, then one decode step (a short prompt and its first token)
    prune      spark_prune over the whole prompt(s)
    prune_kv   spark_prune on the keys and spark_prune_values on the values
    prune_topp spark_prune_topp
    decode     spark_decode_attn                      tail       spark_decode_attn_tail (rows appended since prefill)
    values     spark_decode_attn_values               sampled    spark_decode_attn_sampled, Gaussian recovery
    topp       spark_decode_attn_topp

    batch, lo, hi, lens   sequences and the range of their lengths; the lengths are drawn evenly from it by a generator
                          keyed with `lens`, so that they belong to the case and not to the inputs' seed
    group, hkv            query heads per KV head, KV heads
    keep, keep_v, p       kept key channels, kept value channels, basis points of the top-p rule
    pack                  "bf16" or "int8" storage of the kept key entries
    window                observation-window queries per head
    layout                "HND": rows of a head are contiguous; "NHD": all heads of a token are
    out                   output type of decode, "bf16" or "f32"
    cap                   capacity of the appended-row buffers, which hold a random number of rows per sequence
    sigma, outliers       log-normal row jitter of the keys, outlier channels per head (scaled by 8)
"""
import math
import random

import torch

import paper_2508_15212_amd as spark

D = 128

BASE = {"hkv": 8, "group": 4, "keep": 26, "keep_v": 0, "p": 0, "pack": "bf16", "window": 32, "layout": "HND", "out": "bf16",
        "cap": 0, "sigma": 0.5, "outliers": 8, "lens": 1}


def _case(name, op, batch, lo, hi, **over):
    return {"name": name, "op": op, "batch": batch, "lo": lo, "hi": hi, **BASE, **over}


def listed():
    return [
        # one short prompt: prune and first decode step, a few microseconds of work and three launches
        _case("step_1k", "step", 1, 1024, 1024, keep=64, outliers=4, sigma=0.0, out="f32"),
        # a handful of conversations in the middle of generation: short ragged prefixes, rows appended since prefill, a
        # keep count that has no kernel of its own
        _case("decode_chat_tail", "tail", 4, 700, 3900, keep=32, cap=256, layout="NHD", lens=5),
        # the headline workload: Llama-3.1-8B heads, eight sequences of 32K tokens, 80 % of the key channels pruned
        _case("decode_llama_32k", "decode", 8, 32768, 32768),
        # serving: 64 sequences of an eviction-compressed cache, half of the channels kept
        _case("decode_ragged_64", "decode", 64, 512, 2048, keep=64, layout="NHD", outliers=4, sigma=0.0, lens=4, out="f32"),
        # Qwen3-32B heads at 128K tokens, kept entries as int8 codes: the largest cache
        _case("decode_qwen_128k_int8", "decode", 4, 131072, 131072, group=8, pack="int8", out="f32"),
        # keys and values both pruned (the memory-saving combination), medium contexts of odd length
        _case("decode_values_16k", "values", 4, 12001, 18777, keep_v=64, lens=7),
        # the sampled recovery function of the ablation, which draws a variate per pruned entry
        _case("decode_gaussian_16k", "sampled", 2, 16001, 16001, out="f32"),
        # the adaptive variant: every row keeps as many channels as hold 99 % of its saliency
        _case("decode_topp_32k", "topp", 2, 32768, 32768, p=9900),
        # prefill of one long document, 64 window queries
        _case("prune_128k", "prune", 1, 131072, 131072, window=64),
        # prefill of a ragged batch in the layout that a model's projections leave the keys in
        _case("prune_ragged_64", "prune", 64, 512, 2048, keep=64, layout="NHD", outliers=4, sigma=0.0, lens=4),
        # prefill where both caches are packed, int8 keys, odd length
        _case("prune_kv_40k_int8", "prune_kv", 1, 40003, 40003, group=8, pack="int8", keep_v=38, layout="NHD"),
        # prefill of the adaptive variant
        _case("prune_topp_64k", "prune_topp", 1, 65536, 65536, p=9900),
    ]


def draw(rng):
    """One more case: any operation, sizes spread over the logarithm of the listed cases' range."""
    op = rng.choice(["step", "prune", "prune", "prune_kv", "prune_topp", "decode", "decode", "decode", "tail", "values", "sampled", "topp"])
    # tokens of the whole batch: up to the largest listed case of the operation
    most = {"step": 16384, "prune": 131072, "prune_kv": 40000, "prune_topp": 65536, "decode": 196608, "tail": 65536, "values": 65536,
            "sampled": 32768, "topp": 65536}[op]
    total = int(math.exp(rng.uniform(math.log(256), math.log(most))))
    batch = min(rng.choice([1, 1, 2, 3, 5, 8, 16, 33, 64, 100]), max(1, total // 64))
    mean = max(1, total // batch)
    ragged = batch > 1 and rng.random() < 0.6
    lo, hi = (max(1, mean * 2 // 5), mean * 8 // 5) if ragged else (mean, mean)
    pack = "int8" if op in ("decode", "prune", "prune_kv", "values", "sampled", "tail") and rng.random() < 0.3 else "bf16"
    return {"op": op, "batch": batch, "lo": lo, "hi": hi, **BASE, "lens": rng.randrange(1 << 16),
            "group": rng.choice([1, 2, 4, 4, 4, 8, 8, 16]), "hkv": rng.choice([1, 2, 4, 8, 8, 8]), "pack": pack,
            "keep": rng.choice([25, 26, 26, 38, 64, rng.randint(24, 96)]),
            "keep_v": rng.choice([26, 38, 64, rng.randint(24, 96)]) if op in ("values", "prune_kv") else 0,
            "p": rng.choice([9900, 9900, 9500]) if op in ("prune_topp", "topp") else 0,
            "window": rng.choice([16, 32, 32, 64]), "layout": rng.choice(["HND", "NHD"]), "out": rng.choice(["bf16", "f32"]),
            "cap": rng.choice([64, 256, 700]) if op == "tail" else 0, "sigma": rng.choice([0.0, 0.5]), "outliers": rng.choice([4, 8])}


# ---------------------------------------------------------------- inputs


def _lens(case):
    r = random.Random(case["lens"])
    return [r.randint(case["lo"], case["hi"]) for _ in range(case["batch"])]


def _tail_lens(case):
    r = random.Random(case["lens"] + 1)
    return [r.randint(0, case["cap"]) for _ in range(case["batch"])]


def _inputs(case, seed):
    """What the model hands over: keys, values, window queries, the step's query, appended rows.  bf16, on the GPU."""
    gen = torch.Generator(device="cuda").manual_seed(seed)
    dev = {"device": "cuda", "generator": gen}
    lens = _lens(case)
    total, hkv, batch, hq = sum(lens), case["hkv"], case["batch"], case["hkv"] * case["group"]
    shape = (hkv, total, D) if case["layout"] == "HND" else (total, hkv, D)
    k = torch.empty(shape, dtype=torch.bfloat16, device="cuda")
    v = torch.empty(shape, dtype=torch.bfloat16, device="cuda")
    for h in range(hkv):
        scale = torch.ones(D, device="cuda")
        scale[torch.randperm(D, **dev)[:case["outliers"]]] = 8.0
        x = torch.randn(total, D, **dev) * scale
        if case["p"]:
            # the adaptive rule meets caches whose magnitude sits in a minority of the channels
            quiet = torch.rand(D, **dev) < 0.6
            x *= torch.where(quiet, 0.008 * torch.exp(0.5 * torch.randn(D, **dev)), torch.ones(D, device="cuda"))
        if case["sigma"] > 0.0:
            x *= torch.exp(case["sigma"] * torch.randn(total, 1, **dev))
        y = torch.randn(total, D, **dev) * scale
        if case["layout"] == "HND":
            k[h], v[h] = x, y
        else:
            k[:, h], v[:, h] = x, y
    bf = lambda *s: torch.randn(*s, **dev).to(torch.bfloat16)  # noqa: E731
    x = {"k": k, "v": v, "qwin": bf(batch, hq, case["window"], D), "q": bf(batch, hq, D),
         "cu": torch.tensor([0] + [sum(lens[:i + 1]) for i in range(batch)], dtype=torch.int32, device="cuda")}
    if case["cap"]:
        x["tail_k"], x["tail_v"] = bf(batch, case["cap"], hkv, D), bf(batch, case["cap"], hkv, D)
        x["tail_len"] = torch.tensor(_tail_lens(case), dtype=torch.int32, device="cuda")
    return x


def _desc(case):
    total, hkv = sum(_lens(case)), case["hkv"]
    d = spark.SparkDesc()
    d.batch, d.n_q_heads, d.n_kv_heads, d.head_dim = case["batch"], hkv * case["group"], hkv, D
    d.keep, d.keep_v, d.window, d.total_tokens = case["keep"], case["keep_v"], case["window"], total
    d.pack_dtype = spark.PACK_INT8 if case["pack"] == "int8" else spark.PACK_BF16
    d.out_dtype = spark.OUT_F32 if case["out"] == "f32" else spark.OUT_BF16
    if case["layout"] == "HND":
        d.k_token_stride = d.v_token_stride = D
        d.k_head_stride = d.v_head_stride = total * D
    else:
        d.k_token_stride = d.v_token_stride = hkv * D
        d.k_head_stride = d.v_head_stride = D
    d.stats = 1 if case["op"] == "sampled" else 0
    d.tail_capacity = case["cap"]
    return d


SEED = 1234567890123     # of the sampled recovery: a program changes it per step, the work does not depend on it


def prepare(case, seed):
    """The inputs, the description, and the buffers that the program keeps; for a decode step also the packed cache."""
    s = {"case": case, "desc": _desc(case), **_inputs(case, seed)}
    op, desc = case["op"], s["desc"]
    topp = op in ("prune_topp", "topp")
    # (zeroed: the few bytes of padding that the library never writes are then the same in every run)
    s["packed"] = torch.zeros(spark.packed_topp_bytes(desc) if topp else spark.packed_bytes(desc), dtype=torch.uint8, device="cuda")
    if case["keep_v"]:
        s["packed_v"] = torch.zeros(spark.packed_values_bytes(desc), dtype=torch.uint8, device="cuda")
    if not op.startswith("prune"):
        s["out"] = torch.zeros(case["batch"], desc.n_q_heads, D, dtype=torch.float32 if case["out"] == "f32" else torch.bfloat16, device="cuda")
        s["ws"] = spark.new_decode_workspace(desc)
    if not op.startswith("prune") and op != "step":
        if topp:
            spark.prune_topp(desc, s["k"], s["qwin"], s["cu"], case["p"], s["packed"])
        else:
            spark.prune(desc, s["k"], s["qwin"], s["cu"], s["packed"])
        if op == "values":
            spark.prune_values(desc, s["v"], s["packed_v"])
            del s["v"]
        del s["k"], s["qwin"]      # the program has no further use for the dense keys
    return s


def run(s):
    case, desc = s["case"], s["desc"]
    op = case["op"]
    if op == "step":
        spark.prune(desc, s["k"], s["qwin"], s["cu"], s["packed"])
        spark.decode_attn(desc, s["q"], s["packed"], s["v"], s["cu"], s["out"], s["ws"])
        return {"packed": s["packed"], "out": s["out"]}
    if op == "prune":
        spark.prune(desc, s["k"], s["qwin"], s["cu"], s["packed"])
        return {"packed": s["packed"]}
    if op == "prune_kv":
        spark.prune(desc, s["k"], s["qwin"], s["cu"], s["packed"])
        spark.prune_values(desc, s["v"], s["packed_v"])
        return {"packed": s["packed"], "packed_v": s["packed_v"]}
    if op == "prune_topp":
        spark.prune_topp(desc, s["k"], s["qwin"], s["cu"], case["p"], s["packed"])
        return {"packed": s["packed"]}
    if op == "decode":
        spark.decode_attn(desc, s["q"], s["packed"], s["v"], s["cu"], s["out"], s["ws"])
    elif op == "tail":
        spark.decode_attn_tail(desc, s["q"], s["packed"], s["v"], s["cu"], s["tail_k"], s["tail_v"], s["tail_len"], s["out"], s["ws"])
    elif op == "values":
        spark.decode_attn_values(desc, s["q"], s["packed"], s["packed_v"], s["cu"], s["out"], s["ws"])
    elif op == "sampled":
        spark.decode_attn_sampled(desc, s["q"], s["packed"], s["v"], s["cu"], s["out"], s["ws"], spark.RECOVER_GAUSSIAN, SEED)
    else:
        spark.decode_attn_topp(desc, s["q"], s["packed"], s["v"], s["cu"], s["out"], s["ws"])
    return {"out": s["out"]}


# ---------------------------------------------------------------- what a pass cannot do without


def _row_bytes(case):
    """Bytes of one packed key row: 128-bit mask, statistic, (scale), kept entries.  A top-p row keeps about 51 channels on these keys."""
    if case["op"] in ("prune_topp", "topp"):
        return 16 + 4 + 4 + 2 * 51
    return 16 + 4 + (4 + case["keep"] if case["pack"] == "int8" else 2 * case["keep"]) + (8 if case["op"] == "sampled" else 0)


def work(case):
    rows = sum(_lens(case)) * case["hkv"]
    hq = case["hkv"] * case["group"]
    op, g = case["op"], case["group"]
    out = case["batch"] * hq * D * (4 if case["out"] == "f32" else 2)
    win = case["batch"] * hq * case["window"] * D * 2
    key = _row_bytes(case)
    val = 16 + 2 * case["keep_v"] if case["keep_v"] else 2 * D
    score = 2 * g * (51 if case["p"] else case["keep"]) + 2 * g
    prune = {"bytes": rows * (2 * D + key) + win, "flops": rows * 2 * D}
    decode = {"bytes": rows * (key + val) + 3 * case["batch"] * hq * D + out, "flops": rows * (score + 2 * g * D)}
    if op == "step":     # the packed keys that the prune writes are read again by the decode step
        return {"bytes": prune["bytes"] + decode["bytes"], "flops": prune["flops"] + decode["flops"]}
    if op in ("prune", "prune_topp"):
        return prune
    if op == "prune_kv":
        return {"bytes": prune["bytes"] + rows * (2 * D + val), "flops": prune["flops"]}
    if op == "tail":
        extra = sum(_tail_lens(case)) * case["hkv"]
        return {"bytes": decode["bytes"] + extra * 4 * D, "flops": decode["flops"] + extra * 4 * g * D}
    if op == "sampled":  # a variate per pruned entry: a logarithm, a root, a sine or cosine and their hashes
        return {"bytes": decode["bytes"], "flops": decode["flops"] + rows * (D - case["keep"]) * (2 * g + 20)}
    return decode


def tolerance(case):
    """Decode outputs: float32 sums of bf16 products, probabilities to 16 bits, against exact() in 64 bits.

    Packed caches: masks, counts, kept entries, codes and scales have one right value; the mean of the pruned
    saliencies is a float32 sum whose last bits depend on its order (two tree orders over such rows differ in 0.16 to
    0.68 % of the bytes of rows of 216 to 56 bytes: the last byte of the mean in about a third of the rows).
    """
    packed = {"differ": 0.01}
    if case["op"].startswith("prune"):
        return packed
    if case["out"] == "f32":
        # (seen against exact(): 7e-7 to 1.4e-6, sampled 2.2e-6)
        return {"rel": 1e-5 if case["op"] == "sampled" else 6e-6, **packed}
    # (seen against exact(): 1.5e-3, the rounding of the output itself)
    return {"rel": 5e-3, "max": 2e-2, **packed}


# ---------------------------------------------------------------- the same in 64 bits


def _weights(case, x, b, h):
    """Channel weight a of one (sequence, KV head): mean over the group of |mean window query|, rounded once to float32."""
    g = case["group"]
    qbar = x["qwin"][b, h * g:(h + 1) * g].double().sum(1) / case["window"]
    a = torch.zeros(D, dtype=torch.float64, device="cuda")
    for i in range(g):
        a += qbar[i].abs()
    return (a / g).float()


def _kept(case, w):
    """Order of the channels by saliency (larger first, then lower channel) and how many of them each row keeps."""
    order = torch.sort(w, dim=1, descending=True, stable=True).indices
    if not case["p"]:
        return order, torch.full((w.shape[0], 1), case["keep"], device="cuda")
    bits = w.view(torch.int32).long()
    e = (bits >> 23).clamp(min=1)
    mant = (bits & 0x7FFFFF) + torch.where(bits >> 23 > 0, 0x800000, 0)
    units = mant >> (e.amax(1, keepdim=True) - e).clamp(max=40)
    cum = units.gather(1, order).cumsum(1)
    reached = 10000 * cum >= case["p"] * cum[:, -1:]
    return order, reached.int().argmax(1, keepdim=True) + 1


def _mix(x):
    x = x ^ (x >> 16)
    x = (x * 0x85EBCA6B) & 0xFFFFFFFF
    x = x ^ (x >> 13)
    x = (x * 0xC2B2AE35) & 0xFFFFFFFF
    return x ^ (x >> 16)


def _rebuilt(case, x, b, h, s0, s1):
    """The key rows that the scores are taken on: kept entries as stored, pruned ones recovered from the row's statistics."""
    k = (x["k"][h, s0:s1] if case["layout"] == "HND" else x["k"][s0:s1, h]).float()
    a = _weights(case, x, b, h)
    w = a * k.abs()
    order, count = _kept(case, w)
    keep = torch.zeros_like(w, dtype=torch.bool).scatter_(1, order, torch.arange(D, device="cuda").expand_as(w) < count)
    w64, a64 = w.double(), a.double()
    inv = torch.where(a64 > 0, 1.0 / a64, torch.zeros_like(a64))
    if case["op"] == "sampled":
        mean = w64.mean(1, keepdim=True)
        sigma = (w64 - mean).square().mean(1, keepdim=True).sqrt()
        gold, n = 0x9E3779B9, torch.arange(s0, s1, device="cuda").view(-1, 1)
        base = _mix((_mix((_mix(n) + (SEED & 0xFFFFFFFF)) & 0xFFFFFFFF) + h * gold + (SEED >> 32)) & 0xFFFFFFFF)
        c = torch.arange(D, device="cuda").view(1, -1)
        u = ((_mix((base + c * gold) & 0xFFFFFFFF) >> 9).double() + 0.5) / 8388608.0
        radius, turn = (-2.0 * torch.log(u[:, 0::2])).sqrt(), 2.0 * math.pi * u[:, 1::2]
        rec = mean + sigma * torch.stack([radius * torch.cos(turn), radius * torch.sin(turn)], 2).flatten(1)
    else:
        pruned = (D - count).clamp(min=1)
        rec = torch.where(keep, 0.0, w64).sum(1, keepdim=True) / pruned
    kept = k.double()
    if case["pack"] == "int8":
        # (a tensor as divisor: torch multiplies by the reciprocal of a Python number, which rounds differently)
        scale = torch.where(keep, k.abs(), 0.0).amax(1, keepdim=True) / torch.full((1, 1), 127.0, device="cuda")
        kept = torch.where(scale > 0, torch.round(k / scale), 0.0).double() * scale.double()
    return torch.where(keep, kept, rec * inv)


def _values(case, x, h, s0, s1):
    v = x["v"][h, s0:s1] if case["layout"] == "HND" else x["v"][s0:s1, h]
    if case["op"] != "values":
        return v.double()
    order = torch.sort(v.float().abs(), dim=1, descending=True, stable=True).indices
    return torch.zeros(v.shape, dtype=torch.float64, device="cuda").scatter_(1, order[:, :case["keep_v"]], v.double().gather(1, order[:, :case["keep_v"]]))


def exact(case, seed):
    """Decode outputs in float64 from the same inputs.  A packed cache is bytes in a layout of the library's own: no value here."""
    op = case["op"]
    if op.startswith("prune"):
        return None
    x = _inputs(case, seed)
    g, cu = case["group"], x["cu"].tolist()
    out = torch.zeros(case["batch"], case["hkv"] * g, D, dtype=torch.float64, device="cuda")
    for b in range(case["batch"]):
        for h in range(case["hkv"]):
            k, v = _rebuilt(case, x, b, h, cu[b], cu[b + 1]), _values(case, x, h, cu[b], cu[b + 1])
            if op == "tail":
                n = int(x["tail_len"][b])
                k, v = torch.cat([k, x["tail_k"][b, :n, h].double()]), torch.cat([v, x["tail_v"][b, :n, h].double()])
            heads = slice(h * g, (h + 1) * g)
            out[b, heads] = torch.softmax(x["q"][b, heads].double() @ k.T / math.sqrt(D), 1) @ v
    return {"packed": None, "out": out} if op == "step" else {"out": out}
