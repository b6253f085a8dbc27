"""The performance cases of this library: what its users have it do.

Every case is one pass through ``DecodeAttention``, the library's torch
wrapper: a decode-attention call (one new query token per sequence over its
whole KV cache), the same with the new token's row appended in the launch, a
decode step of several layers replayed as a captured HIP graph, or a prefill
of new tokens over a cached prefix. Head counts, sizes and length ranges are
those of the named workloads in ``workloads/synth.py`` and of the agent the
library serves: prompts and compressed contexts of a few thousand tokens,
observations of 128-2048 new tokens over 8-32K prefixes, full histories of
32K-128K.

A case is a dict of plain values:
  op        "decode", "append" (decode with the fused append), "layers"
            (a captured decode step of ``layers`` layers), or "prefill"
  dtype     "f32", "bf16" or "fp8" (cache codes; q is bf16)
  batch, hq, hkv, d
  lo, hi    context lengths are uniform in [lo, hi], drawn from ``mix``;
            the call's length bound is hi
  page      0 for a contiguous (packed) cache, else tokens per page
  new_lo, new_hi   prefill only: new tokens per sequence, uniform (0 means
            all of the context: an uncached prefill)
  peaked    5% of the keys are scaled by 8 (a peaked softmax)
"""

import math
import random

import torch

from paper_2605_30842_amd.binding import DecodeAttention, kv_cache_pair

DEVICE = "cuda:0"
FP8_SCALE = 2.0 ** -6  # K = code value * scale, V alike


def _case(op, dtype, batch, hq, hkv, d, lo, hi, page=0, mix=1, layers=1, new_lo=0, new_hi=0, peaked=False):
    return dict(op=op, dtype=dtype, batch=batch, hq=hq, hkv=hkv, d=d, lo=lo, hi=hi, page=page, mix=mix,
                layers=layers, new_lo=new_lo, new_hi=new_hi, peaked=peaked)


def listed():
    def named(name, *a, **kw):
        return dict(_case(*a, **kw), name=name)

    return [
        # The smallest workload: a float32 cache, where a step is launch and round-trip latency.
        named("decode_f32_B1_L2048", "decode", "f32", 1, 8, 2, 64, 2048, 2048),
        # One user's decode over a compressed context (summary plus recent buffer), as a decode loop runs
        # it: the layers of one step captured in a graph.
        named("layers16_bf16_B1_L6000", "layers", "bf16", 1, 32, 8, 128, 6001, 6001, layers=16),
        # One user's decode over a full history (the headline workload).
        named("decode_bf16_B1_L32768", "decode", "bf16", 1, 32, 8, 128, 32768, 32768),
        # A batch of full histories of very different lengths, packed.
        named("decode_bf16_ragged_B16_L4k-64k", "decode", "bf16", 16, 32, 8, 128, 4096, 65536, mix=3),
        # A serving batch over a paged cache with some keys far above the others.
        named("decode_bf16_paged16_B64_L2k-16k", "decode", "bf16", 64, 32, 8, 128, 2048, 16384, page=16, mix=4,
              peaked=True),
        # The longest contexts, eight query heads to a KV head: 4 GiB of K and V.
        named("decode_bf16_paged64_B8_L131072_G8", "decode", "bf16", 8, 64, 8, 128, 131072, 131072, page=64),
        # The headline shape over an FP8 cache.
        named("decode_fp8_B1_L32768", "decode", "fp8", 1, 32, 8, 128, 32768, 32768),
        # A small serving batch of agent prompts over an FP8 paged cache, each step appending its token.
        named("append_fp8_paged64_B8_L1k-7k", "append", "fp8", 8, 32, 8, 128, 1000, 7000, page=64, mix=8),
        # A token-granular pool (one-token pages), as prefix-sharing servers keep it.
        named("decode_bf16_paged1_B6_L2k-12k", "decode", "bf16", 6, 32, 8, 128, 2000, 12000, page=1, mix=9),
        # One observation of an agent's step over its cached history.
        named("prefill_bf16_B1_L24k_M300", "prefill", "bf16", 1, 32, 8, 128, 24300, 24300, new_lo=300, new_hi=300),
        # The whole context prefilled anew after a summary update (plain causal attention).
        named("prefill_bf16_uncached_B1_L8192", "prefill", "bf16", 1, 32, 8, 128, 8192, 8192),
        # Observations of several agents over their cached histories, paged.
        named("prefill_bf16_paged16_B8_L8k-32k_M128-2048", "prefill", "bf16", 8, 32, 8, 128, 8192, 32768, page=16,
              mix=12, new_lo=128, new_hi=2048),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


MAX_DECODE_BYTES = 2 << 30   # K and V of a drawn decode case
MAX_PREFILL_FLOPS = 2.0e12   # of a drawn prefill case


def draw(rng):
    """One more case: the listed kinds over their ranges (lengths and batches log-uniform, odd sizes included)."""
    kind = rng.choice(["decode", "decode", "append", "layers", "f32", "prefill", "prefill", "uncached"])
    mix = rng.randrange(1 << 30)
    while True:
        if kind == "f32":
            hkv = rng.choice([2, 4, 8])
            hi = _log_int(rng, 500, 16384)
            c = _case("decode", "f32", _log_int(rng, 1, 8), hkv * rng.choice([1, 2, 4, 8]), hkv, rng.choice([64, 128]),
                      max(1, int(hi * rng.uniform(0.3, 1.0))), hi, page=rng.choice([0, 0, 16]), mix=mix)
        elif kind in ("decode", "append", "layers"):
            hkv = rng.choice([2, 4, 8, 8])
            hq = hkv * rng.choice([1, 2, 4, 4, 8, 16])
            hi = _log_int(rng, 500, 131072 if kind == "decode" else 12000)
            batch = 1 if kind == "layers" else _log_int(rng, 1, 64 if kind == "decode" else 16)
            c = _case(kind, rng.choice(["bf16", "bf16", "fp8"]), batch, hq, hkv, rng.choice([128, 128, 64]),
                      max(1, int(hi * rng.uniform(0.1, 1.0))), hi, page=rng.choice([0, 0, 16, 64, 1]), mix=mix,
                      layers=rng.randint(4, 16) if kind == "layers" else 1, peaked=rng.random() < 0.2)
            if c["dtype"] == "fp8":
                c["peaked"] = False  # scaled keys would leave the codes' range
        elif kind == "prefill":
            hkv = rng.choice([4, 8, 8])
            hi = _log_int(rng, 2100, 32768)
            m = _log_int(rng, 128, 2048)
            c = _case("prefill", "bf16", _log_int(rng, 1, 8), hkv * rng.choice([2, 4, 4, 8]), hkv,
                      rng.choice([128, 128, 64]), max(m, int(hi * rng.uniform(0.25, 1.0))), hi,
                      page=rng.choice([0, 16, 64, 1]), mix=mix, new_lo=max(1, int(m * rng.uniform(0.1, 1.0))), new_hi=m)
        else:
            hkv = rng.choice([4, 8, 8])
            hi = _log_int(rng, 500, 8192)
            c = _case("prefill", "bf16", _log_int(rng, 1, 4), hkv * rng.choice([2, 4, 4, 8]), hkv,
                      rng.choice([128, 128, 64]), max(1, int(hi * rng.uniform(0.5, 1.0))), hi,
                      page=rng.choice([0, 16]), mix=mix)
        w = work(c)
        if c["op"] == "prefill" and w["flops"] <= MAX_PREFILL_FLOPS:
            return c
        if c["op"] != "prefill" and w["bytes"] <= MAX_DECODE_BYTES:
            return c


# ------------------------------------------------------------------ sizes


def _lengths(case):
    r = random.Random(case["mix"])
    return [r.randint(case["lo"], case["hi"]) for _ in range(case["batch"])]


def _new_tokens(case):
    if case["new_hi"] == 0:
        return _lengths(case)
    r = random.Random(case["mix"] + 1)
    return [min(r.randint(case["new_lo"], case["new_hi"]), n) for n in _lengths(case)]


def _elem_bytes(case):
    return {"f32": 4, "bf16": 2, "fp8": 1}[case["dtype"]]


def work(case):
    """K, V, queries and new rows read once, outputs (and appended rows) written once; 2 D flops for q.k and
    2 D for p.v per query head and visible key."""
    lens, d, hq = _lengths(case), case["d"], case["hq"]
    row = 2 * case["hkv"] * d * _elem_bytes(case)  # K and V of one token
    qb = 4 if case["dtype"] == "f32" else 2
    if case["op"] == "prefill":
        new = _new_tokens(case)
        queries = sum(new)
        pairs = sum((n - m) * m + m * (m + 1) // 2 for n, m in zip(lens, new))
    else:
        queries, pairs = len(lens), sum(lens)
    nbytes = sum(lens) * row + queries * hq * (d * qb + d * 4 + 4)
    if case["op"] == "append":
        nbytes += len(lens) * row  # the rows stored; the new rows are read in place of the stored ones
    n = case["layers"]
    return {"bytes": n * nbytes, "flops": n * 4 * d * hq * pairs}


# ------------------------------------------------------------------ inputs


def _fill(t, g, scale_rows, quantize):
    """N(0, 1) values into a cache tensor, in parts (FP8: codes of the values divided by the scale)."""
    rows = t.view(-1, t.shape[-2], t.shape[-1])
    step = max(1, (1 << 26) // (rows.shape[1] * rows.shape[2]))
    for i in range(0, rows.shape[0], step):
        part = rows[i:i + step]
        x = torch.randn(part.shape, generator=g, device=t.device)
        if scale_rows:
            big = torch.rand(part.shape[:2], generator=g, device=t.device) < 0.05
            x *= torch.where(big, 8.0, 1.0)[..., None]
        if quantize:
            part.copy_((x / FP8_SCALE).clamp_(-448.0, 448.0).to(torch.float8_e4m3fn).view(torch.uint8))
        else:
            part.copy_(x)


def _inputs(case, seed):
    """The tensors of a call, made from the seed: a list with one dict for every layer."""
    g = torch.Generator(device=DEVICE).manual_seed(seed)
    lens, hq, hkv, d, page = _lengths(case), case["hq"], case["hkv"], case["d"], case["page"]
    cache_dtype = {"f32": torch.float32, "bf16": torch.bfloat16, "fp8": torch.uint8}[case["dtype"]]
    q_dtype = torch.float32 if case["dtype"] == "f32" else torch.bfloat16
    fp8 = case["dtype"] == "fp8"
    ctx = torch.tensor(lens, dtype=torch.int32, device=DEVICE)
    starts = [sum(lens[:b]) for b in range(len(lens))]
    layers = []
    for _ in range(case["layers"]):
        x = dict(ctx_lens=ctx)
        if page:
            counts = [-(-n // page) for n in lens]
            k, v = kv_cache_pair((sum(counts), page, hkv, d), cache_dtype, DEVICE)
            perm = torch.randperm(sum(counts), generator=g, device=DEVICE).to(torch.int32)
            table = torch.full((len(lens), -(-case["hi"] // page)), -1, dtype=torch.int32, device=DEVICE)
            for b, n in enumerate(counts):
                first = sum(counts[:b])
                table[b, :n] = perm[first:first + n]
            x["block_table"] = table
        else:
            k, v = kv_cache_pair((sum(lens), hkv, d), cache_dtype, DEVICE)
            x["seq_start"] = torch.tensor(starts, dtype=torch.int64, device=DEVICE)
        _fill(k, g, case["peaked"], fp8)
        _fill(v, g, False, fp8)
        x["k"], x["v"] = k, v
        queries = len(lens)
        if case["op"] == "prefill":
            new = _new_tokens(case)
            queries = sum(new)
            x["q_start"] = torch.tensor([sum(new[:b]) for b in range(len(new))], dtype=torch.int64, device=DEVICE)
            x["q_lens"] = torch.tensor(new, dtype=torch.int32, device=DEVICE)
        x["q"] = torch.randn((queries, hq, d), generator=g, device=DEVICE).to(q_dtype)
        if case["op"] == "append":
            for name in ("new_k", "new_v"):
                x[name] = torch.empty((len(lens), hkv, d), dtype=cache_dtype, device=DEVICE)
                _fill(x[name], g, False, fp8)
        layers.append(x)
    return layers


def _call(case, op, x):
    """One attention call of the case on the tensors of one layer; its outputs are x["out"] and x["lse"]."""
    bound, out, lse = case["hi"], x["out"], x["lse"]
    paged = case["page"] > 0
    where = x["block_table"] if paged else x["seq_start"]
    if case["op"] == "prefill":
        call = op.prefill_paged if paged else op.prefill
        call(x["q"], x["q_start"], x["q_lens"], x["max_q_len"], x["k"], x["v"], where, x["ctx_lens"], bound, out=out,
             lse=lse)
    elif case["op"] == "append":
        call = op.append_forward_paged if paged else op.append_forward
        call(x["q"], x["new_k"], x["new_v"], x["k"], x["v"], where, x["ctx_lens"], bound, out=out, lse=lse)
    else:
        call = op.forward_paged if paged else op.forward
        call(x["q"], x["k"], x["v"], where, x["ctx_lens"], bound, out=out, lse=lse)


def prepare(case, seed):
    scales = dict(k_scale=FP8_SCALE, v_scale=FP8_SCALE) if case["dtype"] == "fp8" else {}
    op = DecodeAttention(case["hq"], case["hkv"], case["d"], case["dtype"], 1.0 / math.sqrt(case["d"]), case["batch"],
                         case["hi"], **scales)
    layers = _inputs(case, seed)
    for x in layers:
        queries = x["q"].shape[0]
        x["out"] = torch.empty((queries, case["hq"], case["d"]), dtype=torch.float32, device=DEVICE)
        x["lse"] = torch.empty((queries, case["hq"]), dtype=torch.float32, device=DEVICE)
        if case["op"] == "prefill":
            x["max_q_len"] = max(_new_tokens(case))
    state = dict(case=case, op=op, layers=layers)
    if case["op"] == "layers":
        # The decode loop's step: captured once, replayed for every token.
        for x in layers:
            _call(case, op, x)
        torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph):
            for x in layers:
                _call(case, op, x)
        state["graph"] = graph
    return state


def run(state):
    case, layers = state["case"], state["layers"]
    if case["op"] == "layers":
        state["graph"].replay()
        return [(x["out"], x["lse"]) for x in layers]
    x = layers[0]
    _call(case, state["op"], x)
    if case["op"] == "append":
        return x["out"], x["lse"], x["k"], x["v"]
    return x["out"], x["lse"]


# ------------------------------------------------------------------ the same in 64 bits


def _wide(case, t):
    """A cache tensor's values in 64 bits."""
    if case["dtype"] == "fp8":
        return t.view(torch.float8_e4m3fn).to(torch.float32).to(torch.float64) * FP8_SCALE
    return t.to(torch.float64)


def _attend(q, k, v, limits, scale):
    """softmax(scale q k^T) v of rows q [m, d]; row i sees the first limits[i] keys."""
    s = (q @ k.t()) * scale
    pos = torch.arange(k.shape[0], device=k.device)
    s.masked_fill_(pos[None, :] >= limits[:, None], -math.inf)
    lse = torch.logsumexp(s, dim=1)
    return torch.exp_(s.sub_(lse[:, None])) @ v, lse


def exact(case, seed):
    results = []
    group = case["hq"] // case["hkv"]
    scale = 1.0 / math.sqrt(case["d"])
    lens = _lengths(case)
    new = _new_tokens(case) if case["op"] == "prefill" else [1] * len(lens)
    for x in _inputs(case, seed):
        out = torch.zeros(x["q"].shape, dtype=torch.float64, device=DEVICE)
        lse = torch.zeros(x["q"].shape[:2], dtype=torch.float64, device=DEVICE)
        q0 = 0
        for b, n in enumerate(lens):
            if case["page"]:
                pages = x["block_table"][b, :-(-n // case["page"])].long()
                tokens = torch.arange(n, device=DEVICE)
                rows = pages[tokens // case["page"]] * case["page"] + tokens % case["page"]
            else:
                rows = int(x["seq_start"][b]) + torch.arange(n, device=DEVICE)
            flat_k = x["k"].view(-1, case["hkv"], case["d"])
            flat_v = x["v"].view(-1, case["hkv"], case["d"])
            if case["op"] == "append":
                flat_k[rows[-1]] = x["new_k"][b]
                flat_v[rows[-1]] = x["new_v"][b]
            m = new[b]
            for hk in range(case["hkv"]):
                k = _wide(case, flat_k[rows, hk])
                v = _wide(case, flat_v[rows, hk])
                for h in range(hk * group, (hk + 1) * group):
                    for i in range(0, m, 1024):
                        j = min(i + 1024, m)
                        limits = n - m + 1 + torch.arange(i, j, device=DEVICE)
                        o, s = _attend(x["q"][q0 + i:q0 + j, h].to(torch.float64), k, v, limits, scale)
                        out[q0 + i:q0 + j, h] = o
                        lse[q0 + i:q0 + j, h] = s
            q0 += m
        results.append((out, lse, x["k"], x["v"]) if case["op"] == "append" else (out, lse))
    return results if case["op"] == "layers" else results[0]


def tolerance(case):
    # About four times the largest error against 64-bit arithmetic: float32 sums (2e-7 over the result's
    # norm), and for bf16 and FP8 caches weights carried as two bf16 values, 16 significant bits (5e-6).
    return {"rel": 1e-6, "max": 1e-5} if case["dtype"] == "f32" else {"rel": 2e-5, "max": 3e-4}
