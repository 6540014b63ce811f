"""Timed cases of the mixed prefill+decode attention step on one GPU.

A case is one serving iteration (or the part of it that a program calls by
itself): a batch of decode rows and prefill chunks over a paged KV cache,
through the binding's public calls.  The batches come from the ranges of the
workloads in ``workloads/configs.py`` and of the paper they stand in for (up
to 256 running requests, contexts up to 128K tokens, decode contexts of
65K-98K, chunks on reused prefixes under a per-step token budget, TP4 decode
workers), at whole heads and at one GPU's TP4 share of them.

Fields of a case:

``call``    what the program calls:
            ``step``      append_attention (append and attention in one call)
            ``two_calls`` kv_append, then mixed_paged_attention
            ``rope_step`` kv_append_rope, then mixed_paged_attention
            ``coexec``    kv_append, then coexec_attention (the planner picks
                          one stream or CU-partitioned streams)
            ``mixed``     mixed_paged_attention on an appended cache
``cache``   bf16, fp8 (E4M3 codes beside bf16 rows) or f32
``hq, hkv, d``             query heads, KV heads, head_dim
``rows, ctx_lo, ctx_hi``   decode rows and the range of their contexts
``chunks, c_lo, c_hi, p_lo, p_hi``  prefill chunks, the ranges of their
                           lengths and of their cached prefixes
``lens``    seed of the lengths.  Contexts spread over their range by their
            logarithm where it spans more than a factor of ten.

The seed given to ``prepare`` is one step of that batch: it draws the values
and the block tables, and every decode context is ``seed % 16`` tokens longer
than the case's, as the contexts of a running batch grow from step to step
(so the plan of one state is not the plan of the next).
"""

import math

import numpy as np
import torch

import paper_2609_27085_amd as mpa

BLOCK = 16
K_SCALE, V_SCALE = 0.0141, 0.0167  # fp8: 448 codes cover 6.3 and 7.5 sigma of N(0, 1)
ROPE_BASE = 10000.0


def _case(name, call, cache, heads, rows=0, ctx=(1, 1), chunks=0, c=(2, 2), p=(0, 0), lens=0):
    case = {"name": name} if name else {}
    case.update(call=call, cache=cache, hq=heads[0], hkv=heads[1], d=heads[2], rows=rows, ctx_lo=ctx[0],
                ctx_hi=ctx[1], chunks=chunks, c_lo=c[0], c_hi=c[1], p_lo=p[0], p_hi=p[1], lens=lens)
    return case


def listed():
    return [
        # The smallest step: a few short requests and the tail of a prompt.  Launches and host time.
        _case("tiny_step", "step", "bf16", (4, 2, 64), 4, (64, 256), 1, (32, 32), (96, 96), lens=1),
        # A lightly loaded TP4 worker between prompts: decode only, rotary embedding in the append.
        _case("chat_tp4_rope", "rope_step", "bf16", (8, 2, 128), 16, (200, 8192), lens=2),
        # Two or three agent sessions of the paper's 65K-98K contexts: few rows, long ones.
        _case("few_long", "step", "bf16", (32, 8, 128), 3, (65536, 98304), lens=3),
        # The 64-row decode batch of an 8B-class layer.
        _case("decode8b", "step", "bf16", (32, 8, 128), 64, (512, 8192), lens=4),
        # A larger decode batch on fp8 caches.
        _case("decode_fp8", "step", "fp8", (32, 8, 128), 128, (1024, 16384), lens=5),
        # A prompt's first pass: no prefix, ragged length, rotary embedding, nothing to decode beside it.
        _case("prompt_rope", "rope_step", "bf16", (32, 8, 128), 0, (1, 1), 1, (3001, 3001), (0, 0), lens=6),
        # A lease's small token budget on a TP4 worker of 64-wide heads: a short chunk on a long prefix.
        _case("budget_tp4_d64", "step", "bf16", (16, 2, 64), 48, (2048, 16384), 1, (300, 300), (20011, 20011),
              lens=7),
        # Decode rows beside two chunks of 2,048 tokens: the lent-compute step.
        _case("lent", "step", "bf16", (32, 8, 128), 128, (1024, 16384), 2, (2048, 2048), (0, 8192), lens=8),
        # The same kind of step on fp8 caches, appended by a call of its own.
        _case("mixed_fp8", "two_calls", "fp8", (64, 8, 128), 64, (1024, 16384), 3, (512, 3000), (2048, 16384),
              lens=9),
        # 256 agent sessions and four chunks on long reused prefixes, the planner choosing how to run them.
        _case("agentic", "coexec", "bf16", (64, 8, 128), 256, (512, 32768), 4, (512, 4096), (2048, 20480), lens=10),
        # A float32 step: what a user runs to check a model's numbers.
        _case("f32_step", "step", "f32", (8, 2, 128), 8, (256, 4096), 1, (500, 500), (1000, 1000), lens=11),
        # The largest step: 32 rows of 32K-128K context and an 8,192-token chunk on a 64K prefix.
        _case("longctx", "mixed", "bf16", (32, 8, 128), 32, (32768, 131072), 1, (8192, 8192), (65536, 65536),
              lens=12),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """A case of the listed ranges: 2-64 query heads over 1-8 KV heads, 1-256 decode rows of 1-128K keys, 0-4 chunks
    of 2-8,192 tokens on prefixes of 0-64K, redrawn while its bytes or its work pass about a third of the largest's."""
    while True:
        cache = rng.choice(["bf16", "bf16", "bf16", "fp8", "fp8", "f32"])
        d = rng.choice([64, 128, 128])
        hkv = rng.choice([1, 2, 2, 4, 8, 8])
        hq = hkv * rng.choice([1, 2, 4, 4, 5, 8, 8])
        calls = ["step", "step", "two_calls", "rope_step", "mixed"] + (["coexec"] if cache == "bf16" else [])
        call = rng.choice(calls)
        kind = rng.choice(["decode", "prefill", "mixed", "mixed"])
        rows = chunks = 0
        ctx, c, p = (1, 1), (2, 2), (0, 0)
        if kind != "prefill":
            rows = _log_int(rng, 1, 256)
            lo = _log_int(rng, 1, 32768)
            ctx = (lo, min(131072, lo * _log_int(rng, 1, 16)))
        if kind != "decode":
            chunks = rng.randint(1, 4)
            lo = _log_int(rng, 2, 4096)
            c = (lo, min(8192, lo * rng.randint(1, 4)))
            if rng.random() < 0.8:
                lo = _log_int(rng, 16, 32768)
                p = (lo, min(65536, lo * rng.randint(1, 4)))
        if cache == "f32":  # numbers are checked on small steps
            if rows > 16 or ctx[1] > 16384 or c[1] > 1024 or p[1] > 4096:
                continue
        case = _case("", call, cache, (hq, hkv, d), rows, ctx, chunks, c, p, lens=rng.randrange(1 << 20))
        w = work(case)
        # about a third of longctx in bytes and in work
        if w["bytes"] <= 4e9 and w["flops"] <= 3.5e12:
            return case


def _lengths(case):
    """[(context after the step, new tokens)] of the case, decode rows first."""
    rng = np.random.default_rng(case["lens"])

    def spread(lo, hi):
        if lo > 0 and hi > 10 * lo:
            return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))
        return int(rng.integers(lo, hi, endpoint=True))

    seqs = [(spread(case["ctx_lo"], case["ctx_hi"]), 1) for _ in range(case["rows"])]
    for _ in range(case["chunks"]):
        c = spread(case["c_lo"], case["c_hi"])
        seqs.append((spread(case["p_lo"], case["p_hi"]) + c, c))
    return seqs


def _step_lengths(case, seed):
    grown = int(seed) % 16
    return [(n + grown if q == 1 else n, q) for n, q in _lengths(case)]


def _gen(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed))
    return g


def _normal(shape, dtype, gen, scale=None):
    """N(0, 1) in float32, rounded to dtype (fp8: the codes of the values over `scale`)."""
    t = torch.empty(shape, dtype=torch.uint8 if scale else dtype, device="cuda")
    flat = t.view(-1)
    for i in range(0, flat.numel(), 1 << 28):
        part = flat[i: i + (1 << 28)]
        x = torch.randn(part.numel(), generator=gen, device="cuda")
        part.copy_((x / scale).clamp_(-448, 448).to(torch.float8_e4m3fn).view(torch.uint8) if scale else x)
    return t


def prepare(case, seed):
    seqs = _step_lengths(case, seed)
    hq, hkv, d, cache = case["hq"], case["hkv"], case["d"], case["cache"]
    row = torch.float32 if cache == "f32" else torch.bfloat16
    x = 4 if cache == "f32" else 8
    per = [-(-n // BLOCK) for n, _ in seqs]
    need = sum(-(-(n + 15) // BLOCK) for n, _ in _lengths(case))
    pool = need + need // 20 + 1
    order = np.random.default_rng(seed).permutation(pool).astype(np.int32)
    tables = np.zeros((len(seqs), max(per)), dtype=np.int32)
    at = 0
    for i, n in enumerate(per):
        tables[i, :n] = order[at: at + n]
        at += n
    lens = np.array([n for n, _ in seqs], dtype=np.int32)
    starts = np.concatenate([[0], np.cumsum([q for _, q in seqs])]).astype(np.int32)
    t = int(starts[-1])
    gen = _gen(seed)
    s = {"case": case, "seqs": seqs, "lens": lens, "starts": starts}
    s["q"] = _normal((t, hq, d), row, gen)
    s["k_new"] = _normal((t, hkv, d), row, gen)
    s["v_new"] = _normal((t, hkv, d), row, gen)
    fp8 = cache == "fp8"
    s["k_cache"] = _normal((pool, hkv, d // x, BLOCK, x), row, gen, K_SCALE if fp8 else None)
    s["v_cache"] = _normal((pool, hkv, d, BLOCK), row, gen, V_SCALE if fp8 else None)
    s["scales"] = {"k_scale": K_SCALE, "v_scale": V_SCALE} if fp8 else {}
    dev = lambda a: torch.from_numpy(a).cuda()  # noqa: E731
    s["tables"], s["lens_dev"], s["starts_dev"] = dev(tables), dev(lens), dev(starts)
    s["out"] = torch.empty_like(s["q"])
    s["lse"] = torch.empty((t, hq), dtype=torch.float32, device="cuda")
    if case["call"] == "rope_step":
        s["cos_sin"] = _angles(int(lens.max()), d).float().cuda().contiguous()
    s["workspace"] = mpa.alloc_workspace(s["q"], s["k_cache"], s["tables"], lens, starts)
    return s


def _angles(positions, d):
    j = torch.arange(d // 2, dtype=torch.float64)
    a = torch.arange(positions, dtype=torch.float64)[:, None] * ROPE_BASE ** (-2 * j / d)
    return torch.stack([a.cos(), a.sin()], dim=-1)


def run(s):
    """One step.  Appending is idempotent; the rotary append rotates q in place, so a later pass on the same state
    is a step with other queries of the same size."""
    call = s["case"]["call"]
    meta = (s["tables"], s["lens_dev"], s["starts_dev"], s["lens"], s["starts"])
    caches = (s["k_cache"], s["v_cache"])
    new = (s["k_new"], s["v_new"])
    kw = dict(lse=s["lse"], workspace=s["workspace"], **s["scales"])
    if call == "step":
        mpa.append_attention(s["q"], *new, *caches, *meta, s["out"], **kw)
    else:
        if call == "rope_step":
            mpa.kv_append_rope(s["q"], *new, *caches, *meta, s["cos_sin"], **s["scales"])
        elif call != "mixed":
            mpa.kv_append(*new, *caches, *meta, **s["scales"])
        if call == "coexec":
            mpa.coexec_attention(s["q"], *caches, *meta, s["out"], **kw)
        else:
            mpa.mixed_paged_attention(s["q"], *caches, *meta, s["out"], **kw)
    got = {"out": s["out"], "lse": s["lse"]}
    whole = {1: torch.uint8, 2: torch.int16, 4: torch.int32}  # bits: copied rows are the same or wrong
    if call != "mixed":
        for name in ("k_cache", "v_cache"):
            got[name] = s[name].view(whole[s[name].element_size()])
    if call == "rope_step":
        got["q"] = s["q"].view(whole[s["q"].element_size()])
    return got


def work(case):
    """Keys and values read once per sequence and KV head, queries read, outputs written, new rows read and written;
    4 d operations per query head and visible (query, key) pair."""
    seqs = _lengths(case)
    hq, hkv, d = case["hq"], case["hkv"], case["d"]
    elem = {"bf16": 2, "fp8": 1, "f32": 4}[case["cache"]]
    row = 4 if case["cache"] == "f32" else 2
    t = sum(q for _, q in seqs)
    moved = 2 * sum(n for n, _ in seqs) * hkv * d * elem + 2 * t * hq * d * row + 4 * t * hq
    if case["call"] != "mixed":
        moved += 2 * t * hkv * d * (row + elem)
    if case["call"] == "rope_step":
        moved += t * hq * d * row  # the rotated queries are written
    pairs = sum(q * (n - q) + q * (q + 1) // 2 for n, q in seqs)
    return {"bytes": moved, "flops": 4 * d * hq * pairs}


def tolerance(case):
    """bf16 rows: outputs carry bf16's rounding (2^-9) and that of the probabilities before the value product, f32
    rows the rounding of 32-bit sums.  About four times what the path shows against `exact`; cache bits and rotated
    queries are whole values and stay the same."""
    if case["cache"] == "f32":
        return {"rel": 5e-6, "max": 2e-4}
    return {"rel": 1e-2, "max": 6e-2}


def exact(case, seed):
    """The step in float64 (rotated and appended rows rounded as the cache holds them), sequence by sequence and KV
    head by KV head.  Cache bits and rotated queries have no float64 value."""
    s = prepare(case, seed)
    hq, hkv, d, cache = case["hq"], case["hkv"], case["d"], case["cache"]
    group = hq // hkv
    q, k_new, v_new = s["q"], s["k_new"], s["v_new"]
    if case["call"] == "rope_step":
        pos = np.concatenate([np.arange(n - c, n) for n, c in s["seqs"]])
        cs = s["cos_sin"].double()[torch.from_numpy(pos).cuda()][:, None]
        q, k_new = (_rotated(r, cs) for r in (q, k_new))
    if cache == "fp8":
        code = lambda r, c: (r.float() * (1 / np.float32(c))).clamp(-448, 448).to(torch.float8_e4m3fn)  # noqa: E731
        k_new, v_new = code(k_new, K_SCALE).double() * K_SCALE, code(v_new, V_SCALE).double() * V_SCALE
    out = torch.empty((q.shape[0], hq, d), dtype=torch.float64, device="cuda")
    lse = torch.empty((q.shape[0], hq), dtype=torch.float64, device="cuda")
    for i, (n, c) in enumerate(s["seqs"]):
        t0 = int(s["starts"][i])
        blocks = s["tables"][i, : -(-n // BLOCK)].long()
        for h in range(hkv):
            k = s["k_cache"][blocks, h]  # [blocks][d/x][16][x]
            v = s["v_cache"][blocks, h]  # [blocks][d][16]
            if cache == "fp8":
                k = k.view(torch.float8_e4m3fn).double() * K_SCALE
                v = v.view(torch.float8_e4m3fn).double() * V_SCALE
            k = k.double().permute(0, 2, 1, 3).reshape(-1, d)[:n].contiguous()
            v = v.double().permute(0, 2, 1).reshape(-1, d)[:n].contiguous()
            if case["call"] != "mixed":
                k[n - c:] = k_new[t0: t0 + c, h].double()
                v[n - c:] = v_new[t0: t0 + c, h].double()
            kt = k.t().contiguous()
            heads = slice(h * group, (h + 1) * group)
            for a in range(0, c, 256):
                b = min(c, a + 256)
                rows = q[t0 + a: t0 + b, heads].double().reshape(-1, d)
                seen = n - c + b
                scores = (rows @ kt[:, :seen].contiguous()).view(b - a, group, seen) / math.sqrt(d)
                if c > 1:
                    last = torch.arange(n - c + a, n - c + b, device="cuda")[:, None, None]
                    scores.masked_fill_(torch.arange(seen, device="cuda") > last, -math.inf)
                total = torch.logsumexp(scores, -1)
                p = torch.exp_(scores.sub_(total[..., None]))
                out[t0 + a: t0 + b, heads] = (p.view(-1, seen) @ v[:seen]).view(b - a, group, d)
                lse[t0 + a: t0 + b, heads] = total
    got = {"out": out, "lse": lse}
    if case["call"] != "mixed":
        got.update(k_cache=None, v_cache=None)
    if case["call"] == "rope_step":
        got["q"] = None
    return got


def _rotated(rows, cs):
    half = rows.shape[-1] // 2
    a, b = rows.double()[..., :half], rows.double()[..., half:]
    cos, sin = cs[..., 0], cs[..., 1]
    return torch.cat([a * cos - b * sin, b * cos + a * sin], dim=-1).to(rows.dtype)
