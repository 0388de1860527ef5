"""The work a user of this library has it do, as timed cases.

Each case is one call, or one short sequence of calls, through the Python entry points: decode
attention over a paged KV cache (bf16 and E4M3, head_dim 64 and 128), the same with prefix sharing,
the KV append that precedes it in a decode step, and a whole generation by the decode engine.

``listed()`` gives the fixed cases, ``draw(rng)`` another one of the same ranges: batch 1 to 512,
contexts of 1 to 32K tokens, 1 to 16 query heads per KV head.
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_2504_15930_amd import engine, sl

PAGE = 16
DEV = "cuda:0"


def _attn(name, batch, hq, hkv, d, law, a, b, cap, kv="bf16", api="attn"):
    return dict(name=name, kind="attn", api=api, kv=kv, batch=batch, hq=hq, hkv=hkv, d=d, law=law, a=a, b=b, cap=cap)


def listed():
    return [
        # The smallest decode step in use: a test-sized model, a handful of short contexts. Latency.
        _attn("attn_tiny", 8, 4, 2, 64, "uniform", 1, 256, 0),
        # The end of a generation: a few long samples are left of a 7B-like batch.
        _attn("attn_tail", 5, 28, 4, 128, "uniform", 2048, 16384, 0),
        # An ordinary serving step: a moderate batch of medium contexts, 7B-like heads.
        _attn("attn_mid", 67, 28, 4, 128, "uniform", 128, 4096, 0),
        # The rollout batch of a 7B-like model: long-tailed contexts (the headline workload).
        _attn("attn_7b", 256, 28, 4, 128, "lognormal", 512, 2048, 16384),
        # The same for a 72B-like model: the largest step.
        _attn("attn_72b", 512, 64, 8, 128, "lognormal", 1024, 4096, 32768),
        # Stragglers only: few samples, all of them very long.
        _attn("attn_straggler", 16, 64, 8, 128, "uniform", 8192, 32768, 0),
        # Twice the batch in the same memory: an E4M3 cache.
        _attn("attn_7b_fp8", 512, 28, 4, 128, "lognormal", 512, 2048, 32768, kv="e4m3"),
        # head_dim 64 (the other supported one), a large batch of short and medium contexts.
        _attn("attn_d64", 384, 32, 8, 64, "uniform", 1, 2048, 0),
        # Several samples per prompt share the prompt's pages (GRPO): 8 each, bf16.
        dict(name="prefix_bf16", kind="prefix", kv="bf16", prompts=32, samples=8, prompt=1024, median=512, cap=4096,
             hq=28, hkv=4, d=128),
        # 16 samples per prompt over an E4M3 cache, prompt lengths not a multiple of the page.
        dict(name="prefix_fp8", kind="prefix", kv="e4m3", prompts=16, samples=16, prompt=1000, median=512, cap=4096,
             hq=28, hkv=4, d=128),
        # A layer's whole decode step with an E4M3 cache: quantise-on-write of the new rows, then attention.
        dict(name="step_fp8", kind="step", kv="e4m3", batch=96, hq=28, hkv=4, d=128, law="uniform", a=64, b=2048, cap=0),
        # A whole generation: continuous batching of 96 long-tailed samples on 32 slots, from creating the
        # engine to its last step (thousands of steps; most of them small).
        dict(name="generate", kind="generate", kv="bf16", samples=96, slots=32, prompt_lo=128, prompt_hi=512,
             median=384, cap=3072, hq=28, hkv=4, d=128),
    ]


_HEADS = [(4, 2, 64), (32, 8, 64), (12, 12, 64), (28, 4, 128), (64, 8, 128), (32, 8, 128), (40, 8, 128), (16, 1, 128)]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["attn", "attn", "attn", "prefix", "step", "generate"])
    hq, hkv, d = rng.choice(_HEADS)
    kv = rng.choice(["bf16", "e4m3"])
    if kind in ("attn", "step"):
        batch = _log(rng, 1, 512)
        # the longest context: what keeps the cache within 4 GB, at most 32K
        room = int(4e9 / (batch * hkv * d * 4))
        top = _log(rng, 64, max(65, min(32768, room)))
        law = rng.choice(["uniform", "lognormal"])
        a, b, cap = (rng.randint(1, top), top, 0) if law == "uniform" else (rng.randint(1, max(1, top // 8)), max(2, top // 8), top)
        api = rng.choice(["attn", "attn", "noalloc"]) if kv == "bf16" and kind == "attn" else "attn"
        return dict(kind=kind, api=api, kv=kv, batch=batch, hq=hq, hkv=hkv, d=d, law=law, a=a, b=b, cap=cap)
    if kind == "prefix":
        samples = rng.randint(2, 24)
        return dict(kind="prefix", kv=kv, prompts=_log(rng, 1, 512 // samples), samples=samples, prompt=_log(rng, 33, 4000),
                    median=_log(rng, 16, 1024), cap=4096, hq=hq, hkv=hkv, d=d)
    slots = _log(rng, 1, 48)
    lo = rng.randint(0, 256)
    return dict(kind="generate", kv=kv, samples=slots * rng.randint(1, 3), slots=slots, prompt_lo=lo,
                prompt_hi=lo + rng.randint(0, 256), median=_log(rng, 32, 256), cap=1024, hq=hq, hkv=hkv, d=d)


def _lengths(case):
    """The sequence lengths: part of the case (the same for every seed, so that passes on other inputs do the same
    work), drawn from a generator seeded by the case's own sizes."""
    rng = np.random.default_rng([case["batch"], case["a"], case["b"], case["hq"]])
    if case["law"] == "uniform":
        return rng.integers(case["a"], case["b"] + 1, case["batch"]).astype(np.int64)
    x = np.clip(np.floor(rng.lognormal(math.log(case["b"]), 1.2 if case["hq"] == 64 else 1.0, case["batch"])), 1, case["cap"])
    return case["a"] + x.astype(np.int64)


def _prefix_lengths(case):
    rng = np.random.default_rng([case["prompts"], case["samples"], case["prompt"]])
    n = case["prompts"] * case["samples"]
    gen = np.clip(np.floor(rng.lognormal(math.log(case["median"]), 1.0, n)), 1, case["cap"]).astype(np.int64)
    return case["prompt"] + gen


def _normal(shape, gen):
    """Standard normal values rounded to bf16, made in pieces of bounded size."""
    out = torch.empty(shape, dtype=torch.bfloat16, device=DEV)
    flat = out.view(-1)
    for i in range(0, flat.numel(), 1 << 28):
        n = min(1 << 28, flat.numel() - i)
        flat[i:i + n] = torch.randn(n, generator=gen, device=DEV)
    return out


def _pool(num_pages, case, gen):
    """K or V pages: (pages, scales) with scales None for bf16, else per-(page, KV head) scales max|x| / 448."""
    x = _normal((num_pages, case["hkv"], PAGE, case["d"]), gen)
    if case["kv"] == "bf16":
        return x, None
    codes = torch.empty(x.shape, dtype=torch.uint8, device=DEV)
    scales = torch.empty(x.shape[:2], dtype=torch.float32, device=DEV)
    for i in range(0, num_pages, 1 << 14):
        f = x[i:i + (1 << 14)].float()
        s = f.abs().amax(dim=(2, 3)) / 448.0
        scales[i:i + (1 << 14)] = s
        codes[i:i + (1 << 14)] = (f / s[:, :, None, None]).clamp(-448, 448).to(torch.float8_e4m3fn).view(torch.uint8)
    return codes, scales


def _inputs(case, seed):
    """Lengths, block table (pages scattered over the pool, as after many samples came and went), q and the pools."""
    rng = np.random.default_rng(seed)
    gen = torch.Generator(device=DEV)
    gen.manual_seed(seed)
    if case["kind"] == "prefix":
        lens, shared, per = _prefix_lengths(case), case["prompt"] // PAGE, case["samples"]
    else:
        lens, shared, per = _lengths(case), 0, 1
    blocks = -(-lens // PAGE)
    own = blocks - shared
    groups = len(lens) // per
    total = groups * shared + int(own.sum())
    perm = rng.permutation(total).astype(np.int32)
    table = np.zeros((len(lens), int(blocks.max())), dtype=np.int32)
    at = 0
    for k in range(groups):
        common = perm[at:at + shared]
        at += shared
        for b in range(k * per, (k + 1) * per):
            table[b, :shared] = common
            table[b, shared:blocks[b]] = perm[at:at + own[b]]
            at += own[b]
    s = dict(case=case, scale=1.0 / math.sqrt(case["d"]),
             q=_normal((len(lens), case["hq"], case["d"]), gen),
             table=torch.from_numpy(table).to(DEV), lens=torch.from_numpy(lens.astype(np.int32)).to(DEV))
    s["k"], s["ks"] = _pool(total, case, gen)
    s["v"], s["vs"] = _pool(total, case, gen)
    if case["kind"] == "prefix":
        s["starts"] = torch.arange(0, len(lens) + 1, per, dtype=torch.int32, device=DEV)
        s["shared"] = torch.full((groups,), shared, dtype=torch.int32, device=DEV)
    if case["kind"] == "step":
        s["k_new"] = _normal((len(lens), case["hkv"], case["d"]), gen)
        s["v_new"] = _normal((len(lens), case["hkv"], case["d"]), gen)
    return s


def _generation(case, seed):
    """Prompt and output lengths (part of the case) and estimates off by a lognormal error, as a ranker's would be."""
    rng = np.random.default_rng([case["samples"], case["slots"], case["median"]])
    out = np.clip(np.floor(rng.lognormal(math.log(case["median"]), 1.0, case["samples"])), 1, case["cap"]).astype(np.int32)
    prompt = rng.integers(case["prompt_lo"], case["prompt_hi"] + 1, case["samples"]).astype(np.int32)
    est = np.maximum(1, out * rng.lognormal(0.0, 0.3, case["samples"])).astype(np.int32)
    return dict(case=case, prompt=prompt, out=out, est=est, seed=int(seed) % 100003)


def prepare(case, seed):
    return _generation(case, seed) if case["kind"] == "generate" else _inputs(case, seed)


def run(s):
    case = s["case"]
    kind, fp8 = case["kind"], case["kv"] == "e4m3"
    if kind == "generate":
        eng = engine.Engine(s["prompt"], s["out"], s["est"], batch_slots=case["slots"], num_q_heads=case["hq"],
                            num_kv_heads=case["hkv"], head_dim=case["d"], kv_fp8=fp8, seed=s["seed"])
        eng.run()
        got = dict(out=eng.out, lens=eng.seq_lens, table=eng.block_table, k=eng.k_pages, v=eng.v_pages)
        if fp8:
            got.update(ks=eng.k_scales, vs=eng.v_scales)
        eng.close()
        return got
    if kind == "prefix":
        if fp8:
            return sl.decode_attn_prefix_fp8(s["q"], s["k"], s["v"], s["ks"], s["vs"], s["table"], s["lens"], s["scale"],
                                             s["starts"], s["shared"])
        return sl.decode_attn_prefix(s["q"], s["k"], s["v"], s["table"], s["lens"], s["scale"], s["starts"], s["shared"])
    if kind == "step":
        sl.kv_append(s["k_new"], s["v_new"], s["table"], s["lens"], s["k"], s["v"], k_scales=s["ks"], v_scales=s["vs"])
    if fp8:
        out = sl.decode_attn_fp8(s["q"], s["k"], s["v"], s["ks"], s["vs"], s["table"], s["lens"], s["scale"])
    elif case.get("api") == "noalloc":
        out = sl.decode_attn_noalloc(s["q"], s["k"], s["v"], s["table"], s["lens"], s["scale"])
    else:
        out = sl.decode_attn(s["q"], s["k"], s["v"], s["table"], s["lens"], s["scale"])
    if kind == "step":
        return dict(out=out, k=s["k"], v=s["v"], **(dict(ks=s["ks"], vs=s["vs"]) if fp8 else {}))
    return out


def work(case):
    hq, hkv, d = case["hq"], case["hkv"], case["d"]
    kvb = 1 if case["kv"] == "e4m3" else 2
    page_extra = 8 * hkv if case["kv"] == "e4m3" else 0

    def attention(tokens, pages, entries, rows):
        return tokens * hkv * d * 2 * kvb + pages * page_extra + 4 * entries + rows * (hq * d * 4 + 4)

    if case["kind"] == "generate":
        g = _generation(case, 0)
        p, o = g["prompt"].astype(np.int64), g["out"].astype(np.int64)
        # every step reads each live sample's cache: lengths p + 1 .. p + o; every cached row is written once
        tokens = int((o * p + o * (o + 1) // 2).sum())
        steps = int(o.sum())
        return dict(bytes=attention(tokens, tokens // PAGE, tokens // PAGE, steps) + int((p + o).sum()) * hkv * d * 2 * kvb,
                    flops=4 * tokens * hq * d)
    if case["kind"] == "prefix":
        lens, sh = _prefix_lengths(case), case["prompt"] // PAGE
        own = lens - sh * PAGE
        blocks = -(-own // PAGE)
        return dict(bytes=attention(int(own.sum()) + case["prompts"] * sh * PAGE, int(blocks.sum()) + case["prompts"] * sh,
                                    int(blocks.sum()) + case["prompts"] * sh, len(lens)),
                    flops=4 * int(lens.sum()) * hq * d)
    lens = _lengths(case)
    pages = int((-(-lens // PAGE)).sum())
    got = dict(bytes=attention(int(lens.sum()), pages, pages, len(lens)), flops=4 * int(lens.sum()) * hq * d)
    if case["kind"] == "step":
        got["bytes"] += len(lens) * hkv * (2 * d * (2 + kvb) + (16 if kvb == 1 else 0))
    return got


def tolerance(case):
    # Outputs are bf16 (2^-9 relative rounding each) of a softmax whose weights enter the value product in bf16.
    # Codes, scales, lengths and tables are exact.
    return {"rel": 1e-2}


def _dequant(pages, scales):
    if scales is None:
        return pages.double()
    return pages.view(torch.float8_e4m3fn).double() * scales.double()[:, :, None, None]


def _encode(x):
    return x.clamp(-448.0, 448.0).to(torch.float8_e4m3fn)


def _append(pages, scales, new, table, lens):
    """The documented append rule for one of K and V, in place: the new row of every sequence; E4M3 grows the scale of
    the page-head tile and re-encodes its earlier rows (all of it in 32 bits, so that codes are exact)."""
    t = lens.long() - 1
    page = table.gather(1, (t // PAGE)[:, None])[:, 0].long()
    slot = t % PAGE
    if scales is None:
        pages[page, :, slot] = new
        return
    x = new.float()
    a = x.abs().amax(dim=2)
    old = scales[page]
    fresh = (slot == 0)[:, None]
    grown = torch.where(fresh, torch.where(a > 0, a / 448.0, torch.ones_like(a)), torch.where(a <= old * 448.0, old, a / 448.0))
    tile = pages[page]                                                     # [B, Hkv, 16, D]
    again = _encode(tile.view(torch.float8_e4m3fn).float() * old[:, :, None, None] / grown[:, :, None, None]).view(torch.uint8)
    earlier = torch.arange(PAGE, device=DEV)[None, None, :, None] < slot[:, None, None, None]
    tile = torch.where(earlier & (grown != old)[:, :, None, None] & ~fresh[:, :, None, None], again, tile)
    tile[torch.arange(len(t), device=DEV), :, slot] = _encode(x / grown[:, :, None]).view(torch.uint8)
    pages[page] = tile
    scales[page] = grown


def exact(case, seed):
    if case["kind"] == "generate":
        return None   # the prompts' synthetic values are the engine's own
    s = _inputs(case, seed)
    if case["kind"] == "step":
        _append(s["k"], s["ks"], s["k_new"], s["table"], s["lens"])
        _append(s["v"], s["vs"], s["v_new"], s["table"], s["lens"])
    hq, hkv, d = case["hq"], case["hkv"], case["d"]
    out = torch.empty((len(s["lens"]), hq, d), dtype=torch.float64, device=DEV)
    scale = float(np.float32(s["scale"]))
    for b, n in enumerate(s["lens"].tolist()):
        ids = s["table"][b, :-(-n // PAGE)].long()

        def rows(pages, scales):   # [Hkv, n, D]
            x = _dequant(pages[ids], None if scales is None else scales[ids])
            return x.permute(1, 0, 2, 3).reshape(hkv, -1, d)[:, :n].contiguous()

        q = s["q"][b].double().view(hkv, hq // hkv, d)
        w = torch.softmax(torch.matmul(q, rows(s["k"], s["ks"]).transpose(1, 2).contiguous()) * scale, dim=2)
        out[b] = torch.matmul(w, rows(s["v"], s["vs"])).view(hq, d)
    if case["kind"] == "step":
        return dict(out=out, k=s["k"] if s["ks"] is not None else s["k"].double(),
                    v=s["v"] if s["vs"] is not None else s["v"].double(),
                    **({} if s["ks"] is None else dict(ks=s["ks"].double(), vs=s["vs"].double())))
    return out
