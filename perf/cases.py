"""The calls that are timed: what a rollout engine asks of this library, layer by layer.

Every case is one attention layer's work in one engine step, through the public entry
points of paper_2607_09207_amd.DecodeAttention: decode (plain, with the KV append that
precedes it, and over GRPO groups that share their prompt), verification of drafted
tokens, and prefill (whole prompts and chunks).  Head layouts, lengths and page sizes are
those of the named workloads of paper_2607_09207_amd.inputs, from the smallest to the
largest; lengths follow the same laws (uniform, lognormal, the staleness mix).

A case fixes the multiset of lengths (`lens_seed`); the seed of a preparation fixes the
order of the sequences, the pages they occupy in the pool, and every value.
"""
import math

import numpy as np
import torch

PAGE = 16
DEV = "cuda:0"
KV_TORCH = {"f32": torch.float32, "bf16": torch.bfloat16, "fp8": torch.float8_e4m3fn}
KV_BYTES = {"f32": 4, "bf16": 2, "fp8": 1}
KV_NAME = {"f32": "f32", "bf16": "bf16", "fp8": "fp8_e4m3fn"}


def listed():
    gqa = dict(hq=28, hkv=4, d=128, kv="bf16", out="f32")
    grpo = dict(hq=12, hkv=2, d=128, kv="bf16", out="f32")
    fp8 = dict(hq=40, hkv=8, d=128, kv="fp8", out="f32")
    tail = dict(law="lognormal", median=2048, sigma=1.0, lo=32, hi=16384, max_pages=1024)
    return [
        # The smallest call: 8 short fp32 sequences.  Latency and the launch are all of it.
        dict(name="decode_tiny_f32", kind="decode", hq=4, hkv=4, d=64, kv="f32", out="f32", batch=8,
             law="uniform", lo=1, hi=256, max_pages=16, lens_seed=1000),
        # A small engine step early in the rollout: append the new token's K/V to an fp8
        # cache (page scales kept), then decode; 32 young responses.
        dict(fp8, name="step_small_fp8", kind="step", out="bf16", batch=32, law="uniform", lo=16, hi=1024,
             max_pages=2048, lens_seed=2001),
        # The end of a rollout: the four long responses that are still running.
        dict(gqa, name="decode_stragglers_bf16", kind="decode", batch=4, law="uniform", lo=8192, hi=16384,
             max_pages=1024, lens_seed=2002),
        # An ordinary decode call: 64 sequences with long-tailed lengths.
        dict(gqa, name="decode_longtail_bf16", kind="decode", batch=64, lens_seed=1001, **tail),
        # The largest decode call: 512 sequences, a fifth of them long responses carried
        # over from earlier iterations.
        dict(name="decode_staleness_mix_bf16", kind="decode", hq=64, hkv=8, d=128, kv="bf16", out="f32", batch=512,
             law="mix", lo=16, hi=32768, max_pages=2048, lens_seed=1004),
        # Long-tailed decode on an fp8 cache.
        dict(fp8, name="decode_longtail_fp8", kind="decode", batch=128, law="lognormal", median=4096, sigma=1.0,
             lo=64, hi=32768, max_pages=2048, lens_seed=1003),
        # GRPO: 32 prompts of 512 tokens, 8 responses each, sharing the prompt's pages.
        dict(grpo, name="grouped_prompt512_bf16", kind="grouped", batch=256, group=8, prompt=512, law="lognormal",
             median=1024, sigma=1.2, lo=1, hi=24576, max_pages=1568, lens_seed=1002),
        # GRPO with a long shared prompt (4096 tokens).
        dict(grpo, name="grouped_prompt4096_bf16", kind="grouped", batch=256, group=8, prompt=4096, law="lognormal",
             median=1024, sigma=1.2, lo=1, hi=24576, max_pages=1792, lens_seed=1002),
        # Speculative decoding: the last 4 tokens of every long-tail sequence verified.
        dict(gqa, name="verify4_longtail_bf16", kind="verify", rows=4, batch=64, lens_seed=1007, **tail),
        # Prefill of the 32 GRPO prompts, whole.
        dict(grpo, name="prefill_prompts_bf16", kind="prefill", chunk=512, batch=32, law="uniform", lo=512, hi=512,
             max_pages=32, lens_seed=1005),
        # Chunked prefill: the last 512 tokens of every long-tail sequence.
        dict(gqa, name="prefill_chunks_bf16", kind="prefill", chunk=512, batch=64, lens_seed=1006, **tail),
        # Chunked prefill on an fp8 cache, the largest product.
        dict(fp8, name="prefill_chunks_fp8", kind="prefill", chunk=512, batch=64, law="lognormal", median=4096,
             sigma=1.0, lo=64, hi=32768, max_pages=2048, lens_seed=1008),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more call of these ranges: any kind, dtype, head layout and size, up to about
    two thirds of the largest listed call of its kind."""
    while True:
        kind = rng.choice(["decode", "decode", "decode", "step", "grouped", "verify", "prefill", "prefill"])
        kv = rng.choice(["bf16", "bf16", "fp8"])
        if kind == "decode" and rng.random() < 0.15:
            kv = "f32"
        hq, hkv = rng.choice([(28, 4), (12, 2), (40, 8), (64, 8), (8, 1), (16, 16)])
        d = rng.choice([64, 128, 128])
        if kv == "f32":
            hq, hkv, d = rng.choice([(4, 4, 64), (8, 4, 64), (8, 8, 128), (2, 1, 64)])
        c = dict(kind=kind, hq=hq, hkv=hkv, d=d, kv=kv, out="f32" if kv == "f32" else rng.choice(["f32", "bf16"]),
                 layout=rng.choice(["head", "head", "slot"]), lens_seed=rng.randrange(1 << 30))
        law = rng.choice(["uniform", "lognormal", "mix"])
        if kind == "grouped":
            group = rng.choice([2, 4, 5, 8, 16])
            c.update(batch=group * _log_int(rng, 1, 64), group=group, prompt=PAGE * _log_int(rng, 2, 320),
                     law="lognormal", median=_log_int(rng, 64, 2048), sigma=1.0, lo=1, hi=_log_int(rng, 2048, 16384))
        else:
            c["batch"] = _log_int(rng, 1, 64 if kind == "prefill" or kv == "f32" else 512)
            hi = _log_int(rng, 33, 2048 if kv == "f32" else 32768)
            if law == "lognormal":
                c.update(law=law, median=max(16, hi // 8), sigma=1.0, lo=16, hi=hi)
            else:
                c.update(law=law, lo=rng.choice([1, 16, max(1, hi // 2)]), hi=hi)
                if law == "mix" and hi < 1024:
                    c["law"] = "uniform"
        if kind == "verify":
            c["rows"] = rng.randint(2, min(8, 64 * hkv // hq))
        if kind == "prefill":
            c["chunk"] = rng.choice([64, 200, 512, 777, 1024, 2048])
        lens = _lengths(c)
        c["max_pages"] = int(-(-max(lens) // PAGE)) + rng.choice([0, 0, 3, 64, 500])
        w = work(c)
        if w["bytes"] <= 6e9 and w["flops"] <= 2e12 and _kv_tokens(c) * hkv * d * 2 * KV_BYTES[kv] <= 6e9:
            return c


# ------------------------------------------------------------------ sizes

def _lengths(c):
    """The multiset of sequence lengths (cached tokens, prompt included), sorted by draw."""
    rng = np.random.default_rng(c["lens_seed"])
    n = c["batch"]
    if c["law"] == "uniform":
        lens = rng.integers(c["lo"], c["hi"] + 1, size=n)
    elif c["law"] == "lognormal":
        lens = np.clip(np.rint(c["median"] * np.exp(c["sigma"] * rng.standard_normal(n))), c["lo"], c["hi"])
    else:   # a fifth long, the rest short
        lens = rng.integers(16, 513, size=n)
        k = int(round(0.2 * n))
        lens[rng.choice(n, size=k, replace=False)] = rng.integers(max(1, c["hi"] // 4), c["hi"] + 1, size=k)
    return lens.astype(np.int64) + c.get("prompt", 0)


def _kv_tokens(c):
    """Distinct cached tokens: a group's prompt counts once."""
    lens = _lengths(c)
    if "prompt" not in c:
        return int(lens.sum())
    return int((lens - c["prompt"]).sum()) + len(lens) // c["group"] * c["prompt"]


def _row_counts(c, lens):
    """Query rows of each sequence."""
    most = c.get("rows", c.get("chunk", 1))
    return np.minimum(lens, most)


def work(c):
    lens, eb = _lengths(c), KV_BYTES[c["kv"]]
    rows = _row_counts(c, lens)
    n, total = _kv_tokens(c), int(rows.sum())
    qb, ob = (4 if c["kv"] == "f32" else 2), (2 if c["out"] == "bf16" else 4)
    kv = 2 * n * c["hkv"] * c["d"] * eb
    pages = -(-n // PAGE)
    scales = 8 * pages * c["hkv"] if c["kv"] == "fp8" else 0
    b = kv + scales + 4 * pages + 4 * len(lens) + total * c["hq"] * c["d"] * (qb + ob)
    if c["kind"] == "step":   # the new rows in, and into the cache
        b += 2 * len(lens) * c["hkv"] * c["d"] * (2 + eb)
    # Row i of a sequence sees L - n + i + 1 keys; 2 products of d multiply-adds each.
    seen = rows * lens - rows * (rows - 1) // 2
    return {"bytes": float(b), "flops": 4.0 * c["d"] * c["hq"] * float(seen.sum())}


# ------------------------------------------------------------------ inputs

def _pool(c, gen, npages):
    """One cache (K or V) of N(0, 1) values: [pages][Hkv][16][d], and its fp8 scales
    (the tile's largest magnitude at 448)."""
    shape = (npages, c["hkv"], PAGE, c["d"])
    pool = torch.empty(shape, dtype=KV_TORCH[c["kv"]], device=DEV)
    scale = torch.empty(shape[:2], dtype=torch.float32, device=DEV) if c["kv"] == "fp8" else None
    step = max(1, (1 << 28) // (c["hkv"] * PAGE * c["d"]))
    for i in range(0, npages, step):
        part = (min(step, npages - i),) + shape[1:]
        if c["kv"] == "fp8":
            x = torch.randn(part, dtype=torch.float32, device=DEV, generator=gen)
            s = x.abs().amax(dim=(2, 3)) / 448.0
            scale[i:i + step] = s
            pool[i:i + step] = (x / s[:, :, None, None]).to(pool.dtype)
        else:
            pool[i:i + step] = torch.randn(part, dtype=pool.dtype, device=DEV, generator=gen)
    if c.get("layout") == "slot":   # the same values, stored [pages][16][Hkv][d]
        pool = pool.transpose(1, 2).contiguous().transpose(1, 2)
    return pool, scale


def _inputs(c, seed):
    """Tensors of one call, from the case and the seed alone."""
    rng = np.random.default_rng([seed, 17])
    gen = torch.Generator(device=DEV).manual_seed(seed)
    lens = rng.permutation(_lengths(c))
    used = -(-lens // PAGE)
    B, mp = c["batch"], c["max_pages"]
    table = np.zeros((B, mp), np.int32)
    if "prompt" in c:
        pp, gs = c["prompt"] // PAGE, c["group"]
        perm = rng.permutation(int((used - pp).sum()) + B // gs * pp).astype(np.int32)
        at = B // gs * pp
        for b in range(B):
            own = int(used[b]) - pp
            table[b, :pp] = perm[b // gs * pp:(b // gs + 1) * pp]
            table[b, pp:pp + own] = perm[at:at + own]
            at += own
    else:
        perm = rng.permutation(int(used.sum())).astype(np.int32)
        at = 0
        for b in range(B):
            table[b, :used[b]] = perm[at:at + used[b]]
            at += int(used[b])
    rows = _row_counts(c, lens)
    total = int(rows.sum())
    qd = torch.float32 if c["kv"] == "f32" else torch.bfloat16
    t = {"lens": lens, "rows": rows, "table": table}
    t["q"] = torch.randn((total, c["hq"], c["d"]), dtype=qd, device=DEV, generator=gen)
    t["k"], t["ks"] = _pool(c, gen, len(perm))
    t["v"], t["vs"] = _pool(c, gen, len(perm))
    t["block_table"] = torch.from_numpy(table).to(DEV)
    t["seq_lens"] = torch.from_numpy(lens.astype(np.int32)).to(DEV)
    if c["kind"] in ("verify", "prefill"):
        t["q_start"] = torch.from_numpy(np.concatenate([[0], np.cumsum(rows)]).astype(np.int32)).to(DEV)
    if c["kind"] == "grouped":
        t["prefix_pages"] = torch.full((B // c["group"],), c["prompt"] // PAGE, dtype=torch.int32, device=DEV)
    if c["kind"] == "step":
        t["k_new"] = torch.randn((B, c["hkv"], c["d"]), dtype=qd, device=DEV, generator=gen)
        t["v_new"] = torch.randn((B, c["hkv"], c["d"]), dtype=qd, device=DEV, generator=gen)
    return t


def prepare(c, seed):
    """The layer's handle, its workspace and output, and the call's inputs."""
    from paper_2607_09207_amd import DecodeAttention
    s = _inputs(c, seed)
    s["case"] = c
    s["layer"] = DecodeAttention(c["hq"], c["hkv"], c["d"], c["batch"], c["max_pages"],
                                 "f32" if c["kv"] == "f32" else "bf16", KV_NAME[c["kv"]], c["out"],
                                 kv_strides=s["k"].stride()[:3])
    s["layer"].workspace(s["q"].device, grouped=c["kind"] == "grouped")
    s["o"] = torch.empty(s["q"].shape, dtype=torch.bfloat16 if c["out"] == "bf16" else torch.float32, device=DEV)
    return s


def run(s):
    c, layer = s["case"], s["layer"]
    cache = (s["k"], s["v"], s["block_table"], s["seq_lens"])
    if c["kind"] in ("verify", "prefill"):
        return layer.multi(s["q"], *cache, s["q_start"], k_scale=s["ks"], v_scale=s["vs"], out=s["o"],
                           max_q_len=c.get("rows", 0))
    if c["kind"] == "grouped":
        return layer(s["q"], *cache, k_scale=s["ks"], v_scale=s["vs"], out=s["o"], group_size=c["group"],
                     prefix_pages=s["prefix_pages"], prompt_pages_hint=c["prompt"] // PAGE)
    if c["kind"] == "step":
        layer.append(s["k_new"], s["v_new"], *cache, k_scale=s["ks"], v_scale=s["vs"])
        layer(s["q"], *cache, k_scale=s["ks"], v_scale=s["vs"], out=s["o"])
        return {"out": s["o"], "k": s["k"], "v": s["v"], "ks": s["ks"], "vs": s["vs"]}
    return layer(s["q"], *cache, k_scale=s["ks"], v_scale=s["vs"], out=s["o"])


# ------------------------------------------------------------------ what the results should be

def _take(cache, pages):
    """Pages of a cache (fp8 moves as bytes)."""
    return cache.view(torch.uint8)[pages].view(cache.dtype) if cache.element_size() == 1 else cache[pages]


def _put(cache, pages, tiles):
    if cache.element_size() == 1:
        cache.view(torch.uint8)[pages] = tiles.view(torch.uint8)
    else:
        cache[pages] = tiles


def _append(c, t, cache, scale, new):
    """The append in plain torch, in place: bf16 rows as given; an fp8 page's scale grows
    to cover the new row (earlier rows re-encoded), a page's first row sets it."""
    last = torch.from_numpy(t["lens"] - 1).to(DEV)
    page = t["block_table"].long().gather(1, (last // PAGE)[:, None])[:, 0]
    slot = last % PAGE
    tile, x = _take(cache, page).float(), new.float()     # [B][Hkv][16][d], [B][Hkv][d]
    if scale is None:
        tile.scatter_(2, slot[:, None, None, None].expand(-1, c["hkv"], 1, c["d"]), x[:, :, None])
        _put(cache, page, tile.to(cache.dtype))
        return
    amax, old = x.abs().amax(dim=2), scale[page]
    grow = (slot == 0)[:, None] | (amax > 448.0 * old)
    s = torch.where(grow, amax / 448.0, old)
    ratio = torch.where(grow, old / s, torch.ones_like(s))
    tile = (tile * ratio[:, :, None, None]).clamp(-448, 448).to(cache.dtype)
    row = (x / s[:, :, None]).clamp(-448, 448).to(cache.dtype)
    before = torch.arange(PAGE, device=DEV)[None, :] < slot[:, None]
    keep = torch.where((before[:, None, :, None] & grow[:, :, None, None]), tile.float(), _take(cache, page).float())
    keep.scatter_(2, slot[:, None, None, None].expand(-1, c["hkv"], 1, c["d"]), row.float()[:, :, None])
    _put(cache, page, keep.to(cache.dtype))
    scale[page] = s


def exact(c, seed):
    """The same call in float64, one sequence and KV head at a time, on the GPU."""
    t = _inputs(c, seed)
    if c["kind"] == "step":
        _append(c, t, t["k"], t["ks"], t["k_new"])
        _append(c, t, t["v"], t["vs"], t["v_new"])
    G, d = c["hq"] // c["hkv"], c["d"]
    out = torch.empty(t["q"].shape, dtype=torch.float64, device=DEV)
    at = 0
    for b in range(c["batch"]):
        L, n = int(t["lens"][b]), int(t["rows"][b])
        # float64 is 8 bytes a value: long chunks go a KV head and 512 rows at a time.
        heads = range(0, c["hkv"], c["hkv"] if n == 1 else 1)
        pages = torch.from_numpy(t["table"][b, :-(-L // PAGE)].astype(np.int64)).to(DEV)
        for g in heads:
            g1 = g + (c["hkv"] if n == 1 else 1)
            k, v = (_take(x, pages)[:, g:g1].double() for x in (t["k"], t["v"]))
            if t["ks"] is not None:
                k = k * t["ks"][pages, g:g1].double()[:, :, None, None]
                v = v * t["vs"][pages, g:g1].double()[:, :, None, None]
            k = k.permute(1, 3, 0, 2).reshape(g1 - g, d, -1)[:, :, :L].contiguous()     # [heads][d][L]
            v = v.permute(1, 0, 2, 3).reshape(g1 - g, -1, d)[:, :L].contiguous()        # [heads][L][d]
            for r in range(0, n, 512):
                m = min(512, n - r)
                q = t["q"][at + r:at + r + m, g * G:g1 * G].double()                     # [m][heads * G][d]
                q = q.reshape(m, g1 - g, G, d).permute(1, 0, 2, 3).reshape(g1 - g, m * G, d).contiguous()
                s = torch.matmul(q, k) / math.sqrt(d)
                if n > 1:
                    limit = L - n + r + torch.arange(m, device=DEV).repeat_interleave(G)
                    s.masked_fill_(torch.arange(L, device=DEV)[None, :] > limit[:, None], -math.inf)
                o = torch.matmul(torch.softmax(s, dim=-1), v)
                out[at + r:at + r + m, g * G:g1 * G] = o.reshape(g1 - g, m, G, d).permute(1, 0, 2, 3).reshape(m, -1, d)
        at += n
    if c["kind"] == "step":
        scale = lambda x: None if x is None else x.double()
        return {"out": out, "k": t["k"].double(), "v": t["v"].double(), "ks": scale(t["ks"]), "vs": scale(t["vs"])}
    return out


def tolerance(c):
    """About four times the error against float64 that was measured (2-norms): 1.5e-7
    for fp32; 1.1e-3 to 1.7e-3 where the probabilities are rounded to bf16 for the
    matrix products (fp8 caches as well: their values are bf16 values); 2.4e-3 with the
    output rounded to bf16 too."""
    if c["kv"] == "f32":
        return {"rel": 1e-6}
    return {"rel": 1e-2 if c["out"] == "bf16" else 7e-3}
