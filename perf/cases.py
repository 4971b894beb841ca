"""The calls a user of this library makes, with their inputs, work and 64-bit results.

A rollout instance runs, per GPU:
  decode    one step of batched decode attention over the paged bf16 cache, through
            DecodeAttention (plan, attention and merge in one call) or, where nothing may
            be allocated, through sf_decode_attn_scratch on a plan already on the device;
  fp8       the same step over an fp8 (E4M3) cache with per-(page, KV head) scales;
  append    the step of a growing cache: every sequence's newest token joins the
            attention and is stored into the pools;
  quantize  pages of the bf16 pools become fp8 codes and scales;
  extend    re-prefill: causal attention of new tokens over their cached prefix, with
            the new tokens' keys and values stored first.
Head layouts and length distributions are those of the workloads in
paper_2601_12784_amd/workloads.py (skewed trajectory lengths), from a single short
prompt to the full long-tail batch. Every tensor is drawn on the GPU from the seed;
lengths follow from the case alone.
"""
import math

import numpy as np
import torch

from paper_2601_12784_amd import binding as B

PAGE = 16
DEV = "cuda"
HEADS = {"4/1x64": (4, 1, 64), "14/2x64": (14, 2, 64), "8/8x64": (8, 8, 64), "28/4x128": (28, 4, 128),
         "32/8x128": (32, 8, 128), "40/8x128": (40, 8, 128), "16/1x128": (16, 1, 128)}


def listed():
    return [
        # four short sequences of a small model: latency of one call, and nothing else
        dict(name="decode_tiny", kind="decode", via="runner", heads="4/1x64", lens="tiny", batch=4, a=0, b=0,
             k_mult=1.0, lens_seed=1000),
        # the last trajectory of a rollout still running: one long sequence
        dict(name="decode_last", kind="decode", via="runner", heads="28/4x128", lens="uniform", batch=1, a=32768,
             b=32768, k_mult=1.0, lens_seed=1004),
        # an ordinary batch of a 7B-like model, 512 to 4096 cached tokens each
        dict(name="decode_7b", kind="decode", via="runner", heads="28/4x128", lens="uniform", batch=64, a=512,
             b=4096, k_mult=1.0, lens_seed=1001),
        # the long-tail batch: 256 trajectories, median 2048, up to 16384 tokens
        dict(name="decode_longtail", kind="decode", via="runner", heads="28/4x128", lens="lognormal", batch=256,
             a=2048, b=16384, k_mult=1.0, lens_seed=1002),
        # a 32B-like model's batch with sharper attention (keys times 3), up to 32768 tokens
        dict(name="decode_32b", kind="decode", via="runner", heads="40/8x128", lens="lognormal", batch=128, a=4096,
             b=32768, k_mult=3.0, lens_seed=1003),
        # the long-tail batch over an fp8 cache
        dict(name="fp8_longtail", kind="fp8", heads="28/4x128", lens="lognormal", batch=256, a=2048, b=16384,
             k_mult=1.0, lens_seed=1002),
        # one step of a growing cache: 502 short trajectories and 10 of 32768 tokens
        dict(name="append_straggler", kind="append", heads="28/4x128", lens="straggler", batch=512, a=2048, b=32768,
             k_mult=1.0, lens_seed=1004),
        # a whole bf16 cache quantized (the long-tail batch's pages)
        dict(name="quantize_cache", kind="quantize", heads="28/4x128", pages=44152, partial=256, k_mult=1.0),
        # the pages that one decode step of 512 trajectories has filled
        dict(name="quantize_step", kind="quantize", heads="28/4x128", pages=32, partial=0, k_mult=1.0),
        # resumed trajectories recomputed whole: 32 of the long-tail lengths, every token new
        dict(name="extend_reprefill", kind="extend", heads="28/4x128", lens="lognormal", batch=32, a=2048, b=16384,
             new=0, k_mult=1.0, lens_seed=1005),
        # four trajectories go on with 256 new tokens each over a cached prefix of about 8000
        dict(name="extend_resume", kind="extend", heads="28/4x128", lens="uniform", batch=4, a=7936, b=8448, new=256,
             k_mult=1.0, lens_seed=1006),
        # one prompt
        dict(name="extend_prompt", kind="extend", heads="28/4x128", lens="uniform", batch=1, a=1000, b=1000, new=0,
             k_mult=1.0, lens_seed=1007),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["decode", "decode", "decode", "fp8", "append", "quantize", "extend", "extend", "extend"])
    c = dict(kind=kind, heads=rng.choice(sorted(HEADS) + ["28/4x128", "40/8x128"]))
    if kind == "quantize":
        c["pages"] = _log_int(rng, 1, 40000)
        c["partial"] = rng.randint(0, min(c["pages"], 256))
        c["k_mult"] = 1.0
        return c
    if kind == "extend":
        c["batch"] = _log_int(rng, 1, 32)
        c["lens"] = rng.choice(["uniform", "lognormal"])
        median = _log_int(rng, 16, 16384)
        c["a"], c["b"] = (median, min(16384, 8 * median)) if c["lens"] == "lognormal" else (median // 2 + 1, median)
        c["new"] = rng.choice([0, _log_int(rng, 1, 4096)])
    else:
        if kind == "decode":
            c["via"] = rng.choice(["runner", "runner", "runner", "scratch"])
        c["batch"] = _log_int(rng, 1, 512)
        c["lens"] = rng.choice(["uniform", "lognormal"])
        median = _log_int(rng, 16, 32768)
        c["a"], c["b"] = (median, min(32768, 16 * median)) if c["lens"] == "lognormal" else (median // 4 + 1, median)
    c["k_mult"] = rng.choice([1.0, 1.0, 3.0])
    c["lens_seed"] = rng.randint(0, 1 << 30)
    while work(c)["bytes"] > 1.7e9 or work(c)["flops"] > 3.5e12:
        c["batch"] = max(1, c["batch"] * 2 // 3)
        c["a"], c["b"] = max(1, c["a"] * 9 // 10), max(1, c["b"] * 9 // 10)
    return c


# --------------------------------------------------------------------------
# lengths and pages
# --------------------------------------------------------------------------
def _lengths(c):
    """Cached tokens per sequence, from the case alone (int32)."""
    rng = np.random.default_rng(c["lens_seed"])
    n = c["batch"]
    if c["lens"] == "tiny":
        x = np.array([17, 64, 130, 300])
    elif c["lens"] == "uniform":
        x = rng.integers(c["a"], c["b"], size=n, endpoint=True)
    elif c["lens"] == "lognormal":
        x = np.clip(np.rint(np.exp(math.log(c["a"]) + rng.standard_normal(n))), max(1, c["a"] // 8), c["b"])
    else:   # straggler: ten of b tokens, the others up to a
        x = np.concatenate([rng.integers(1, c["a"], size=n - 10, endpoint=True), np.full(10, c["b"])])[rng.permutation(n)]
    return x.astype(np.int32)


def _new_lengths(c, lens):
    """New tokens per sequence of an extend pass (int32): all of them, or up to `new`."""
    return lens.copy() if c["new"] == 0 else np.minimum(lens, c["new"]).astype(np.int32)


def _tables(lens, rng):
    """A random scatter of the sequences' pages over a pool that just holds them."""
    pages = (lens.astype(np.int64) + PAGE - 1) // PAGE
    perm = rng.permutation(int(pages.sum()))
    bt = np.full((lens.size, int(pages.max())), -1, dtype=np.int32)
    bt[np.arange(bt.shape[1])[None, :] < pages[:, None]] = perm
    return bt, int(pages.sum())


def _normal(g, shape, mult=1.0):
    x = torch.randn(shape, generator=g, device=DEV, dtype=torch.bfloat16)
    return x.mul_(mult) if mult != 1.0 else x


def _pools(g, n, hkv, d, k_mult):
    return _normal(g, (n, hkv, d // 8, PAGE, 8), k_mult), _normal(g, (n, hkv, d, PAGE))


def _codes(g, shape):
    """E4M3 codes of normal values quantized with their largest magnitude near 448."""
    x = torch.randn(shape, generator=g, device=DEV, dtype=torch.bfloat16).mul_(100.0).clamp_(-448.0, 448.0)
    return x.to(torch.float8_e4m3fn).view(torch.uint8)


# --------------------------------------------------------------------------
# prepare and run
# --------------------------------------------------------------------------
def prepare(c, seed):
    hq, hkv, d = HEADS[c["heads"]]
    rng = np.random.default_rng(seed)
    g = torch.Generator(device=DEV)
    g.manual_seed(int(seed))
    s = dict(c=c, scale=1.0 / math.sqrt(d))
    if c["kind"] == "quantize":
        # pages scattered over a pool twice as large as the list, `partial` of them partly filled
        n = c["pages"]
        pool = n + max(1, min(n, 64))
        s["kp"], s["vp"] = _pools(g, pool, hkv, d, c["k_mult"])
        valid = np.full(n, PAGE, dtype=np.int32)
        at = rng.permutation(n)[: c["partial"]]
        valid[at] = rng.integers(1, PAGE, size=at.size)
        s["pages"] = torch.from_numpy(rng.permutation(pool)[:n].astype(np.int32)).to(DEV)
        s["valid"] = torch.from_numpy(valid).to(DEV)
        s["k8"] = torch.zeros((pool, hkv, PAGE * d), dtype=torch.uint8, device=DEV)
        s["v8"] = torch.zeros_like(s["k8"])
        s["ks"] = torch.zeros((pool, hkv), dtype=torch.float32, device=DEV)
        s["vs"] = torch.zeros_like(s["ks"])
        s["desc"] = B.make_desc(1, hq, hkv, d, 1, pool, 1.0)
        return s

    lens = _lengths(c)
    bt, n = _tables(lens, rng)
    s["lens"] = lens
    if c["kind"] == "fp8":
        s["kp"], s["vp"] = _codes(g, (n, hkv, PAGE * d)), _codes(g, (n, hkv, PAGE * d))
        s["ks"] = torch.rand((n, hkv), generator=g, device=DEV).mul_(0.004).add_(0.008).mul_(c["k_mult"])
        s["vs"] = torch.rand((n, hkv), generator=g, device=DEV).mul_(0.004).add_(0.008)
    else:
        s["kp"], s["vp"] = _pools(g, n, hkv, d, c["k_mult"])
    if c["kind"] == "extend":
        s["new"] = _new_lengths(c, lens)
        rows = int(s["new"].sum())
        s["kn"], s["vn"] = _normal(g, (rows, hkv, d), c["k_mult"]), _normal(g, (rows, hkv, d))
        s["call"] = B.ExtendAttention(hq, hkv, d)
    else:
        rows = lens.size
        if c["kind"] == "append":
            # the newest token's page is new in this step where the token opens one
            opens = (lens - 1) % PAGE == 0
            at = (lens - 1) // PAGE
            s["fresh"] = np.where(opens, bt[np.arange(lens.size), at], -1).astype(np.int32)
            bt[np.nonzero(opens)[0], at[opens]] = -1
            s["kn"], s["vn"] = _normal(g, (rows, hkv, d), c["k_mult"]), _normal(g, (rows, hkv, d))
        if c.get("via") == "scratch":
            s["desc"] = B.make_desc(rows, hq, hkv, d, bt.shape[1], n, s["scale"])
            s["info"], work_list = B.sf_decode_attn_plan(s["desc"], lens)
            s["work"] = torch.from_numpy(work_list).to(DEV)
        else:
            s["call"] = B.DecodeAttention(hq, hkv, d)
            s["call"].reserve(lens, n, bt.shape[1], fp8=c["kind"] == "fp8")
    s["bt"] = torch.from_numpy(bt).to(DEV)
    s["q"] = _normal(g, (rows, hq, d))
    s["out"] = torch.empty((rows, hq, d), dtype=torch.float32, device=DEV)
    s["lse"] = torch.empty((rows, hq), dtype=torch.float32, device=DEV)
    return s


def run(s):
    kind = s["c"]["kind"]
    if kind == "quantize":
        B.sf_kv_quantize_fp8(s["desc"], s["kp"], s["vp"], s["pages"], s["valid"], s["k8"], s["v8"], s["ks"], s["vs"])
        return dict(k8=s["k8"], v8=s["v8"], ks=s["ks"], vs=s["vs"])
    if kind == "extend":
        out = s["call"](s["q"], s["kp"], s["vp"], s["bt"], s["lens"], s["new"], s["scale"], out=s["out"], lse=s["lse"],
                        k_new=s["kn"], v_new=s["vn"])
        return dict(out=out, lse=s["lse"], kp=s["kp"], vp=s["vp"])
    if s["c"].get("via") == "scratch":
        B.sf_decode_attn_scratch(s["desc"], s["info"], s["work"], s["q"], s["kp"], s["vp"], s["bt"], s["out"], s["lse"])
        return dict(out=s["out"], lse=s["lse"])
    append = (s["kn"], s["vn"], s["fresh"]) if kind == "append" else None
    fp8 = (s["ks"], s["vs"]) if kind == "fp8" else None
    out = s["call"](s["q"], s["kp"], s["vp"], s["bt"], s["lens"], s["scale"], out=s["out"], lse=s["lse"],
                    append=append, fp8=fp8)
    if kind == "append":
        return dict(out=out, lse=s["lse"], kp=s["kp"], vp=s["vp"], bt=s["bt"])
    return dict(out=out, lse=s["lse"])


# --------------------------------------------------------------------------
# work, tolerance and the 64-bit result
# --------------------------------------------------------------------------
def work(c):
    hq, hkv, d = HEADS[c["heads"]]
    if c["kind"] == "quantize":
        tiles = 2 * c["pages"] * hkv
        # bf16 values in, codes and one scale per tile out
        return {"bytes": tiles * (PAGE * d * 3 + 4) + 8 * c["pages"], "flops": 2 * tiles * PAGE * d}
    lens = _lengths(c).astype(np.int64)
    kv = int(lens.sum()) * hkv * d * 2
    if c["kind"] == "extend":
        new = _new_lengths(c, lens)
        rows, old = int(new.sum()), lens - new
        # the cached prefix once, the new keys and values in and stored, queries in, results out
        data = (int(old.sum()) + 2 * rows) * hkv * d * 4 + rows * hq * (6 * d + 4)
        pairs = int((new * (old + 1) + new * (new - 1) // 2).sum())
        return {"bytes": data, "flops": pairs * hq * 4 * d}
    element = 1 if c["kind"] == "fp8" else 2
    data = kv * element + lens.size * hq * (6 * d + 4)
    if c["kind"] == "fp8":
        data += int(((lens + PAGE - 1) // PAGE).sum()) * hkv * 8
    if c["kind"] == "append":
        data += lens.size * hkv * d * 4
    return {"bytes": data, "flops": 2 * kv * (hq // hkv) * 2}


def tolerance(c):
    if c["kind"] == "quantize":
        return "exact"
    if c["kind"] == "extend":
        return {"rel": 8e-4}    # weights rounded to fp16, fp32 sums: 1.4e-4 to 2.1e-4 off 64 bits
    return {"rel": 1e-5}        # weights of about 16 bits, fp32 sums: 0.7e-6 to 2.6e-6 off 64 bits


def _widen(s, pages):
    """The keys and values of a sequence's pages in 64 bits, each [Hkv, tokens, D]."""
    hq, hkv, d = HEADS[s["c"]["heads"]]
    k, v, n = s["kp"][pages], s["vp"][pages], pages.numel()
    if s["c"]["kind"] == "fp8":
        k = k.view(torch.float8_e4m3fn).double() * s["ks"][pages].double()[:, :, None]
        v = v.view(torch.float8_e4m3fn).double() * s["vs"][pages].double()[:, :, None]
        # K byte ((d/64*4 + (d%32)/8)*16 + t)*16 + (d/32%2)*8 + d%8, V byte ((d/64*4 + t/4)*16 + d%16)*16 + (d/16%4)*4 + t%4
        k = k.view(n, hkv, d // 64, 4, PAGE, 2, 8).permute(1, 0, 4, 2, 5, 3, 6)
        v = v.view(n, hkv, d // 64, 4, 16, 4, 4).permute(1, 0, 3, 6, 2, 5, 4)
    else:
        k = k.double().permute(1, 0, 3, 2, 4)
        v = v.double().permute(1, 0, 3, 2)
    return k.reshape(hkv, n * PAGE, d).contiguous(), v.reshape(hkv, n * PAGE, d).contiguous()


def exact(c, seed):
    s = prepare(c, seed)
    hq, hkv, d = HEADS[c["heads"]]
    if c["kind"] == "quantize":
        slot = torch.arange(PAGE, device=DEV)
        ks, vs = torch.zeros_like(s["ks"], dtype=torch.float64), torch.zeros_like(s["vs"], dtype=torch.float64)
        for at in range(0, c["pages"], 4096):
            pages = s["pages"][at:at + 4096].long()
            ok = (slot[None, :] < s["valid"][at:at + 4096, None])
            for pool, to, shape in ((s["kp"], ks, (-1, 1, 1, PAGE, 1)), (s["vp"], vs, (-1, 1, 1, PAGE))):
                top = pool[pages].double().abs().mul_(ok.view(shape)).flatten(2).amax(2)
                to[pages] = torch.where(top > 0, top / 448.0, torch.ones_like(top))
        return dict(k8=None, v8=None, ks=ks, vs=vs)

    lens, table = s["lens"], s["bt"].cpu().numpy().copy()
    if c["kind"] == "append":
        table[np.arange(lens.size), (lens - 1) // PAGE] = np.where(s["fresh"] >= 0, s["fresh"], table[np.arange(lens.size), (lens - 1) // PAGE])
    new = s["new"] if c["kind"] == "extend" else np.ones_like(lens)
    out = torch.zeros((int(new.sum()), hq, d), dtype=torch.float64, device=DEV)
    lse = torch.zeros((int(new.sum()), hq), dtype=torch.float64, device=DEV)
    row = 0
    for i, (n, e) in enumerate(zip(lens.tolist(), new.tolist())):
        pages = torch.from_numpy(table[i, : -(-n // PAGE)].astype(np.int64)).to(DEV)
        k, v = _widen(s, pages)
        k, v = k[:, :n].contiguous(), v[:, :n].contiguous()
        if c["kind"] in ("append", "extend"):
            k[:, n - e:], v[:, n - e:] = s["kn"][row:row + e].double().transpose(0, 1), s["vn"][row:row + e].double().transpose(0, 1)
        for at in range(0, e, 1024):
            m = min(1024, e - at)
            q = s["q"][row + at:row + at + m].double().view(m, hkv, hq // hkv, d)
            last = n - e + at + torch.arange(m, device=DEV)          # the last key each new token sees
            keys = n - e + at + m
            for h in range(hkv):
                z = (q[:, h].reshape(-1, d) @ k[h, :keys].t().contiguous()).mul_(s["scale"]).view(m, hq // hkv, keys)
                if c["kind"] == "extend":
                    z.masked_fill_((torch.arange(keys, device=DEV)[None, :] > last[:, None])[:, None, :], -math.inf)
                top = z.amax(2, keepdim=True)
                p = z.sub_(top).exp_()
                total = p.sum(2, keepdim=True)
                heads = slice(h * (hq // hkv), (h + 1) * (hq // hkv))
                out[row + at:row + at + m, heads] = (p.view(-1, keys) @ v[h, :keys]).view(m, -1, d) / total
                lse[row + at:row + at + m, heads] = (top + total.log())[:, :, 0]
        row += e
    r = dict(out=out, lse=lse)
    if c["kind"] in ("append", "extend"):
        r.update(kp=None, vp=None)
    if c["kind"] == "append":
        r.update(bt=None)
    return r
