"""The work whose speed this repository answers for: its public entry points at
the sizes a program meets, from one short prompt to a 9 GB cache.

Kinds of case (one pass each):
  prefill  quantize K and V into the paged cache, then attend (Algorithm 1)
  first    a layer's first prompt: head priorities, quantization, the start of
           the int8 buffer, attention with the row statistics
  blocks   the prefill at another (B_r, B_c) pair of Table 3
  project  the QKV projection with its quantization; with "attend" also the
           prefill on its codes
  decode   one decoding step: append the new key and value, then attend the
           cache and the buffer (without "tail": attend full groups only)
  softmax  Algorithm 3 on the rows of a score matrix

Inputs follow paper_2412_08585_amd/workloads.py: N(0, 1) activations with four
key channels per (sequence, KV head) scaled by 10, shuffled page tables, half
of the KV heads at 2 bits for "mixed".
"""
import math
import random

import torch

import paper_2412_08585_amd as ta

D = 128      # head dimension
GROUP = 64   # tokens of a cache group
QMAX = 119.0
POLY = (-0.1025, 0.4626, -0.9922, 0.9996)
TABLE3 = ((32, 32), (32, 64), (64, 32), (64, 64), (64, 128), (128, 64), (128, 128))
HEADS = ((4, 4), (16, 16), (32, 16), (40, 10), (32, 8), (64, 8), (32, 2))
MAX_BYTES = 9.0e9           # traffic of a drawn case, at most
MAX_PREFILL = 32 * 16384.0 ** 2  # B * Hq * N^2 of a drawn case, at most


def listed():
    return [
        # a short prompt of a small model: launches and latency
        dict(name="prefill-512", kind="prefill", B=1, Hq=4, Hkv=4, N=512, bits="int4", causal=True),
        # the first prompts of a Phi-3-medium layer, of no round length
        dict(name="first-1001", kind="first", B=2, Hq=40, Hkv=10, N=1001, bits="mixed", causal=True),
        # the benchmark's Phi-3-medium prefill and the long Llama-3-8B one
        dict(name="prefill-4k", kind="prefill", B=4, Hq=40, Hkv=10, N=4096, bits="int4", causal=True),
        dict(name="prefill-16k", kind="prefill", B=1, Hq=32, Hkv=8, N=16384, bits="int4", causal=True),
        # Table 3's largest tiles, as in its block-size comparison
        dict(name="blocks-128x128", kind="blocks", B=1, Hq=40, Hkv=10, N=3000, br=128, bc=128,
             causal=True),
        # the fused projection of the benchmark's prefill
        dict(name="project-4k", kind="project", B=4, Hq=40, Hkv=10, N=4096, D=5120, bits="int4",
             attend=False),
        # a single mid-sized prompt through the fused path: projection, then attention
        dict(name="project-777", kind="project", B=1, Hq=32, Hkv=8, N=777, D=4096, bits="int4",
             attend=True),
        # one conversation's decoding step: nothing but latency
        dict(name="decode-1x4k", kind="decode", B=1, Hq=32, Hkv=8, N=4000, bits="int4", tail=True,
             ragged=False, split=0),
        # the benchmark's Phi-3-medium decode
        dict(name="decode-64x8k", kind="decode", B=64, Hq=40, Hkv=10, N=8192, bits="mixed",
             tail=False, ragged=False, split=0),
        # a serving batch with eight query heads per KV head and lengths of every size
        dict(name="decode-ragged", kind="decode", B=32, Hq=64, Hkv=8, N=16383, bits="mixed",
             tail=True, ragged=True, split=0),
        # long-context batched decode: a 9 GB cache
        dict(name="decode-256x32k", kind="decode", B=256, Hq=32, Hkv=8, N=32720, bits="int4",
             tail=True, ragged=False, split=0),
        # the score rows of one ragged prompt
        dict(name="softmax-1001", kind="softmax", rows=40 * 1001, cols=1001),
    ]


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    kind = rng.choice(("prefill", "first", "blocks", "project", "decode", "decode", "decode",
                       "softmax"))
    if kind == "softmax":
        cols = _log_int(rng, 33, 16384)
        if rng.random() < 0.5:
            cols = (cols + 3) // 4 * 4
        return dict(kind=kind, rows=_log_int(rng, 64, max(64, min(163840, int(6.7e8) // cols))),
                    cols=cols)
    Hq, Hkv = rng.choice(HEADS)
    bits = rng.choice(("int4", "mixed"))
    if kind == "decode":
        while True:
            c = dict(kind=kind, B=_log_int(rng, 1, 256), Hq=Hq, Hkv=Hkv,
                     N=_log_int(rng, 64, 32768), bits=bits, tail=rng.random() < 0.75,
                     ragged=rng.random() < 0.5, split=rng.choice((0, 0, -1)))
            if not c["tail"]:
                c["N"] = c["N"] // GROUP * GROUP
            if work(c)["bytes"] <= MAX_BYTES:
                return c
    while True:
        c = dict(kind=kind, B=_log_int(rng, 1, 8), Hq=Hq, Hkv=Hkv,
                 N=_log_int(rng, 64, 4096 if kind != "prefill" else 16384), bits=bits)
        if c["B"] * Hq * float(c["N"]) ** 2 <= MAX_PREFILL:
            break
    if kind == "project":
        c.update(B=min(c["B"], 4), D=64 * _log_int(rng, 8, 80), attend=rng.random() < 0.5)
    else:
        c["causal"] = rng.random() < 0.8
    if kind == "blocks":
        c.pop("bits")
        c["br"], c["bc"] = rng.choice(TABLE3)
    return c


# ---- inputs ------------------------------------------------------------------
def _gen(*key):
    s = 0x5EED
    for k in key:
        s = (s * 1000003 + int(k) + 1) % (2 ** 62)
    return torch.Generator(device="cuda").manual_seed(s)


def _kv(B, Hkv, N, *key):
    """fp16 K, V [B][Hkv][N][128], four channels of every key head scaled by 10."""
    g = _gen(*key)
    k = torch.randn(B, Hkv, N, D, generator=g, device="cuda", dtype=torch.float16)
    v = torch.randn(B, Hkv, N, D, generator=g, device="cuda", dtype=torch.float16)
    gain = torch.ones(B, Hkv, 1, D, device="cuda", dtype=torch.float16)
    ch = torch.rand(B, Hkv, 1, D, generator=g, device="cuda").argsort(dim=-1)[..., :4]
    return k * gain.scatter_(-1, ch, 10.0), v


def _randn(shape, *key):
    return torch.randn(*shape, generator=_gen(*key), device="cuda", dtype=torch.float16)


def _head_bits(c):
    bits = [4] * c["Hkv"]
    if c["bits"] == "mixed":
        for h in random.Random(c["Hkv"]).sample(range(c["Hkv"]), c["Hkv"] // 2):
            bits[h] = 2
    return bits


def _lengths(c):
    """Cached tokens of each sequence before the step: N, or spread up to N."""
    if not c["ragged"]:
        return [c["N"]] * c["B"]
    rng = random.Random(c["B"] * 1000003 + c["N"])
    n = [c["N"]] + [_log_int(rng, max(1, c["N"] // 64), c["N"]) for _ in range(c["B"] - 1)]
    if not c["tail"]:
        n = [max(GROUP, x // GROUP * GROUP) for x in n]
    rng.shuffle(n)
    return n


def _tables(B, mg, *key):
    g = _gen(*key)
    bt = torch.randperm(B * 4 * mg, generator=g, device="cuda").to(torch.int32).view(B, 4 * mg)
    gt = torch.randperm(B * mg, generator=g, device="cuda").to(torch.int32).view(B, mg)
    return bt, gt


def _slabs(lens, Hkv, most=1 << 27):
    """Runs of sequences of one length, at most `most` key values each."""
    b = 0
    while b < len(lens):
        n = 1
        while b + n < len(lens) and lens[b + n] == lens[b] and (n + 1) * Hkv * lens[b] * D <= most:
            n += 1
        yield b, n, lens[b]
        b += n


def prepare(c, seed):
    kind = c["kind"]
    if kind == "softmax":
        std = math.sqrt((124 + 400) / 128)  # of q.k / sqrt(128) for these activations
        x = torch.randn(c["rows"], c["cols"], generator=_gen(seed, 1), device="cuda")
        return dict(c=c, x=x.mul_(std))
    B, Hq, Hkv, N = c["B"], c["Hq"], c["Hkv"], c["N"]
    s = dict(c=c)
    if kind == "decode":
        lens = _lengths(c)
        mg = max(lens) // GROUP + 1
        s["bt"], s["gt"] = _tables(B, mg, seed, 2)
        s["cache"] = ta.PagedKVCache(B * 4 * mg, B * mg, _head_bits(c))
        s["tail"] = ta.KVTail(B, Hkv) if c["tail"] else None
        for b, n, length in _slabs(lens, Hkv):
            k, v = _kv(n, Hkv, length, seed, 3, b)
            _, _, sk, sv = ta.turbo_quantize_kv(k, v, s["cache"], s["bt"][b:b + n], s["gt"][b:b + n])
            if c["tail"]:
                ta.turbo_tail_init(k, v, sk, sv, s["tail"].narrow(b, n))
        s["q"] = _randn((B, Hq, D), seed, 4)
        if c["tail"]:
            k, v = _kv(B, Hkv, 1, seed, 5)
            s["k_new"], s["v_new"] = k.view(B, Hkv, D), v.view(B, Hkv, D)
        s["before"] = torch.tensor(lens, dtype=torch.int32, device="cuda")
        s["len"] = s["before"] + 1 if c["tail"] else s["before"]
        s["split"] = ta.decode_auto_split(B, Hq, Hkv, mg) if c["split"] < 0 else c["split"]
        s["ws"] = ta.decode_workspace(B, Hq, Hkv, mg, s["split"], with_tail=c["tail"])
        return s
    if kind == "project":
        F = (Hq + 2 * Hkv) * D
        s["x"] = _randn((B, N, c["D"]), seed, 6)
        w = torch.randn(F, c["D"], generator=_gen(seed, 7), device="cuda") / math.sqrt(c["D"])
        w.view(Hq + 2 * Hkv, D, -1)[Hq:Hq + Hkv, :4] *= 10.0
        s["w"] = w.half()
    else:
        s["q"] = _randn((B, Hq, N, D), seed, 4)
        s["k"], s["v"] = _kv(B, Hkv, N, seed, 3)
    if kind != "blocks":
        mg = (N + GROUP - 1) // GROUP
        s["bt"], s["gt"] = _tables(B, mg, seed, 2)
        s["cache"] = ta.PagedKVCache(B * 4 * mg, B * mg, _head_bits(c))
    if kind == "first":
        s["tail"] = ta.KVTail(B, Hkv)
    return s


def run(s):
    c = s["c"]
    kind = c["kind"]
    if kind == "softmax":
        return ta.turbo_sas_softmax(s["x"])
    if kind == "blocks":
        kv = ta.turbo_quantize_kv(s["k"], s["v"], block_cols=c["bc"])
        return dict(o=ta.turbo_attn_prefill(s["q"], *kv, causal=c["causal"], block_rows=c["br"],
                                            block_cols=c["bc"]))
    cache, bt, gt = s["cache"], s["bt"], s["gt"]
    if kind == "decode":
        tail = s["tail"]
        if tail is None:
            o, lse = ta.turbo_attn_decode(s["q"], cache, s["len"], bt, gt, workspace=s["ws"],
                                          kv_split_groups=s["split"], return_lse=True)
            return dict(o=o, lse=lse)
        ta.turbo_append_kv(s["k_new"], s["v_new"], s["before"], cache, tail, bt, gt)
        o, lse = ta.turbo_attn_decode(s["q"], cache, s["len"], bt, gt, workspace=s["ws"],
                                      kv_split_groups=s["split"], return_lse=True, tail=tail)
        out = dict(o=o, lse=lse, k=tail.k, v=tail.v)
        if c["ragged"]:  # some sequences fill their buffer: a group of the cache is written
            out.update(pages=cache.pages, meta=cache.group_meta)
        return out
    if kind == "project":
        q8, sq, k8, v8, sk, sv = ta.turbo_qkv_project(s["x"], s["w"], c["Hq"], c["Hkv"], cache, bt, gt)
        if c["attend"]:
            return dict(o=ta.turbo_attn_prefill_q8(q8, sq, k8, v8, sk, sv, c["N"]),
                        pages=cache.pages, meta=cache.group_meta)
        return dict(q8=q8, sq=sq, k8=k8, v8=v8, sk=sk, sv=sv, pages=cache.pages,
                    meta=cache.group_meta)
    out = dict(pages=cache.pages, meta=cache.group_meta)
    if kind == "first":
        out["priority"] = ta.turbo_head_priority(s["k"])
    kv = ta.turbo_quantize_kv(s["k"], s["v"], cache, bt, gt)
    if kind == "first":
        ta.turbo_tail_init(s["k"], s["v"], kv[2], kv[3], s["tail"])
        out.update(tk=s["tail"].k, tv=s["tail"].v)
        out["o"], out["lse"] = ta.turbo_attn_prefill(s["q"], *kv, causal=c["causal"],
                                                     return_lse=True)
    else:
        out["o"] = ta.turbo_attn_prefill(s["q"], *kv, causal=c["causal"])
    return out


# ---- what a pass cannot do without -------------------------------------------
def _group_bytes(c):
    """Bytes of one cached group over all KV heads: codes, s and z, block scales."""
    return sum(2 * GROUP * D * b // 8 + 4 * D + 8 for b in _head_bits(c))


def work(c):
    kind = c["kind"]
    if kind == "softmax":
        return dict(bytes=8.0 * c["rows"] * c["cols"], flops=10.0 * c["rows"] * c["cols"])
    B, Hq, Hkv, N = c["B"], c["Hq"], c["Hkv"], c["N"]
    if kind == "decode":
        done = [n + 1 if c["tail"] else n for n in _lengths(c)]
        nbytes = 4.0 * B * Hq * D + 4.0 * B * Hq
        nbytes += sum(n // GROUP * _group_bytes(c) for n in done)
        if c["tail"]:
            nbytes += sum(2.0 * (n % GROUP) * Hkv * D for n in done) + 6.0 * B * Hkv * D
        return dict(bytes=nbytes, flops=4.0 * D * Hq * sum(done))
    causal = c.get("causal", True)
    attend = 4.0 * D * B * Hq * (N * (N + 1) / 2 if causal else float(N) * N)
    q, kv = 2.0 * B * Hq * N * D, 2.0 * B * Hkv * N * D
    cached = 0.0 if kind == "blocks" else float(B * (N // GROUP) * _group_bytes(c))
    if kind == "project":
        F = (Hq + 2 * Hkv) * D
        nbytes = 2.0 * B * N * c["D"] + 2.0 * F * c["D"] + cached + (q if c["attend"] else q / 2 + kv)
        return dict(bytes=nbytes, flops=2.0 * B * N * c["D"] * F + (attend if c["attend"] else 0.0))
    return dict(bytes=2 * q + 2 * kv + cached, flops=attend)


def tolerance(c):
    kind = c["kind"]
    if kind == "softmax":
        return {"rel": 1e-6, "max": 1e-5}
    if kind == "project":
        # a sum in another order moves a few fp16 roundings and with them codes
        # (seen with fp32 inputs to the same product: 9e-4, 0.37, 6e-5)
        return {"rel": 4e-3, "max": 0.9, "differ": 3e-4}
    # the codes are fixed; fp32 sums in another order, rounded to fp16
    return {"rel": 1e-3, "max": 4e-3, "differ": 0.0}


# ---- the same results in 64 bits ----------------------------------------------
def _blocks(x, block):
    """(codes [.., nb, block, 128], scales [.., nb]) of step 1, rows past N zero.
    A code is the nearest integer of x * inv with inv = 119 / max rounded to
    binary32 once per block, which settles the many ties at half the maximum."""
    n = x.shape[-2]
    nb = (n + block - 1) // block
    x = torch.nn.functional.pad(x.double(), (0, 0, 0, nb * block - n))
    x = x.reshape(*x.shape[:-2], nb, block, D)
    top = x.abs().amax((-2, -1))
    inv = torch.where(top > 0, QMAX / top, 0.0).float().double()
    return torch.round(x * inv[..., None, None]), top / QMAX


def _sas(y):
    """e^-y by the table and the cubic; 0 beyond 6 and for y = inf."""
    k = y.clamp(max=6.0).floor()
    f = (y - k).clamp(max=1.0)
    p = ((POLY[0] * f + POLY[1]) * f + POLY[2]) * f + POLY[3]
    return torch.where(y <= 6.0, torch.exp(-k) * p, 0.0)


def _exact_attend(q8, sq, br, k8, sk, v8, sv, bc, N, causal):
    """Algorithm 1 on quantized operands: q8 [B][Hq][nq][br][128] and so on."""
    B, Hq = q8.shape[:2]
    Hkv = k8.shape[1]
    G, U = Hq // Hkv, B * Hkv
    nq, nk = q8.shape[2], k8.shape[2]
    q8 = q8.reshape(U, G, nq * br, D)
    sq = sq.reshape(U, G, nq, 1, 1)
    k8, v8 = k8.reshape(U, nk, bc, D), v8.reshape(U, nk, bc, D)
    sk, sv = sk.reshape(U, nk, 1, 1, 1, 1), sv.reshape(U, nk, 1, 1, 1, 1)
    R = nq * br
    o = torch.zeros(U, G, R, D, dtype=torch.float64, device=q8.device)
    m = torch.full((U, G, R, 1), -math.inf, dtype=torch.float64, device=q8.device)
    l = torch.zeros_like(m)
    rows = torch.arange(R, device=q8.device)
    for j in range(nk):
        i0 = j * bc // br if causal else 0
        r0, n = i0 * br, nq - i0
        keys = j * bc + torch.arange(bc, device=q8.device)
        vis = (keys < N) & (rows[r0:, None] < N)
        if causal:
            vis = vis & (keys <= rows[r0:, None])
        x = torch.bmm(q8[:, :, r0:].reshape(U, -1, D), k8[:, j].mT.contiguous())
        x = x.view(U, G, n, br, bc) * (sq[:, :, i0:] * sk[:, j] / math.sqrt(D))
        x = torch.where(vis, x.view(U, G, -1, bc), -math.inf)
        mo = m[:, :, r0:]
        mn = torch.maximum(mo, x.amax(-1, keepdim=True))
        p = torch.where(vis, _sas(mn - x), 0.0)
        a = torch.where(mn > mo, _sas(mn - mo), 1.0)
        l[:, :, r0:] = a * l[:, :, r0:] + p.sum(-1, keepdim=True)
        m[:, :, r0:] = mn
        p = p.view(U, G, n, br, bc)
        sp = p.amax((-2, -1), keepdim=True) / QMAX
        p8 = torch.round(p / torch.where(sp > 0, sp, 1.0))
        pv = torch.bmm(p8.view(U, -1, bc), v8[:, j]).view(U, G, n, br, D) * (sp * sv[:, j])
        o[:, :, r0:] = a * o[:, :, r0:] + pv.view(U, G, -1, D)
    o, lse = (o / l)[:, :, :N], (m + torch.log(l))[:, :, :N, 0]
    return o.reshape(B, Hq, N, D), lse.reshape(B, Hq, N)


def _expand(x8, levels):
    """int8 values [.., 64, 128] of groups after step 2 to `levels` + 1 levels."""
    z = x8.amin(-2, keepdim=True)
    s = torch.clamp(torch.ceil((x8.amax(-2, keepdim=True) - z) / levels), min=1.0)
    return torch.floor((2 * (x8 - z) + s) / (2 * s)) * s + z


def _universal(x, s):
    """Codes of the int8 buffer: the scale and its inverse are binary32."""
    inv = torch.where(s > 0, 1.0 / s.float(), 0.0).double()
    return torch.round(x.double() * inv).clamp(-QMAX, QMAX)


def _merge(parts):
    ms = torch.stack([p[0] for p in parts])
    top = ms.amax(0)
    w = torch.where(ms < top, _sas(top - ms), 1.0)
    den = sum(w[i] * p[1] for i, p in enumerate(parts))
    num = sum(w[i] * p[2] for i, p in enumerate(parts))
    return (num / den)[..., 0, :], (top + torch.log(den))[..., 0, 0]


def _exact_chunk(q8, sq, k8, sk, v8, sv, vis=None):
    """State (m, l, O) of one chunk: q8 [U][G][128], k8 [U][n][t][128]."""
    U, n, t = k8.shape[:3]
    G = q8.shape[1]
    x = torch.bmm(q8, k8.reshape(U, n * t, D).mT.contiguous()).view(U, G, n, t)
    x = x * (sq * sk[:, None] / math.sqrt(D))[..., None]
    if vis is not None:
        x = torch.where(vis, x, -math.inf)
    m = torch.cummax(x.amax(-1), -1).values
    p = _sas(m[..., None] - x)
    step = torch.where(m[..., 1:] > m[..., :-1], _sas(m[..., 1:] - m[..., :-1]), 1.0)
    fall = torch.cat([step, torch.ones_like(m[..., :1])], -1).flip(-1).cumprod(-1).flip(-1)
    sp = p.amax(-1, keepdim=True) / QMAX
    p8 = torch.round(p / torch.where(sp > 0, sp, 1.0)) * (sp * (sv[:, None] * fall)[..., None])
    o = torch.bmm(p8.view(U, G, n * t), v8.reshape(U, n * t, D))
    return m[..., -1:, None], (p.sum(-1) * fall).sum(-1)[..., None, None], o[:, :, None]


def _chunk_len(ng, split):
    if split > 0:
        return split
    return max(ng, 1) if ng <= 32 else 32 if ng <= 128 else -(-ng // 4)


def _exact_decode(c, seed):
    B, Hq, Hkv = c["B"], c["Hq"], c["Hkv"]
    G = Hq // Hkv
    lens = _lengths(c)
    split = ta.decode_auto_split(B, Hq, Hkv, max(lens) // GROUP + 1) if c["split"] < 0 else c["split"]
    levels = torch.tensor([(1 << b) - 1 for b in _head_bits(c)], dtype=torch.float64, device="cuda")
    levels = levels.view(1, Hkv, 1, 1, 1)
    q8, sq = _blocks(_randn((B, Hq, D), seed, 4)[..., None, :], 1)
    q8, sq = q8.view(B, Hkv, G, D), sq.view(B, Hkv, G, 1)
    if c["tail"]:
        kn, vn = _kv(B, Hkv, 1, seed, 5)
    o = torch.empty(B, Hq, D, dtype=torch.float64, device="cuda")
    lse = torch.empty(B, Hq, dtype=torch.float64, device="cuda")
    for b0, count, length in _slabs(lens, Hkv):
        kv = _kv(count, Hkv, length, seed, 3, b0)
        at, step = 0, max(1, (1 << 25) // (Hkv * length * D))
        while at < count:
            n = min(step, count - at)
            U, sl = n * Hkv, slice(b0 + at, b0 + at + n)
            ops = []  # per tensor: expanded groups, their scales, buffered codes, their scale
            for x, new in zip(kv, (kn, vn) if c["tail"] else (None, None)):
                x8, sx = _blocks(x[at:at + n], GROUP)
                full = length // GROUP
                us = sx.amax(-1)[..., None, None]
                x8, sx = _expand(x8[:, :, :full], levels), sx[:, :, :full]
                buf = None
                if c["tail"]:
                    buf = torch.cat([x[at:at + n, :, full * GROUP:], new[sl]], -2)
                    buf = _universal(buf, us)
                    if buf.shape[-2] == GROUP:
                        x8 = torch.cat([x8, _expand(buf[:, :, None], levels)], 2)
                        sx = torch.cat([sx, us[..., 0]], 2)
                        buf = None
                ops.append((x8.reshape(U, -1, GROUP, D), sx.reshape(U, -1),
                            None if buf is None else buf.reshape(U, 1, -1, D), us.reshape(U, 1)))
            (k8, sk, kb, uk), (v8, sv, vb, uv) = ops
            qu, su = q8[sl].reshape(U, G, D), sq[sl].reshape(U, G, 1)
            ng = k8.shape[1]
            ch = _chunk_len(ng, split)
            parts = [_exact_chunk(qu, su, k8[:, g:g + ch], sk[:, g:g + ch], v8[:, g:g + ch],
                                  sv[:, g:g + ch]) for g in range(0, ng, ch)]
            if kb is not None:
                parts.append(_exact_chunk(qu, su, kb, uk, vb, uv))
            ou, lu = _merge(parts)
            o[sl], lse[sl] = ou.view(n, Hq, D), lu.view(n, Hq)
            at += n
    out = dict(o=o, lse=lse)
    if c["tail"]:
        out.update(k=None, v=None)
        if c["ragged"]:
            out.update(pages=None, meta=None)
    return out


def exact(c, seed):
    kind = c["kind"]
    s = prepare(c, seed) if kind != "decode" else None
    if kind == "softmax":
        y = torch.empty(s["x"].shape, dtype=torch.float64, device="cuda")
        for x, out in zip(s["x"].split(8192), y.split(8192)):
            e = _sas(x.double().amax(-1, keepdim=True) - x.double())
            torch.div(e, e.sum(-1, keepdim=True), out=out)
        return y
    if kind == "decode":
        return _exact_decode(c, seed)
    N, br, bc = c["N"], c.get("br", 64), c.get("bc", 64)
    if kind == "project":
        y = torch.matmul(s["x"].double().view(-1, c["D"]), s["w"].double().t().contiguous())
        y = y.view(c["B"], N, -1, D).transpose(1, 2)
        q, k, v = y.split([c["Hq"], c["Hkv"], c["Hkv"]], 1)
    else:
        q, k, v = s["q"], s["k"], s["v"]
    (q8, sq), (k8, sk), (v8, sv) = _blocks(q, br), _blocks(k, bc), _blocks(v, bc)
    if kind == "project" and not c["attend"]:
        return dict(q8=None, sq=sq, k8=None, v8=None, sk=sk, sv=sv, pages=None, meta=None)
    o, lse = _exact_attend(q8, sq, br, k8, sk, v8, sv, bc, N, c.get("causal", True))
    if kind == "blocks":
        return dict(o=o)
    out = dict(pages=None, meta=None, o=o)
    if kind == "first":
        kd = s["k"].double()
        hi, lo = kd.amax((0, 2)), kd.amin((0, 2))
        out["priority"] = (hi.amax(-1) - lo.amin(-1)) * (hi - lo).std(-1, unbiased=False)
        out.update(tk=None, tv=None, lse=lse)
    return out
