"""Decode with one, two, four and eight waves per chunk: the waves share the
groups of a chunk, and the result is that of one wave, bit for bit.

The number of waves follows the number of chunks in the launch and their length,
so one sequence is decoded alone and repeated 160, 500 and 1000 times (two KV
heads, one chunk each: 2, 320, 1000 and 2000 chunks); its rows must have the same
bits each time, and the lone one is checked against the CPU oracle.  With 7 and 9
groups that is eight, four, two and one wave for every number of rows; with 31 and
eight rows eight, four, two and two, with sixteen eight, four, two and four; with 64
and eight rows eight, four, four and two, with sixteen eight, four, four and four.
"""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

SM = 1 / np.sqrt(128)


@pytest.fixture(scope="module")
def dev():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch.device("cuda:0")


@pytest.fixture(scope="module")
def ta(dev):
    import paper_2412_08585_amd as ta
    ta.lib()
    return ta


def _rand(shape, seed):
    return torch.randn(*shape, generator=torch.Generator().manual_seed(seed)).half()


def _bits(t):
    return t.contiguous().view(torch.int16 if t.dtype == torch.float16 else torch.int32)


# groups: below, at and past the steps of 2, 4 and 8 groups; one group; past the
# 64 table entries a lane holds at a time (515: 64 steps of 8 groups; 130 with one
# row: twice with one wave, once with two); the lengths past which long chunks take
# other numbers of waves
CASES = [(G, ng) for G in (1, 2, 4, 8, 16) for ng in (1, 9, 31)] + [
    (3, 16), (5, 22), (2, 515), (1, 130), (8, 7), (8, 64), (16, 64)]


@pytest.mark.parametrize("G,ng", CASES)
def test_decode_waves_give_the_bits_of_one(orc, ta, dev, G, ng):
    print(f"decode waves G={G} ng={ng}", flush=True)
    Hkv, bits = 2, [4, 2]
    Hq = G * Hkv
    k, v = _rand((1, Hkv, 64 * ng, 128), 10 * ng + G), _rand((1, Hkv, 64 * ng, 128), 11 * ng + G)
    k[..., 7] *= 10
    if ng > 20:  # a maximum near the end: factors that cut the earlier groups off
        k[:, :, 64 * (ng - 3)] *= 4
    q = _rand((1, Hq, 128), 12 * ng + G)
    rng = np.random.default_rng(ng)
    bt = rng.permutation(4 * ng).astype(np.int32)[None]
    gt = rng.permutation(ng).astype(np.int32)[None]
    cache = ta.PagedKVCache(4 * ng, ng, bits, dev)
    btd, gtd, qd = torch.from_numpy(bt).to(dev), torch.from_numpy(gt).to(dev), q.to(dev)
    ta.turbo_quantize_kv(k.to(dev), v.to(dev), cache, btd, gtd)
    sl = torch.full((1,), 64 * ng, dtype=torch.int32, device=dev)

    def run(B, bt_, gt_):
        args = (qd.repeat(B, 1, 1), cache, sl.repeat(B), bt_.repeat(B, 1), gt_.repeat(B, 1))
        o, lse = ta.turbo_attn_decode(*args, SM, 1000, return_lse=True)
        o2, lse2 = ta.turbo_attn_decode(*args, SM, 2, return_lse=True)  # chunks of two groups
        torch.cuda.synchronize()
        return o, lse, o2, lse2

    alone = run(1, btd, gtd)
    ref = orc.quantize_kv(k, v, bits)
    ro, rl = orc.attn_decode(q, ref, [64 * ng], SM, split=ng)
    err = np.abs(alone[0].float().cpu().numpy() - ro) / np.abs(ro).max(axis=-1, keepdims=True)
    assert err.max() < 1e-3
    assert np.abs(alone[1].cpu().numpy() - rl).max() < 1e-4
    skip = gtd.clone()
    skip[0, ng // 2] = -1  # a group that is not attended
    skipped = run(1, btd, skip)
    for B in (160, 500, 1000):
        for got, want in zip(run(B, btd, gtd) + run(B, btd, skip), alone + skipped):
            assert torch.equal(_bits(got), _bits(want).expand(B, *want.shape[1:])), B


@pytest.mark.parametrize("G", [1, 2, 4, 8, 16])
def test_decode_waves_trace_the_same_integers(ta, dev, G):
    ng, Hkv, bits = 11, 2, [2, 4]
    k, v = _rand((1, Hkv, 64 * ng, 128), 50 + G), _rand((1, Hkv, 64 * ng, 128), 60 + G)
    q = _rand((1, G * Hkv, 128), 70 + G).to(dev)
    bt = torch.arange(4 * ng, dtype=torch.int32, device=dev)[None]
    gt = torch.arange(ng, dtype=torch.int32, device=dev)[None]
    cache = ta.PagedKVCache(4 * ng, ng, bits, dev)
    ta.turbo_quantize_kv(k.to(dev), v.to(dev), cache, bt, gt)
    sl = torch.full((1,), 64 * ng, dtype=torch.int32, device=dev)
    for (h, g) in ((0, 0), (G, 6), (2 * G - 1, ng - 1)):
        want = None
        for B in (1, 160, 500, 1000):
            print(f"decode waves trace G={G} B={B} h={h} g={g}", flush=True)
            _, t = ta.turbo_attn_decode_trace(q.repeat(B, 1, 1), cache, sl.repeat(B),
                                              bt.repeat(B, 1), gt.repeat(B, 1), (B - 1, h, g), SM,
                                              1000)
            want = t if want is None else want
            assert np.any(t["pvacc"])
            for name in t:
                assert np.array_equal(t[name], want[name]), (B, name)


@pytest.mark.parametrize("G,ng,N", [(1, 8, 23), (4, 14, 64), (8, 6, 1), (16, 31, 40)])
def test_decode_waves_with_a_buffer(ta, dev, G, ng, N):
    """N rows in the int8 buffer, whose work-groups count for the number of waves:
    1, 160, 300, 500 and 1000 times the same sequence give the bits of one."""
    print(f"decode waves with a buffer G={G} ng={ng} N={N}", flush=True)
    Hkv, bits, n = 2, [4, 2], 64 * ng + N % 64
    k, v = _rand((1, Hkv, n, 128), 110 + G), _rand((1, Hkv, n, 128), 120 + G)
    q = _rand((1, G * Hkv, 128), 130 + G).to(dev)
    width = ng + (N % 64 > 0)
    cache = ta.PagedKVCache(4 * width, width, bits, dev)
    bt = torch.arange(4 * width, dtype=torch.int32, device=dev)[None]
    gt = torch.arange(width, dtype=torch.int32, device=dev)[None]
    res = ta.turbo_quantize_kv(k.to(dev), v.to(dev), cache, bt, gt)
    one = ta.KVTail(1, Hkv, dev)
    ta.turbo_tail_init(k.to(dev), v.to(dev), res[2], res[3], one)
    want = None
    for B in (1, 160, 300, 500, 1000):
        tail = ta.KVTail(B, Hkv, dev)
        tail.k.copy_(one.k.expand_as(tail.k))
        tail.v.copy_(one.v.expand_as(tail.v))
        tail.scale.copy_(one.scale.expand_as(tail.scale))
        sl = torch.full((B,), n, dtype=torch.int32, device=dev)
        got = ()
        for split in (1000, 3):
            got += tuple(ta.turbo_attn_decode(q.repeat(B, 1, 1), cache, sl, bt.repeat(B, 1),
                                              gt.repeat(B, 1), SM, split, return_lse=True,
                                              tail=tail))
        torch.cuda.synchronize()
        want = got if want is None else want
        for g, w in zip(got, want):
            assert torch.equal(_bits(g), _bits(w).expand(B, *w.shape[1:])), B


@pytest.mark.parametrize("G,B", [(1, 3), (4, 21), (8, 9)])
def test_decode_tables_wider_than_the_sequences(ta, dev, G, B):
    """The work-groups of a chunk number are rotated by the sequence, over as many
    chunks as the table's width asks for (one, two, three and four here, and five
    and six by an explicit split); sequences of every number of chunks, and empty
    ones, give the bits that each gives alone in a table of its own width."""
    print(f"decode wide tables G={G} B={B}", flush=True)
    Hkv, bits = 2, [4, 2]
    groups = [(0, 1, 3, 9, 20, 31)[i % 6] + i // 6 for i in range(B)]
    total = sum(groups)
    k, v = _rand((1, Hkv, 64 * total, 128), 80 + G), _rand((1, Hkv, 64 * total, 128), 90 + G)
    q = _rand((B, G * Hkv, 128), 100 + G).to(dev)
    cache = ta.PagedKVCache(4 * total, total, bits, dev)
    gall = torch.randperm(total, generator=torch.Generator().manual_seed(B)).int()
    ball = (4 * gall[:, None] + torch.arange(4)).int()
    ta.turbo_quantize_kv(k.to(dev), v.to(dev), cache, ball.reshape(1, -1).to(dev),
                         gall[None].to(dev))

    def run(rows, width, split):
        gt = torch.full((len(rows), width), -1, dtype=torch.int32)
        bt = torch.full((len(rows), width, 4), -1, dtype=torch.int32)
        for i, r in enumerate(rows):
            at, n = sum(groups[:r]), groups[r]
            gt[i, :n], bt[i, :n] = gall[at:at + n], ball[at:at + n]
        sl = torch.tensor([64 * groups[r] for r in rows], dtype=torch.int32, device=dev)
        o, lse = ta.turbo_attn_decode(q[rows], cache, sl, bt.view(len(rows), -1).to(dev),
                                      gt.to(dev), SM, split, return_lse=True)
        torch.cuda.synchronize()
        return o, lse

    for split, widths in ((0, (max(groups), 40, 70, 400)), (8, (40, 45))):
        alone = [run([r], max(groups[r], 1), split) for r in range(B)]
        for width in widths:
            o, lse = run(list(range(B)), width, split)
            for r in range(B):
                assert torch.equal(_bits(o[r]), _bits(alone[r][0][0])), (split, width, r)
                assert torch.equal(_bits(lse[r]), _bits(alone[r][1][0])), (split, width, r)
