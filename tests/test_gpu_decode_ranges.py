"""Decode over equal ranges of the batch's steps ("decode_ranges"): ranges that cut requests anywhere, hold many of them, or
outnumber the steps; 16-bit and FP8 cache, with the fused append, against the oracle."""
import numpy as np
import pytest
import torch

from oracle import decode as odecode
from oracle import fp8 as ofp8
from paper_2401_11181_amd import synth, tetri
from test_gpu_decode import build, reference
import gpu_common as gc

pytestmark = pytest.mark.gpu
DEV = gc.DEV

# tokens of the requests (cached ones and the new one), heads, kv heads, head dim
BATCHES = {
    "ragged": ([1, 2, 33, 32, 65, 700, 16, 17, 300, 1, 129], 4, 4, 128),
    "gqa": ([900, 5, 33, 64, 31], 16, 2, 128),                       # 8 query heads: two rounds of the merge area
    "d64": ([1, 450, 97, 96, 33, 2, 2, 2, 700], 6, 2, 64),
    "many": ([int(x) for x in np.random.default_rng(5).integers(1, 70, size=150)], 2, 1, 128),   # several requests per lane of the look-up
}


def run(w, fn, ranges, args, out):
    h = tetri.Tetri(w.num_q_heads, w.num_kv_heads, w.head_dim, 64, w.num_pages, args[4].shape[1], 8)
    if ranges is not None:
        h.tetri_set_option("decode_ranges", ranges)
    for _ in range(2):                                   # the second call finds the counters as the first one left them
        out.fill_(7.0)
        fn(h)
    torch.cuda.synchronize()
    h.close()
    return out.cpu()


@pytest.mark.parametrize("ranges", [2, 3, 11, 200])
@pytest.mark.parametrize("name", sorted(BATCHES))
def test_16_bit_cache(name, ranges):
    lens, hq, hkv, d = BATCHES[name]
    w = synth.small("ranges-" + name, lens, 64, hq, hkv, d, seed=900 + sorted(BATCHES).index(name))
    q, k, v, pool, bt, ctx = build(w, stale=float("nan"))
    args = [t.to(DEV) for t in (q, k, v, pool)] + [torch.from_numpy(bt).to(DEV), torch.from_numpy(ctx).to(DEV)]
    out = torch.zeros(q.shape, dtype=torch.bfloat16, device=DEV)
    got = run(w, lambda h: h.tetri_decode_attn_append(*args, len(ctx), int(ctx.max()), w.scale, out), ranges, args, out)
    gc.compare([got], [reference(w, q, k, v, pool, bt, ctx)], label=name)
    after = args[3].cpu()
    for b in range(len(ctx)):
        page, slot = bt[b, ctx[b] // 16], ctx[b] % 16
        assert torch.equal(after[page, 0, :, slot].view(torch.int16), k[b].view(torch.int16))
        assert torch.equal(after[page, 1, :, slot].view(torch.int16), v[b].view(torch.int16))


@pytest.mark.parametrize("ranges", [2, 11, 200])
@pytest.mark.parametrize("name", sorted(BATCHES))
def test_fp8_cache(name, ranges):
    lens, hq, hkv, d = BATCHES[name]
    w = synth.small("ranges8-" + name, lens, 64, hq, hkv, d, seed=910 + sorted(BATCHES).index(name))
    q, k, v, pool, bt, ctx = build(w)
    ks, vs = 0.0137, 0.0171
    codes = np.full(tuple(pool.shape), 0x7f, np.uint8)               # unused slots hold the code that is not a number
    clean = pool.float().numpy()
    for b in range(len(ctx)):
        for j in range(ctx[b]):
            page, slot = bt[b, j // 16], j % 16
            codes[page, 0, :, slot] = ofp8.quantize(clean[page, 0, :, slot], ks)
            codes[page, 1, :, slot] = ofp8.quantize(clean[page, 1, :, slot], vs)
    deq = np.zeros(pool.shape, np.float32)
    deq[:, 0], deq[:, 1] = ofp8.dequantize(codes[:, 0], ks), ofp8.dequantize(codes[:, 1], vs)
    deq = np.nan_to_num(deq, nan=0.0)
    args = [q.to(DEV), k.to(DEV), v.to(DEV), torch.from_numpy(codes).to(DEV), torch.from_numpy(bt).to(DEV), torch.from_numpy(ctx).to(DEV)]
    out = torch.zeros(q.shape, dtype=torch.bfloat16, device=DEV)
    got = run(w, lambda h: h.tetri_decode_attn_fp8(*args, len(ctx), int(ctx.max()), w.scale, ks, vs, 1, out), ranges, args, out)
    ref = odecode.decode_attn(q.float().numpy(), k.float().numpy(), v.float().numpy(), deq, bt, ctx, w.scale)
    gc.compare([got], [ref], label=name)
    after = args[3].cpu().numpy()
    for b in range(len(ctx)):
        page, slot = bt[b, ctx[b] // 16], ctx[b] % 16
        assert np.array_equal(after[page, 0, :, slot], ofp8.quantize(k[b].float().numpy(), ks))
        assert np.array_equal(after[page, 1, :, slot], ofp8.quantize(v[b].float().numpy(), vs))


# Batches that the library itself cuts into ranges (of at least four steps each, unlike forced ones): the bound of the
# context lengths that the host is told makes them much to read.  Cached and new tokens; 22 requests, so that 8 kv heads
# reach the rule with codes too (host_launches.cpp, decode_division, pins it).
RULE_LENS = [1, 33, 4, 700, 128, 129, 65, 1, 1300, 31, 64, 257, 2, 90, 511, 3, 16, 17, 1, 420, 96, 32]


@pytest.mark.parametrize("fp8", [False, True], ids=["16-bit", "fp8"])
def test_ranges_by_the_librarys_own_rule(fp8):
    w = synth.small("ranges-rule", RULE_LENS, 64, 16, 8, 128, seed=930)
    q, k, v, pool, bt, ctx = build(w)
    bt = np.pad(bt, ((0, 0), (0, 300 - bt.shape[1])))
    ks, vs = 0.0137, 0.0171
    clean = pool.float().numpy()
    if fp8:
        codes = np.full(tuple(pool.shape), 0x7f, np.uint8)
        used = np.zeros(tuple(pool.shape[:1]) + (16,), bool)
        for b in range(len(ctx)):
            for j in range(ctx[b]):
                used[bt[b, j // 16], j % 16] = True
        for which, scale in ((0, ks), (1, vs)):
            x = np.moveaxis(clean[:, which], 2, 1)                       # [page][slot][head][d]
            c = np.moveaxis(codes[:, which], 2, 1)
            c[used] = ofp8.quantize(x[used], scale)
        clean = np.stack([ofp8.dequantize(codes[:, 0], ks), ofp8.dequantize(codes[:, 1], vs)], axis=1)
        pool = torch.from_numpy(codes)
    args = [t.to(DEV) for t in (q, k, v, pool)] + [torch.from_numpy(bt).to(DEV), torch.from_numpy(ctx).to(DEV)]
    out = torch.zeros(q.shape, dtype=torch.bfloat16, device=DEV)
    if fp8:
        got = run(w, lambda h: h.tetri_decode_attn_fp8(*args, len(ctx), 4700, w.scale, ks, vs, 0, out), None, args, out)
    else:
        got = run(w, lambda h: h.tetri_decode_attn(*args, len(ctx), 4700, w.scale, out), None, args, out)
    ref = odecode.decode_attn(q.float().numpy(), k.float().numpy(), v.float().numpy(), np.nan_to_num(clean, nan=0.0), bt, ctx, w.scale)
    gc.compare([got], [ref], label="rule")
