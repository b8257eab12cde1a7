"""Parity of the kernel for chunks with little work (tetri_short.hip), forced with "attn_variant" 3: every number of
wavefronts it is launched with, key ranges split over workgroups or not, edges of row blocks, pages and steps, 16-bit and
FP8 pool; outputs against the oracle, cached rows bit for bit."""
import numpy as np
import pytest
import torch

from oracle import tetri_oracle
from oracle import fp8 as ofp8
from paper_2401_11181_amd import synth, tetri
import gpu_common as gc

pytestmark = pytest.mark.gpu

# name: prompt lengths, chunk size, heads, kv heads, head dim
CASES = {
    "one-row": ([1], 16, 2, 2, 128),                                 # 8 / 4 wavefronts, most of them idle
    "edges": ([31, 32, 33, 15, 16, 17, 1, 64], 96, 4, 2, 64),        # row blocks and contexts that end around 16 and 32
    "edges-128": ([31, 32, 33, 15, 16, 17, 1, 64], 96, 4, 2, 128),
    "ragged-ctx": ([250], 37, 6, 2, 64),                             # contexts of 37, 74, ...: mid-page, mid-step
    "split": ([700], 64, 2, 1, 128),                                 # few row blocks: up to 16 workgroups share their keys
    "split-64": ([900, 333], 128, 4, 4, 64),
    "split-uneven": ([530], 33, 3, 3, 128),                          # parts of different lengths, some with nothing
    "four": ([300, 260], 256, 40, 40, 128),                          # 257..512 workgroups
    "two": ([512, 70], 512, 40, 8, 128),                             # 513..1152
    "one": ([17] * 30, 512, 40, 40, 128),                            # more, short key ranges
    "one-then-two": ([20] * 28 + [400], 1024, 32, 8, 128),
    "wide": ([60] * 10 + [131], 731, 40, 40, 128),                # 30 MB read and written: output by way of the caches
}


@pytest.mark.parametrize("fused", [False, True])
@pytest.mark.parametrize("name", sorted(CASES))
def test_16_bit_pool(name, fused):
    lens, chunk, hq, hkv, d = CASES[name]
    w = synth.small("short-" + name, lens, chunk, hq, hkv, d, seed=700 + sorted(CASES).index(name))
    qs, ks, vs, tables = gc.workload_tensors(w)
    outs, pool, _sess, _ = gc.gpu_prefill(w, qs, ks, vs, tables, pad_fill=float("nan"), variant=3, fused=fused)
    ref, _, _ = gc.oracle_prefill(tetri_oracle, w, qs, ks, vs, tables)
    gc.compare(outs, ref, label=w.name)
    bits = gc.oracle_pool_bits(tetri_oracle, w, ks, vs, tables)
    assert np.array_equal(pool.cpu().view(torch.int16).numpy().view(np.uint16), bits)


@pytest.mark.parametrize("name", sorted(CASES))
def test_fp8_pool(name):
    lens, chunk, hq, hkv, d = CASES[name]
    w = synth.small("short8-" + name, lens, chunk, hq, hkv, d, seed=720 + sorted(CASES).index(name))
    qs, ks, vs, tables = gc.workload_tensors(w)
    outs, pool, _sess = gc.gpu_prefill_fp8(w, qs, ks, vs, tables, 0.0137, 0.0171, variant=3)
    ref, codes = gc.oracle_prefill_fp8(w, qs, ks, vs, tables, 0.0137, 0.0171)
    gc.compare(outs, ref, label=w.name)
    assert np.array_equal(pool.cpu().numpy(), codes)


@pytest.mark.parametrize("scale", [0.0, -0.11, 3.0])
def test_softmax_scales(scale):
    w = synth.small("short-scale", [75, 130], 96, 4, 2, 128, seed=741)
    w.scale = scale
    qs, ks, vs, tables = gc.workload_tensors(w)
    outs, _pool, _sess, _ = gc.gpu_prefill(w, qs, ks, vs, tables, variant=3)
    ref, _, _ = gc.oracle_prefill(tetri_oracle, w, qs, ks, vs, tables)
    gc.compare(outs, ref, label=w.name)


@pytest.mark.parametrize("fp8", [0, 1], ids=["16-bit", "fp8"])
@pytest.mark.parametrize("hq, hkv, rows, ctx", [(8, 2, 33, 20011), (32, 8, 250, 3017), (24, 8, 500, 3003)],
                         ids=["split", "eight-wavefronts", "four-wavefronts"])
def test_long_contexts(hq, hkv, rows, ctx, fp8):
    """Chunks behind long cached contexts that the library's own rule gives to this kernel (but for the codes of the last one),
    all rows against attention in 64 bits over the same values."""
    d, mb = 128, -(-(ctx + rows) // 16)
    g = torch.Generator().manual_seed(751)
    rnd = lambda *shape: torch.randn(shape, generator=g).to(torch.bfloat16)
    q, k, v = rnd(rows, hq, d), rnd(rows, hkv, d), rnd(rows, hkv, d)
    past = rnd(2, hkv, mb * 16, d)
    ks, vs = (0.0137, 0.0171) if fp8 else (1.0, 1.0)
    if fp8:
        codes = np.stack([ofp8.quantize(past[i].float().numpy(), s) for i, s in ((0, ks), (1, vs))])
        values = np.stack([ofp8.dequantize(codes[i], s) for i, s in ((0, ks), (1, vs))])
        past, held = torch.from_numpy(values), torch.from_numpy(codes)
        held[:, :, ctx:] = gc.NAN_CODE
    else:
        held = past.clone()
        held[:, :, ctx:] = float("nan")
    order = torch.randperm(mb, generator=g)
    pool = torch.empty((mb, 2, hkv, 16, d), dtype=held.dtype)
    pool[order] = held.reshape(2, hkv, mb, 16, d).permute(2, 0, 1, 3, 4)
    cu, cl = np.array([0, rows], np.int32), np.array([ctx], np.int32)
    h = tetri.Tetri(hq, hkv, d, rows, mb, mb, 1)
    out = torch.full((rows, hq, d), 7.0, dtype=torch.bfloat16, device=gc.DEV)
    dev = [t.to(gc.DEV) for t in (q, k, v, pool, order.to(torch.int32), torch.from_numpy(cu), torch.from_numpy(cl))]
    h.tetri_chunk_prefill_planned(*dev, 1, d ** -0.5, 0, fp8, ks, vs, cu, cl, out)
    torch.cuda.synchronize()
    want = torch.empty((rows, hq, d), dtype=torch.float64)
    for head in range(hq):
        kh = head // (hq // hkv)
        keys = torch.cat([past[0, kh, :ctx].double(), k[:, kh].double()])
        vals = torch.cat([past[1, kh, :ctx].double(), v[:, kh].double()])
        s = q[:, head].double() @ keys.T * d ** -0.5
        s.masked_fill_(torch.arange(ctx + rows)[None, :] > torch.arange(rows)[:, None] + ctx, float("-inf"))
        want[:, head] = s.softmax(dim=1) @ vals
    gc.compare([out.cpu()], [want.numpy()], label="long context")
    h.close()
