"""Parity of the kernel for chunks with little work (tetri_short.hip), forced with "attn_variant" 3: every number of
wavefronts it is launched with, key ranges split over workgroups or not, edges of row blocks, pages and steps, 16-bit and
FP8 pool; outputs against the oracle, cached rows bit for bit."""
import numpy as np
import pytest
import torch

from oracle import tetri_oracle
from paper_2401_11181_amd import synth
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
