"""Parity of the shared-tile kernel on a division made by the host (tetri_planned.hip), forced with "attn_variant" 4 and 5: tiles
cut into several pieces, workgroups with several jobs, ragged segments, every kind of edge, 16-bit and FP8 pool; outputs against
the oracle, cached rows bit for bit."""
import numpy as np
import pytest
import torch

from oracle import tetri_oracle
from paper_2401_11181_amd import synth, tetri
import gpu_common as gc

pytestmark = pytest.mark.gpu

# name: prompt lengths, chunk size, heads, kv heads
CASES = {
    "one-row": ([1], 16, 8, 8),
    "edges": ([31, 32, 33, 15, 16, 17, 1, 64, 127, 128, 129], 96, 4, 2),   # row blocks, pages and stages that end around their edges
    "pieces": ([1500], 64, 4, 4),                    # one tile of up to 12 stages: cut into pieces for 4 workgroups
    "own-rows": ([900, 333], 300, 8, 8),             # 256-row tiles: their own rows in two stages, mid-page starts
    "jobs": ([20] * 30 + [300], 512, 40, 40),        # 5 head groups a pool: several jobs to a workgroup
    "gqa": ([700, 70, 260], 256, 32, 8),
    "gqa-odd": ([515], 130, 24, 8),                  # three query heads to a kv head
    "few-groups": ([640], 96, 6, 2),                 # six head groups: two XCDs without work
}


@pytest.mark.parametrize("variant", [4, 5])
@pytest.mark.parametrize("name", sorted(CASES))
def test_16_bit_pool(name, variant):
    lens, chunk, hq, hkv = CASES[name]
    w = synth.small("planned-" + name, lens, chunk, hq, hkv, 128, seed=800 + sorted(CASES).index(name))
    qs, ks, vs, tables = gc.workload_tensors(w)
    outs, pool, _sess, _ = gc.gpu_prefill(w, qs, ks, vs, tables, pad_fill=float("nan"), variant=variant, fused=True)
    ref, _, _ = gc.oracle_prefill(tetri_oracle, w, qs, ks, vs, tables)
    gc.compare(outs, ref, label=w.name)
    bits = gc.oracle_pool_bits(tetri_oracle, w, ks, vs, tables)
    assert np.array_equal(pool.cpu().view(torch.int16).numpy().view(np.uint16), bits)


@pytest.mark.parametrize("variant", [4, 5])
@pytest.mark.parametrize("name", sorted(CASES))
def test_fp8_pool(name, variant):
    lens, chunk, hq, hkv = CASES[name]
    w = synth.small("planned8-" + name, lens, chunk, hq, hkv, 128, seed=820 + sorted(CASES).index(name))
    qs, ks, vs, tables = gc.workload_tensors(w)
    outs, pool, _sess = gc.gpu_prefill_fp8(w, qs, ks, vs, tables, 0.0137, 0.0171, variant=variant)
    ref, codes = gc.oracle_prefill_fp8(w, qs, ks, vs, tables, 0.0137, 0.0171)
    gc.compare(outs, ref, label=w.name)
    assert np.array_equal(pool.cpu().numpy(), codes)


@pytest.mark.parametrize("variant", [4, 5])
@pytest.mark.parametrize("segs, hq, hkv", [([(256, 5003)], 16, 16), ([(100, 9001), (412, 0)], 32, 8), ([(250, 777), (37, 4000), (225, 31)], 8, 2)],
                         ids=["mha", "ragged", "few-groups"])
def test_long_contexts(segs, hq, hkv, variant):
    """Several launches of one chunk in a row: pieces meet in the same places and counters each time, with the same bits."""
    d, rows = 128, sum(n for n, _ in segs)
    g = torch.Generator().manual_seed(831)
    rnd = lambda *shape: torch.randn(shape, generator=g).to(torch.bfloat16)
    need = [-(-(n + c) // 16) for n, c in segs]
    q, k, v, pool = rnd(rows, hq, d), rnd(rows, hkv, d), rnd(rows, hkv, d), rnd(sum(need), 2, hkv, 16, d)
    order, at = torch.randperm(sum(need), generator=g), 0
    bt = torch.zeros((len(segs), max(need)), dtype=torch.int32)
    for i, n in enumerate(need):
        bt[i, :n] = order[at:at + n].to(torch.int32)
        at += n
    cu, cl = np.cumsum([0] + [n for n, _ in segs]).astype(np.int32), np.array([c for _, c in segs], np.int32)
    h = tetri.Tetri(hq, hkv, d, rows, sum(need), max(need), len(segs))
    h.tetri_set_option("attn_variant", variant)
    dev = [t.to(gc.DEV) for t in (q, k, v, pool, bt, torch.from_numpy(cu), torch.from_numpy(cl))]
    outs = []
    for _ in range(6):
        outs.append(torch.full((rows, hq, d), 7.0, dtype=torch.bfloat16, device=gc.DEV))
        h.tetri_chunk_prefill_planned(*dev, len(segs), d ** -0.5, 0, 0, 1.0, 1.0, cu, cl, outs[-1])
    torch.cuda.synchronize()
    want = torch.empty((rows, hq, d), dtype=torch.float64)
    for i, (n, ctx) in enumerate(segs):
        past = pool[bt[i].long()].permute(1, 2, 0, 3, 4).reshape(2, hkv, -1, d)[:, :, :ctx].double()
        r = slice(int(cu[i]), int(cu[i + 1]))
        for head in range(hq):
            kh = head // (hq // hkv)
            s = q[r, head].double() @ torch.cat([past[0, kh], k[r, kh].double()]).T * d ** -0.5
            s.masked_fill_(torch.arange(ctx + n)[None, :] > torch.arange(n)[:, None] + ctx, float("-inf"))
            want[r, head] = s.softmax(dim=1) @ torch.cat([past[1, kh], v[r, kh].double()])
    gc.compare([outs[0].cpu()], [want.numpy()], label="long context")
    for o in outs[1:]:
        assert torch.equal(o, outs[0])
    h.close()
