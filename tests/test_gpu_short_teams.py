"""Parity of the kernel for chunks with little work (tetri_short.hip) where row blocks of one launch have teams of different sizes:
segments of very different contexts, several teams to a workgroup and one, an odd and an even number of steps of codes to a
wavefront, ragged ends; against attention in 64 bits over the same values, cached rows bit for bit."""
import numpy as np
import pytest
import torch

from oracle import fp8 as ofp8
from paper_2401_11181_amd import tetri
import gpu_common as gc

pytestmark = pytest.mark.gpu

# heads, kv heads, head dim, (rows, cached tokens) of the segments
CASES = {
    "1-2-4-8": (8, 2, 128, [(33, 2001), (40, 700), (64, 333), (130, 64), (200, 0), (5, 31)]),
    "many-heads": (40, 40, 128, [(17, 900), (70, 160), (1, 1), (31, 32), (64, 0), (300, 0)]),
    "odd-heads": (24, 8, 128, [(100, 1500), (37, 95), (63, 0), (200, 0)]),
    "one-to-a-workgroup": (6, 3, 128, [(40, 450), (60, 97), (32, 0)]),
    "eight-wavefronts-in-packs": (32, 8, 128, [(120, 50), (128, 301), (97, 700), (33, 0)]),
    "long": (24, 8, 128, [(500, 3003)]),
    "head-dim-64": (12, 4, 64, [(33, 1203), (64, 129), (90, 0), (301, 17), (2, 600)]),
    "head-dim-64-many": (40, 40, 64, [(50, 1100), (400, 30), (128, 0)]),
    "twos": (40, 40, 64, [(1031, 17)]),                        # more than one round of workgroups, no row block with one wavefront
}


@pytest.mark.parametrize("fp8", [0, 1], ids=["16-bit", "fp8"])
@pytest.mark.parametrize("name", sorted(CASES))
def test_teams(name, fp8):
    hq, hkv, d, segs = CASES[name]
    g = torch.Generator().manual_seed(900 + sorted(CASES).index(name))
    rnd = lambda *shape: torch.randn(shape, generator=g).to(torch.bfloat16)
    rows, need = sum(n for n, _ in segs), [-(-(n + c) // 16) for n, c in segs]
    q, k, v, past = rnd(rows, hq, d), rnd(rows, hkv, d), rnd(rows, hkv, d), rnd(2, hkv, sum(need) * 16, d)
    ks, vs = (0.0137, 0.0171) if fp8 else (1.0, 1.0)
    held = past
    if fp8:
        codes = np.stack([ofp8.quantize(past[i].float().numpy(), s) for i, s in ((0, ks), (1, vs))])
        held, past = torch.from_numpy(codes), torch.from_numpy(np.stack([ofp8.dequantize(codes[i], s) for i, s in ((0, ks), (1, vs))]))
    held = held.clone()                                    # tokens in order of segments; past each context: NaN
    at = np.cumsum([0] + need) * 16
    for i, (n, c) in enumerate(segs):
        held[:, :, at[i] + c:at[i + 1]] = gc.NAN_CODE if fp8 else float("nan")
    order = torch.randperm(sum(need), generator=g)
    pool = torch.empty((sum(need), 2, hkv, 16, d), dtype=held.dtype)
    pool[order] = held.reshape(2, hkv, sum(need), 16, d).permute(2, 0, 1, 3, 4)
    bt = torch.zeros((len(segs), max(need)), dtype=torch.int32)
    for i, n in enumerate(need):
        bt[i, :n] = order[at[i] // 16:at[i] // 16 + n].to(torch.int32)
    cu, cl = np.cumsum([0] + [n for n, _ in segs]).astype(np.int32), np.array([c for _, c in segs], np.int32)
    h = tetri.Tetri(hq, hkv, d, rows + 3, sum(need), max(need), len(segs))
    h.tetri_set_option("attn_variant", 3)
    pad = lambda t: torch.cat([t, torch.full((3, *t.shape[1:]), float("nan"), dtype=t.dtype)])
    dev = [t.to(gc.DEV) for t in (pad(q), pad(k), pad(v), pool, bt, torch.from_numpy(cu), torch.from_numpy(cl))]
    out = torch.full((rows + 3, hq, d), 7.0, dtype=torch.bfloat16, device=gc.DEV)
    h.tetri_chunk_prefill_planned(*dev, len(segs), d ** -0.5, 1, fp8, ks, vs, cu, cl, out)
    torch.cuda.synchronize()
    want = torch.zeros((rows + 3, hq, d), dtype=torch.float64)
    after = held.clone()
    for i, (n, c) in enumerate(segs):
        r = slice(int(cu[i]), int(cu[i + 1]))
        for head in range(hq):
            kh = head // (hq // hkv)
            s = q[r, head].double() @ torch.cat([past[0, kh, at[i]:at[i] + c].double(), k[r, kh].double()]).T * d ** -0.5
            s.masked_fill_(torch.arange(c + n)[None, :] > torch.arange(n)[:, None] + c, float("-inf"))
            want[r, head] = s.softmax(dim=1) @ torch.cat([past[1, kh, at[i]:at[i] + c].double(), v[r, kh].double()])
        for m, (new, s) in enumerate(((k, ks), (v, vs))):
            new = new[r].permute(1, 0, 2)
            after[m, :, at[i] + c:at[i] + c + n] = torch.from_numpy(ofp8.quantize(new.float().numpy(), s)) if fp8 else new
    gc.compare([out.cpu()], [want.numpy()], label=name)
    got = dev[3].cpu()[order].permute(1, 2, 0, 3, 4).reshape(after.shape)
    bits = torch.uint8 if fp8 else torch.int16
    assert torch.equal(got.view(bits), after.view(bits))
    h.close()
