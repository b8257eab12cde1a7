"""GPU parity of tetri_kv_export / tetri_kv_import and of their FP8 forms (through the C ABI) against the numpy oracle: bit-exact."""
import numpy as np
import pytest
import torch

from oracle import fp8 as ofp8, kv_transfer
from paper_2401_11181_amd import synth, tetri
import gpu_common as gc

pytestmark = pytest.mark.gpu
DEV = gc.DEV
P = 16


def make_case(lens, firsts, hkv, d, seed, spare_pages=5):
    """Random pool bits, distinct randomly placed pages for every request."""
    rng = np.random.default_rng(seed)
    need = [-(-(f + n) // P) for n, f in zip(lens, firsts)]
    mb = max(max(need), 1) + 1
    num_pages = sum(need) + spare_pages
    perm = rng.permutation(num_pages)
    bt = np.zeros((len(lens), mb), dtype=np.int32)
    at = 0
    for r, k in enumerate(need):
        bt[r, :k] = perm[at:at + k]
        at += k
    pool = rng.integers(0, 1 << 16, size=(num_pages, 2, hkv, P, d), dtype=np.uint16)
    cu = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    return pool, bt, cu, np.asarray(firsts, dtype=np.int32)


def handle_for(hkv, d, num_pages, mb):
    return tetri.Tetri(hkv, hkv, d, 64, num_pages, mb, 8)


def dev(a):
    if a.dtype == np.uint16:
        return torch.from_numpy(a.view(np.int16)).to(DEV)
    return torch.from_numpy(a).to(DEV)


def bits(t):
    return t.cpu().numpy().view(np.uint16)


def check_both_ways(lens, firsts, hkv, d, seed, pass_first=True):
    pool, bt, cu, first = make_case(lens, firsts, hkv, d, seed)
    h = handle_for(hkv, d, pool.shape[0], bt.shape[1])
    total = int(cu[-1])
    d_pool, d_bt, d_cu = dev(pool), dev(bt), dev(cu)
    d_first = dev(first) if pass_first else None
    buf = torch.full((max(2 * hkv * d * total, 8),), 0x5a5a, dtype=torch.int16, device=DEV)
    h.tetri_kv_export(d_pool, d_bt, d_cu, d_first, len(lens), total, buf)
    torch.cuda.synchronize()
    want = kv_transfer.kv_export(pool, bt, cu, first)
    assert np.array_equal(bits(buf)[:want.size], want)
    assert np.array_equal(bits(d_pool), pool), "export must not write the pool"
    # the receiver: other placement (reversed page order), sentinel contents
    bt2 = (pool.shape[0] - 1 - bt).astype(np.int32)
    sent = np.full(pool.shape, 0x1234, dtype=np.uint16)
    d_dst = dev(sent)
    h.tetri_kv_import(buf, dev(bt2), d_cu, d_first, len(lens), total, d_dst)
    torch.cuda.synchronize()
    ref = sent.copy()
    kv_transfer.kv_import(want, ref, bt2, cu, first)
    assert np.array_equal(bits(d_dst), ref)
    h.close()


CASES = {
    "ragged-request-level": ([1, 15, 16, 17, 63, 64, 65, 200], [0] * 8, 2, 128),
    "chunk-level-mid-page": ([40, 3, 129, 64], [5, 31, 16, 77], 3, 128),
    "d64": ([100, 1, 33], [0, 9, 48], 2, 64),
    "d64-one-head": ([70], [3], 1, 64),
    "five-heads": ([257, 30], [0, 100], 5, 128),
    "empty-requests-between": ([0, 20, 0, 0, 65, 0], [0, 0, 4, 0, 1, 0], 2, 128),
}


@pytest.mark.parametrize("name", sorted(CASES))
def test_transfer_cases(name):
    lens, firsts, hkv, d = CASES[name]
    check_both_ways(lens, firsts, hkv, d, seed=200 + sorted(CASES).index(name))


def test_null_first_tokens_means_zero():
    check_both_ways([33, 64, 2], [0, 0, 0], 2, 128, seed=230, pass_first=False)


def test_more_requests_than_one_lookup_step():
    """150 requests (the request lookup walks 64 at a time), some empty, some longer than a tile."""
    rng = np.random.default_rng(231)
    lens = [int(x) for x in rng.choice([0, 1, 7, 16, 64, 70, 130], size=150)]
    firsts = [int(x) for x in rng.integers(0, 20, size=150)]
    check_both_ways(lens, firsts, 2, 64, seed=232)


@pytest.mark.parametrize("n", [1, 2, 3, 4, 5, 63, 64, 65, 127, 128, 129])
@pytest.mark.parametrize("pass_first", [True, False])
def test_requests_at_the_edges_of_the_lookup(n, pass_first):
    """The prefix sum runs over as many lanes as a lookup step has requests: powers of two and their neighbours, one step
    and several, the last request (whose lane is the last that counts) never empty."""
    rng = np.random.default_rng(240 + n)
    lens = [int(x) for x in rng.choice([0, 1, 15, 16, 17, 40], size=n - 1)] + [33]
    firsts = [int(x) for x in rng.integers(0, 20, size=n)] if pass_first else [0] * n
    check_both_ways(lens, firsts, 2, 128, seed=260 + n, pass_first=pass_first)


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("n", [1, 2, 5, 63, 64, 65, 129])
def test_fp8_requests_at_the_edges_of_the_lookup(n, d):
    """The quantising export and the import of its codes, one lookup step and several, first tokens inside a page, empty
    requests, and three kv heads, so that K ends inside a run of slabs.  Codes and the receiver's pool bit for bit."""
    hkv, k_scale, v_scale = 3, 0.0137, 0.31
    rng = np.random.default_rng(270 + n)
    lens = [int(x) for x in rng.choice([0, 1, 15, 16, 17, 33], size=n - 1)] + [40]
    firsts = [int(x) for x in rng.integers(1, 16, size=n)]
    pool, bt, cu, first = make_case(lens, firsts, hkv, d, seed=280 + n)
    values = (np.arange(65536, dtype=np.uint32) << 16).view(np.float32)
    pool[np.isnan(values)[pool]] = 0x3F80                    # (a NaN has no defined code)
    values[np.isnan(values)] = 1.0
    codes = np.empty(pool.shape, dtype=np.uint8)             # the code of every bf16 value, once for K's scale and once for V's
    for half, scale in enumerate((k_scale, v_scale)):
        codes[:, half] = ofp8.quantize(values, scale)[pool[:, half]]
    want = kv_transfer.kv_export(codes, bt, cu, first)
    if n <= 2:
        assert np.array_equal(want, kv_transfer.kv_export_fp8(values[pool], bt, cu, first, k_scale, v_scale))
    h = handle_for(hkv, d, pool.shape[0], bt.shape[1])
    total = int(cu[-1])
    d_pool, d_cu, d_first = dev(pool), dev(cu), dev(first)
    buf = torch.full((want.size + 64,), 0x5a, dtype=torch.uint8, device=DEV)
    h.tetri_kv_export_fp8(d_pool, dev(bt), d_cu, d_first, n, total, k_scale, v_scale, buf)
    torch.cuda.synchronize()
    got = buf.cpu().numpy()
    assert np.array_equal(got[:want.size], want) and (got[want.size:] == 0x5a).all()
    assert np.array_equal(bits(d_pool), pool), "export must not write the pool"
    bt2 = (pool.shape[0] - 1 - bt).astype(np.int32)
    ref = np.full(pool.shape, 0x12, dtype=np.uint8)
    d_dst = dev(ref.copy())
    h.tetri_kv_import_fp8(buf, dev(bt2), d_cu, d_first, n, total, d_dst)
    torch.cuda.synchronize()
    kv_transfer.kv_import(want, ref, bt2, cu, first)
    assert np.array_equal(d_dst.cpu().numpy(), ref)
    h.close()


def test_many_tokens_several_slabs_per_workgroup():
    """Enough tiles that a workgroup takes more than one (K / V, head) slab."""
    check_both_ways([5000, 3000, 4097, 2500, 3333], [0, 16, 5, 0, 1], 3, 64, seed=233)


def test_zero_tokens_launches_nothing():
    pool, bt, cu, first = make_case([0, 0], [0, 0], 2, 128, seed=234)
    h = handle_for(2, 128, pool.shape[0], bt.shape[1])
    d_pool = dev(pool)
    h.tetri_kv_export(d_pool, dev(bt), dev(cu), None, 2, 0, None)
    h.tetri_kv_import(None, dev(bt), dev(cu), None, 2, 0, d_pool)
    torch.cuda.synchronize()
    assert np.array_equal(bits(d_pool), pool)
    h.close()


def test_argument_errors():
    pool, bt, cu, first = make_case([20], [0], 2, 128, seed=235)
    h = handle_for(2, 128, pool.shape[0], bt.shape[1])
    d_pool, d_bt, d_cu = dev(pool), dev(bt), dev(cu)
    buf = torch.zeros(2 * 2 * 128 * 20 + 8, dtype=torch.int16, device=DEV)
    for bad in (lambda: h.tetri_kv_export(None, d_bt, d_cu, None, 1, 20, buf),
                lambda: h.tetri_kv_export(d_pool, None, d_cu, None, 1, 20, buf),
                lambda: h.tetri_kv_export(d_pool, d_bt, None, None, 1, 20, buf),
                lambda: h.tetri_kv_export(d_pool, d_bt, d_cu, None, 0, 20, buf),
                lambda: h.tetri_kv_export(d_pool, d_bt, d_cu, None, 1, -1, buf),
                lambda: h.tetri_kv_export(d_pool, d_bt, d_cu, None, 1, bt.shape[1] * P + 1, buf),
                lambda: h.tetri_kv_export(d_pool, d_bt, d_cu, None, 1, 20, None),
                lambda: h.tetri_kv_export(d_pool, d_bt, d_cu, None, 1, 20, buf[1:]),
                lambda: h.tetri_kv_import(buf[1:], d_bt, d_cu, None, 1, 20, d_pool),
                lambda: h.tetri_kv_import(buf, d_bt, d_cu, None, 1, 20, None)):
        with pytest.raises(tetri.TetriError) as e:
            bad()
        assert e.value.status == tetri.TETRI_ERR_INVALID_ARG
    torch.cuda.synchronize()
    assert np.array_equal(bits(d_pool), pool)
    h.close()


def test_export_after_prefill_is_k_and_v_of_every_request(oracle):
    """The cache that the chunked prefill built on the GPU, exported request-level (the granularity the
    paper implements) and chunk-level: the closed form [Hkv][n][D] of the inputs, and the oracle."""
    w = synth.small("xfer-prefill", [150, 40, 7, 300], 128, 4, 2, 128, seed=236)
    qs, ks, vs, tables = gc.workload_tensors(w)
    _, pool, sess, _ = gc.gpu_prefill(w, qs, ks, vs, tables, fused=True)
    mb = max(len(t) for t in tables)
    bt = np.zeros((len(tables), mb), dtype=np.int32)
    for r, t in enumerate(tables):
        bt[r, :len(t)] = t
    cu = np.concatenate([[0], np.cumsum(w.prompt_lens)]).astype(np.int32)
    total = int(cu[-1])
    hkv, d = w.num_kv_heads, w.head_dim
    h = handle_for(hkv, d, w.num_pages, mb)
    buf = torch.zeros(2 * hkv * d * total, dtype=torch.int16, device=DEV)
    h.tetri_kv_export(pool, dev(bt), dev(cu), None, len(tables), total, buf)
    torch.cuda.synchronize()
    got = bits(buf)
    for r, n in enumerate(w.prompt_lens):
        block = got[2 * hkv * d * cu[r]: 2 * hkv * d * cu[r + 1]].reshape(2, hkv, n, d)
        assert np.array_equal(block[0], ks[r].view(torch.int16).numpy().view(np.uint16).transpose(1, 0, 2))
        assert np.array_equal(block[1], vs[r].view(torch.int16).numpy().view(np.uint16).transpose(1, 0, 2))
    assert np.array_equal(got, kv_transfer.kv_export(bits(pool.view(torch.int16)), bt, cu))
    # chunk-level: the attention call's own metadata arrays name the slice each chunk produced
    dst = torch.full_like(pool.view(torch.int16), 0x0777)
    for c in range(sess.n_chunks):
        segs = sess.chunk_segments(c)
        n_real = sum(n for _, _, n in segs)
        d_cu, d_ctx, d_bt, _ = sess.meta[c]
        piece = torch.zeros(2 * hkv * d * n_real, dtype=torch.int16, device=DEV)
        h.tetri_kv_export(pool, d_bt, d_cu, d_ctx, len(segs), n_real, piece)
        h.tetri_kv_import(piece, d_bt, d_cu, d_ctx, len(segs), n_real, dst)
    torch.cuda.synchronize()
    ref = np.full(bits(dst).shape, 0x0777, dtype=np.uint16)
    kv_transfer.kv_import(got, ref, bt, cu)
    assert np.array_equal(bits(dst), ref)
    h.close()


def test_opt13b_request_level_full_size():
    """The benchmark configuration: one 2048-token request, 40 heads x 128: every element."""
    w = synth.workload("opt13b")
    n = w.prompt_lens[0]
    pool, bt, cu, first = make_case([n], [0], w.num_kv_heads, w.head_dim, seed=237, spare_pages=3)
    h = handle_for(w.num_kv_heads, w.head_dim, pool.shape[0], bt.shape[1])
    buf = torch.zeros(2 * w.num_kv_heads * w.head_dim * n, dtype=torch.int16, device=DEV)
    h.tetri_kv_export(dev(pool), dev(bt), dev(cu), None, 1, n, buf)
    torch.cuda.synchronize()
    assert np.array_equal(bits(buf), kv_transfer.kv_export(pool, bt, cu))
    h.close()
