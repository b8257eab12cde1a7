"""The staging ring of a repeatable step (tetri_batch_*): every upload carries the plan of its own step, whatever the
turn of the ring and the stream, and host metadata that is no chunk of the handle is rejected."""
import numpy as np
import pytest
import torch

from paper_2401_11181_amd import synth, tetri
from paper_2401_11181_amd.prefill import ChunkedPrefill, PrefillPipeline

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("one_stream", [True, False])
def test_ring_uploads_the_plan_of_every_step(one_stream):
    w = synth.small("ring", [70, 33, 150], 64, 4, 4, 64, seed=5)
    pipe = PrefillPipeline(w.prompt_lens, [0, 1, 2], 64, 4, 4, 64, w.num_pages, synth.place_pages(w), w.scale, device=DEV)
    streams = [torch.cuda.Stream(device=DEV) for _ in range(1 if one_stream else 3)]
    orders = [[0, 1, 2], [2, 1, 0], [1, 0, 2], [1, 2, 0]]
    got, want = [], []
    for step in range(3 * tetri.lib().tetri_batch_slots() + 3):
        pipe.order[:] = orders[step % 4]
        st = streams[(step // 3) % len(streams)]
        st.wait_stream(streams[((step - 1) // 3) % len(streams)])     # (one metadata buffer: the copies stay in order)
        pipe.batch.upload(*pipe._plan_args, st)
        with torch.cuda.stream(st):
            got.append(pipe.meta_dev.clone())
        meta, layout = np.zeros(pipe.meta_len, np.int32), np.zeros((pipe.n_chunks, 4), np.int32)
        tetri.tetri_plan_metadata(pipe.lens, pipe.order, 64, pipe.req_bt, meta, layout)
        want.append((meta, layout))
    torch.cuda.synchronize()
    for g, (meta, layout) in zip(got, want):
        g = g.cpu().numpy()
        for o_cu, o_ctx, o_bt, S in layout:
            for at, n in ((o_cu, S + 1), (o_ctx, S), (o_bt, S * pipe.max_blocks)):
                assert np.array_equal(g[at:at + n], meta[at:at + n])


@pytest.mark.parametrize("spare", [0, 300], ids=["in-the-arguments", "staged"])
def test_ring_waits_for_uploads_that_have_not_run(spare):
    """More uploads than the ring has buffers while the stream is still busy with other work: a buffer is not written again
    before its upload has run, so every plan arrives.  (Block tables with room to spare make the plan too large for the
    upload kernel's arguments.)"""
    w = synth.small("ring-busy", [70, 33, 150], 64, 4, 4, 64, seed=5)
    tables = [[int(p) for p in t] + [0] * spare for t in synth.place_pages(w)]
    pipe = PrefillPipeline(w.prompt_lens, [0, 1, 2], 64, 4, 4, 64, w.num_pages, tables, w.scale, device=DEV)
    assert (pipe.meta_len > 896) == (spare > 0)
    big = torch.randn(8192, 8192, device=DEV).to(torch.bfloat16)
    acc = torch.empty_like(big)
    torch.matmul(big, big, out=acc)
    st = torch.cuda.Stream(device=DEV)
    torch.cuda.synchronize()
    orders, got, want = [[0, 1, 2], [2, 1, 0], [1, 0, 2], [1, 2, 0], [2, 0, 1]], [], []
    with torch.cuda.stream(st):
        for _ in range(40):                                 # some ten milliseconds of work ahead of the uploads
            torch.matmul(big, big, out=acc)
        for step in range(2 * tetri.lib().tetri_batch_slots() + 3):
            pipe.order = orders[step % 5]
            pipe.batch.upload(*pipe._plan_args, st)
            got.append(pipe.meta_dev.clone())
            meta, layout = np.zeros(pipe.meta_len, np.int32), np.zeros((pipe.n_chunks, 4), np.int32)
            tetri.tetri_plan_metadata(pipe.lens, pipe.order, 64, pipe.req_bt, meta, layout)
            want.append((meta, layout))
            if step == 0:
                assert not st.query(), "the stream should still be busy"
    torch.cuda.synchronize()
    for g, (meta, layout) in zip(got, want):
        g = g.cpu().numpy()
        for o_cu, o_ctx, o_bt, S in layout:
            for at, n in ((o_cu, S + 1), (o_ctx, S), (o_bt, S * pipe.max_blocks)):
                assert np.array_equal(g[at:at + n], meta[at:at + n])


@pytest.mark.parametrize("table", [1, 2, 3, 4, 5, 244, 247, 248, 249, 252, 253, 884, 887, 888, 889, 892, 893, 1500])
def test_uploads_of_every_length(table):
    """Plans around the sizes at which the upload changes its form (256 and 896 int32): what arrives is the plan, and nothing
    behind it is written."""
    n = min(16 * table, 60)
    tables = [list(range(table))]
    pipe = PrefillPipeline([n], None, 64, 4, 4, 64, table, tables, 0.1, device=DEV)
    pipe.req_bt[0] = np.random.default_rng(table).permutation(table)
    dev = torch.full((pipe.meta_len + 64,), -5, dtype=torch.int32, device=DEV)
    batch = tetri.Batch(pipe.handle, pipe.meta_len, dev)
    for _ in range(3):
        batch.upload(*pipe._plan_args, None)
    torch.cuda.synchronize()
    meta, layout = np.full(pipe.meta_len, -7, np.int32), np.zeros((1, 4), np.int32)
    tetri.tetri_plan_metadata(pipe.lens, None, 64, pipe.req_bt, meta, layout)
    got = dev.cpu().numpy()
    o_cu, o_ctx, o_bt, S = layout[0]
    for at, ln in ((o_cu, S + 1), (o_ctx, S), (o_bt, S * table)):
        assert np.array_equal(got[at:at + ln], meta[at:at + ln])
    assert (got[pipe.meta_len:] == -5).all()


@pytest.mark.parametrize("cu, ctx", [([0, 40, 40], [0, 0]), ([1, 40, 64], [0, 0]), ([0, 40, 65], [0, 0]), ([0, 40, 64], [0, -1]),
                                     ([0, 40, 64], [0, 100])])
def test_planned_launch_rejects_host_metadata_that_is_no_chunk(cu, ctx):
    w = synth.small("bad", [40, 90], 64, 4, 4, 64, seed=6)
    s = ChunkedPrefill(w.prompt_lens, None, 64, 4, 4, 64, w.num_pages, synth.place_pages(w), device=DEV)
    z = torch.zeros((64, 4, 64), dtype=torch.bfloat16, device=DEV)
    pool = torch.zeros((w.num_pages, 2, 4, 16, 64), dtype=torch.bfloat16, device=DEV)
    dcu, dctx, dbt, S = s.meta[0]
    assert S == 2
    with pytest.raises(tetri.TetriError) as e:
        s.handle.tetri_chunk_prefill_planned(z, z, z, pool, dbt, dcu, dctx, S, 0.1, 1, 0, 1.0, 1.0, np.array(cu, np.int32),
                                             np.array(ctx, np.int32), torch.zeros_like(z))
    assert e.value.status == tetri.TETRI_ERR_INVALID_ARG and "host metadata" in str(e.value)
