"""The host side of prefill.py without a GPU: a step plans from what the pipeline's attributes hold at that moment, and a
chunk's launch uses the metadata that `meta` holds at that moment.  The handle and the staging ring are stand-ins; the
plan is made by the C library from the arguments they are given."""
import ctypes
import gc

import numpy as np
import pytest
import torch

from paper_2401_11181_amd import prefill, synth, tetri


class Recorder:
    """A handle that writes down its calls."""
    def __init__(self, *_args, **_kw):
        self.h, self.calls = None, []

    def __getattr__(self, name):
        return lambda *args: self.calls.append((name, args))


class Ring:
    """A staging ring: upload and step plan into a buffer as tetri_batch_upload and tetri_batch_step do, from the arguments' addresses."""
    def __init__(self, handle, meta_len, _meta_dev):
        self.meta = np.zeros(meta_len, np.int32)
        self.slots = [self.meta]
        self.max_blocks = handle.max_blocks

    def upload(self, lens, n, order, n_order, req_bt, layout, n_chunks, _stream):
        at = lambda a: None if a is None else ctypes.c_void_p(a if isinstance(a, int) else a.ctypes.data)
        got = tetri.lib().tetri_plan_metadata(at(lens), n, at(order), n_order, 64, at(req_bt), self.max_blocks, at(self.meta),
                                              self.meta.size, at(layout), n_chunks, ctypes.byref(ctypes.c_int64()))
        assert got == n_chunks

    def launch(self, *_args):
        pass

    def step(self, lens, n, order, n_order, req_bt, layout, n_chunks, *_launch_args):
        self.upload(lens, n, order, n_order, req_bt, layout, n_chunks, None)


@pytest.fixture(params=["one call", "upload and launch"])
def pipe(request, monkeypatch):
    monkeypatch.setattr(tetri, "Batch", Ring)
    w = synth.small("host-step", [70, 33, 150], 64, 4, 4, 64, seed=5)
    handle = Recorder()
    handle.max_blocks = max(len(t) for t in synth.place_pages(w))
    p = prefill.PrefillPipeline(w.prompt_lens, [0, 1, 2], 64, 4, 4, 64, w.num_pages, synth.place_pages(w), w.scale, device="cpu",
                                handle=handle)
    t = torch.zeros((p.n_chunks, 1))
    p.bind(t, t, t, t, t)
    if request.param != "one call":                      # (what a step with a graph or with chunks exported inside does)
        p.step = lambda: (p.batch.upload(*p._plan_args, None), p._launch_all())
    return p


def planned(pipe):
    meta, layout = np.zeros(pipe.meta_len, np.int32), np.zeros((pipe.n_chunks, 4), np.int32)
    tetri.tetri_plan_metadata(pipe.lens, pipe.order, 64, pipe.req_bt, meta, layout)
    return [meta[at:at + n].tolist() for o_cu, o_ctx, o_bt, S in layout
            for at, n in ((o_cu, S + 1), (o_ctx, S), (o_bt, S * pipe.max_blocks))]


CHANGES = {
    "nothing": lambda p: None,
    "order in place": lambda p: p.order.__setitem__(slice(None), [2, 0, 1]),
    "order": lambda p: setattr(p, "order", np.array([1, 2, 0], np.int32)),
    "order, a list": lambda p: setattr(p, "order", [2, 1, 0]),
    "no order": lambda p: setattr(p, "order", None),
    "lens, 64-bit": lambda p: setattr(p, "lens", np.array([33, 70, 150], np.int64)),
    "block table": lambda p: setattr(p, "req_bt", p.req_bt + 1),
    "block table, strided": lambda p: setattr(p, "req_bt", np.repeat(p.req_bt + 2, 2, axis=1)[:, ::2]),
    "layout": lambda p: setattr(p, "layout_np", np.zeros_like(p.layout_np)),
}


@pytest.mark.parametrize("name", sorted(CHANGES))
def test_step_plans_from_the_attributes_of_the_moment(pipe, name):
    CHANGES[name](pipe)
    gc.collect()
    keep = [np.full(pipe.req_bt.shape, 99, np.int32) for _ in range(20)]     # (takes the place of what has been freed)
    pipe.step()
    got = [pipe.batch.meta[at:at + n].tolist() for o_cu, o_ctx, o_bt, S in pipe.layout_np
           for at, n in ((o_cu, S + 1), (o_ctx, S), (o_bt, S * pipe.max_blocks))]
    assert got == planned(pipe) and len(keep) == 20


@pytest.mark.parametrize("table", [lambda t: t[:, :-1], lambda t: t[:2], lambda t: t[0]], ids=["narrow", "short", "flat"])
def test_block_tables_of_another_shape_are_refused(pipe, table):
    pipe.req_bt = table(pipe.req_bt)
    with pytest.raises(ValueError):
        pipe.step()


@pytest.mark.parametrize("call, general", [
    (lambda s: s.attn(1, 0, 0, 0, 0, 0.1, 0), "tetri_chunk_prefill_attn"),
    (lambda s: s.attn_append(1, 0, 0, 0, 0, 0.1, 0), "tetri_chunk_prefill_attn_append"),
    (lambda s: s.attn_fp8(1, 0, 0, 0, 0, 0.1, 0.2, 0.3, 1, 0), "tetri_chunk_prefill_attn_fp8"),
    (lambda s: s.append(1, 0, 0, 0), "tetri_kv_append")], ids=["attn", "attn_append", "attn_fp8", "append"])
@pytest.mark.parametrize("change", ["nothing", "replaced", "written"])
def test_launch_uses_the_metadata_of_the_moment(monkeypatch, call, general, change):
    monkeypatch.setattr(tetri, "Tetri", Recorder)
    w = synth.small("host-chunk", [70, 33, 150], 64, 4, 4, 64, seed=5)
    s = prefill.ChunkedPrefill(w.prompt_lens, None, 64, 4, 4, 64, w.num_pages, synth.place_pages(w), device="cpu")
    if change == "replaced":
        cu, ctx, bt, S = s.meta[1]
        s.meta[1] = (cu.clone(), ctx.clone() + 1, bt.clone(), S)
    elif change == "written":
        s.meta[1][1].add_(1)
    call(s)
    name, args = s.handle.calls[-1]
    assert name == (general if change != "nothing" or general == "tetri_kv_append" else "tetri_chunk_prefill_planned")
    cu, ctx, bt, S = s.meta[1]
    assert any(isinstance(a, int) and a == S for a in args)
    for t in (cu, ctx, bt):
        assert any((isinstance(a, torch.Tensor) and a.data_ptr() == t.data_ptr()) or (isinstance(a, int) and a == t.data_ptr()) for a in args)
