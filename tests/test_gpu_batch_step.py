"""A batch's step in one call (tetri_batch_step), whose first launch brings the metadata of all of them where it can: bit for bit what
tetri_batch_upload followed by tetri_batch_launch leaves in the output, the pool and the metadata, for plans on both sides of the
sizes at which they stop fitting the first launch's arguments (672 int32) and the upload's (896), for first chunks that go to other kernels, with padding rows."""
import numpy as np
import pytest
import torch

from paper_2401_11181_amd import synth, tetri
from paper_2401_11181_amd.prefill import PrefillPipeline
import gpu_common as gc

pytestmark = pytest.mark.gpu

# prompts, chunk size, heads, kv heads, head dim, entries added to every block-table row, "attn_variant"
CASES = {
    "one-chunk": ([60], 64, 4, 4, 64, 0, 0),                          # 12 int32
    "small": ([70, 33, 150], 64, 4, 4, 64, 0, 0),
    "split": ([300], 64, 2, 1, 128, 0, 0),                            # keys split over workgroups in later chunks
    "eight-wavefronts": ([300, 90], 256, 32, 8, 128, 0, 3),
    "first-launch-full": ([512], 128, 8, 2, 128, 128, 0),             # 4 chunks x (8 + 160) = 672 int32
    "one-more": ([512], 128, 8, 2, 128, 129, 0),
    "own-launch-full": ([512], 128, 8, 2, 128, 184, 0),               # 4 x (8 + 216) = 896
    "staged": ([512], 128, 8, 2, 128, 188, 0),
    "shared-tiles": ([260, 70], 128, 4, 4, 128, 0, 2),                # no launch of the short kernel
}


@pytest.mark.parametrize("fused", [True, False], ids=["fused", "two-launches"])
@pytest.mark.parametrize("name", sorted(CASES))
def test_step_is_upload_and_launch(name, fused):
    lens, chunk, hq, hkv, d, spare, variant = CASES[name]
    w = synth.small("step-" + name, lens, chunk, hq, hkv, d, seed=960)
    tables = [[int(p) for p in t] + [0] * spare for t in synth.place_pages(w)]
    pipe = PrefillPipeline(lens, None, chunk, hq, hkv, d, w.num_pages, tables, w.scale, device=gc.DEV, fused=fused)
    if variant:
        pipe.handle.tetri_set_option("attn_variant", variant)
    if name in ("first-launch-full", "own-launch-full"):
        assert pipe.meta_len == (672 if name == "first-launch-full" else 896)
    g = torch.Generator(device=gc.DEV).manual_seed(961)
    rnd = lambda *s: torch.randn(s, device=gc.DEV, generator=g).to(torch.bfloat16)
    n = pipe.n_chunks
    q, k, v = rnd(n, chunk, hq, d), rnd(n, chunk, hkv, d), rnd(n, chunk, hkv, d)
    pool, out = torch.zeros((w.num_pages, 2, hkv, 16, d), dtype=torch.bfloat16, device=gc.DEV), torch.empty_like(q)
    pipe.bind(q, k, v, pool, out)
    got = []
    for step in (pipe.step, lambda: (pipe.batch.upload(*pipe._plan_args, None), pipe._launch_all()), pipe.step):
        pool.zero_()
        out.fill_(7.0)
        pipe.meta_dev.fill_(-9)
        step()
        torch.cuda.synchronize()
        got.append((pool.clone(), out.clone(), pipe.meta_dev.clone()))
    for pool_, out_, meta in (got[0], got[2]):
        assert torch.equal(pool_.view(torch.int16), got[1][0].view(torch.int16))
        assert torch.equal(out_.view(torch.int16), got[1][1].view(torch.int16))
        want = np.zeros(pipe.meta_len, np.int32), np.zeros((n, 4), np.int32)
        tetri.tetri_plan_metadata(pipe.lens, None, chunk, pipe.req_bt, *want)
        for at, x in ((meta.cpu().numpy(), want[0]), (got[1][2].cpu().numpy(), want[0])):
            for o_cu, o_ctx, o_bt, S in want[1]:
                for first, count in ((o_cu, S + 1), (o_ctx, S), (o_bt, S * pipe.max_blocks)):
                    assert np.array_equal(at[first:first + count], x[first:first + count])


# 16-bit rows of head_dim 128, 4 MB or more of them in a next chunk, and places for as much beside a chunk's row blocks: that launch asks for
# rows of the next chunk.  prompts, chunk size, heads, kv heads
AHEAD = {
    "ragged": ([200, 312, 139], 512, 40, 40),                         # the first launch brings the metadata; 139 rows of 10 KB: whole KBs
    "gqa": ([100, 412, 511], 512, 32, 8),
    "odd-kb": ([150, 362, 301, 211, 333], 512, 36, 9),                # 301 + 211 and 333 rows of 2304 bytes of K: 333 rows end inside a KB
    "staged": ([60] * 8 + [32] + [200] * 5, 512, 40, 40),             # a plan that the first launch cannot bring
    "eight-wavefronts": ([480], 160, 40, 40),
    "past-the-caches": ([250] * 53, 512, 40, 40),                     # more than 256 MB of new K and V in a call: stored otherwise than in calls of one chunk
}


@pytest.mark.parametrize("fused", [True, False], ids=["fused", "two-launches"])
@pytest.mark.parametrize("name", sorted(AHEAD))
def test_rows_asked_for_ahead_change_nothing(name, fused):
    """Against the same chunks launched one to a call, which know of no next chunk."""
    lens, chunk, hq, hkv = AHEAD[name]
    d = 128
    w = synth.small("ahead-" + name, lens, chunk, hq, hkv, d, seed=970)
    spare = 64 if name == "staged" else 0
    tables = [[int(p) for p in t] + [0] * spare for t in synth.place_pages(w)]
    pipe = PrefillPipeline(lens, None, chunk, hq, hkv, d, w.num_pages, tables, w.scale, device=gc.DEV, fused=fused)
    pipe.handle.tetri_set_option("attn_variant", 3)
    rows = [sum(n for _r, _s, n in pipe.chunk_segments(c)) for c in range(pipe.n_chunks)]
    assert max(rows[1:]) * (hq + 2 * hkv) * d * 2 >= 4 << 20
    assert (pipe.meta_len > 672) == (name in ("staged", "past-the-caches"))
    if name == "odd-kb":
        assert any(r * hkv * d * 2 % 1024 for r in rows[1:])
    g = torch.Generator(device=gc.DEV).manual_seed(971)
    rnd = lambda *s: torch.randn(s, device=gc.DEV, generator=g).to(torch.bfloat16)
    n = pipe.n_chunks
    q, k, v = rnd(n, chunk, hq, d), rnd(n, chunk, hkv, d), rnd(n, chunk, hkv, d)
    out = torch.empty_like(q)
    pool = torch.zeros((w.num_pages, 2, hkv, 16, d), dtype=torch.bfloat16, device=gc.DEV)
    pipe.bind(q, k, v, pool, out)

    def one_by_one():
        pipe.batch.upload(*pipe._plan_args, None)
        for c in range(pipe.n_chunks):
            pipe.batch.launch(pipe.layout_np, c, 1, *pipe._batch_args, pipe._mode, None)

    got = []
    for step in (one_by_one, pipe.step, lambda: (pipe.batch.upload(*pipe._plan_args, None), pipe._launch_all()), pipe.step):
        pool.zero_()
        out.fill_(7.0)
        pipe.meta_dev.fill_(-9)
        step()
        torch.cuda.synchronize()
        got.append((pool.clone().view(torch.int16), out.clone().view(torch.int16)))
    for other in got[1:]:
        assert torch.equal(got[0][0], other[0]) and torch.equal(got[0][1], other[1])


def test_metadata_is_sent_where_the_launch_is_refused():
    """An error before the first launch leaves the plan on the device, as the two calls do."""
    w = synth.small("step-refused", [70, 33], 64, 4, 4, 64, seed=962)
    pipe = PrefillPipeline(w.prompt_lens, None, 64, 4, 4, 64, w.num_pages, synth.place_pages(w), w.scale, device=gc.DEV)
    t = torch.zeros((pipe.n_chunks, 64, 4, 64), dtype=torch.bfloat16, device=gc.DEV)
    pool = torch.zeros((w.num_pages, 2, 4, 16, 64), dtype=torch.bfloat16, device=gc.DEV)
    pipe.bind(t, t, t, pool, torch.zeros_like(t))
    pipe.meta_dev.fill_(-9)
    args = list(pipe._batch_args)
    args[5] = float("nan")
    with pytest.raises(tetri.TetriError) as e:
        pipe.batch.step(*pipe._plan_args, *args, tetri.BATCH_FUSED, None)
    assert "scale" in str(e.value)
    torch.cuda.synchronize()
    assert (pipe.meta_dev != -9).any()
