// Host layer of libtetri: handle, argument checks, launch shapes and the debug validator.
// (The chunk packer and the scheduler are in tetri_plan.cpp, which needs no HIP.)
#include <algorithm>
#include <climits>
#include <cmath>
#include <cstdarg>
#include <cstdio>
#include <cstring>
#include <functional>
#include <new>
#include <vector>

#include "tetri_internal.h"
#include "tetri_plan.h"

namespace {

tetri_status fail(tetri_ctx *h, tetri_status st, const char *fmt, ...)
{
    char buf[512];
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(buf, sizeof buf, fmt, ap);
    va_end(ap);
    if (h) h->err = buf; else tetri_set_thread_error(buf);
    return st;
}

bool aligned16(const void *p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }

// Query-head grouping of a workgroup: its 4 (host's division: 8) row/head slots are
// (hpw heads that share a kv head) x (rb blocks of 32 rows).
void wave_grouping(int g, int slots, int *hpw, int *rb)
{
    if (g % 4 == 0) *hpw = 4;
    else if (g % 2 == 0) *hpw = 2;
    else *hpw = 1;
    *rb = slots / *hpw;
}

// Upper bound of the number of row tiles of a chunk: each of the S segments and the padding
// range may end in a partial tile.
int tile_bound(int C, int S, int BM) { return (C + (S + 1) * (BM - 1)) / BM; }

}  // namespace

extern "C" {

int32_t tetri_abi_version(void) { return 1; }

const char *tetri_last_error(const tetri_ctx *ctx)
{
    return ctx ? ctx->err.c_str() : tetri_thread_error();
}

tetri_status tetri_create(const tetri_config *c, tetri_ctx **out)
{
    if (!c || !out) return fail(nullptr, TETRI_ERR_INVALID_ARG, "tetri_create: null argument");
    *out = nullptr;
    if (c->num_q_heads < 1 || c->num_kv_heads < 1 || c->num_q_heads % c->num_kv_heads != 0)
        return fail(nullptr, TETRI_ERR_INVALID_ARG, "tetri_create: num_q_heads=%d must be a positive multiple of num_kv_heads=%d",
                    c->num_q_heads, c->num_kv_heads);
    if (c->chunk_size < 1 || c->num_pages < 1 || c->max_blocks_per_seq < 1 || c->max_segs_per_chunk < 1)
        return fail(nullptr, TETRI_ERR_INVALID_ARG, "tetri_create: chunk_size, num_pages, max_blocks_per_seq and max_segs_per_chunk must be positive");
    if (c->max_segs_per_chunk > c->chunk_size)
        return fail(nullptr, TETRI_ERR_INVALID_ARG, "tetri_create: max_segs_per_chunk=%d exceeds chunk_size=%d (segments are non-empty)",
                    c->max_segs_per_chunk, c->chunk_size);
    if (c->head_dim != 64 && c->head_dim != 128)
        return fail(nullptr, TETRI_ERR_UNSUPPORTED, "tetri_create: head_dim=%d (supported: 64, 128)", c->head_dim);
    if (c->page_size != 16)
        return fail(nullptr, TETRI_ERR_UNSUPPORTED, "tetri_create: page_size=%d (supported: 16)", c->page_size);
    if (c->dtype != TETRI_BF16)
        return fail(nullptr, TETRI_ERR_UNSUPPORTED, "tetri_create: dtype=%d (supported: TETRI_BF16)", c->dtype);
    int ndev = 0;
    hipError_t e = hipGetDeviceCount(&ndev);
    if (e != hipSuccess || ndev < 1)
        return fail(nullptr, TETRI_ERR_HIP, "tetri_create: no usable HIP device (%s)", e == hipSuccess ? "device count is 0" : hipGetErrorString(e));
    tetri_ctx *h = new (std::nothrow) tetri_ctx;
    if (!h) return fail(nullptr, TETRI_ERR_NOMEM, "tetri_create: out of host memory");
    h->cfg = *c;
    // Scratch memory for launches that divide the stages of a head group evenly over workgroups: such
    // a launch has at most one workgroup per CU, 4 (row block, head) slots each, and a workgroup leaves at
    // most two partial results per slot (its first and its last job); a partial result is O (32 x head_dim
    // floats), m and the row sum.  Arrival counters: one per (head group, row tile, slot), fewer than two
    // tiles per CU in such a launch; several sets, used in turn.  As much twice more for launches on a division of the
    // host's, whose kernels are for head_dim 128.
    hipDeviceProp_t prop;
    if ((e = hipGetDevice(&h->device)) != hipSuccess || (e = hipGetDeviceProperties(&prop, h->device)) != hipSuccess) {
        delete h;
        return fail(nullptr, TETRI_ERR_HIP, "tetri_create: %s", hipGetErrorString(e));
    }
    h->num_cus = prop.multiProcessorCount;
    h->scratch_units = (size_t)h->num_cus * 4;
    h->unit_bytes = (size_t)32 * c->head_dim * 4 + 2 * 32 * 4;
    h->n_counters = (int32_t)(2 * h->scratch_units);
    const size_t copies = c->head_dim == 128 ? 3 : 1, scratch_bytes = 2 * h->scratch_units * h->unit_bytes;
    const size_t set_bytes = kCounterSets * (size_t)h->n_counters * sizeof(int32_t), counter_bytes = set_bytes + 256 + (copies - 1) * set_bytes;
    if ((e = hipMalloc(reinterpret_cast<void **>(&h->scratch), copies * scratch_bytes)) != hipSuccess ||
        (e = hipMalloc(reinterpret_cast<void **>(&h->counters), counter_bytes)) != hipSuccess ||
        (e = hipMemset(h->counters, 0, counter_bytes)) != hipSuccess ||
        (e = hipEventCreateWithFlags(&h->plan_done, hipEventDisableTiming)) != hipSuccess) {
        tetri_destroy(h);
        return fail(nullptr, TETRI_ERR_HIP, "tetri_create: scratch memory: %s", hipGetErrorString(e));
    }
    for (size_t i = 1; i < copies; ++i) {
        h->plan_memory[i - 1].scratch = h->scratch + i * scratch_bytes;
        h->plan_memory[i - 1].counters = h->counters + (256 + i * set_bytes) / sizeof(int32_t);
    }
    // the static memory of tetri_decode_attn_static: its addresses on this device, looked up here so that the
    // entry point itself makes no runtime call besides the launch
    if ((e = tetri_decode_static_memory(&h->decode_static)) != hipSuccess) {
        tetri_destroy(h);
        return fail(nullptr, TETRI_ERR_HIP, "tetri_create: static scratch array: %s", hipGetErrorString(e));
    }
    *out = h;
    return TETRI_OK;
}

void tetri_destroy(tetri_ctx *ctx)
{
    if (!ctx) return;
    if (ctx->scratch) (void)hipFree(ctx->scratch);
    if (ctx->counters) (void)hipFree(ctx->counters);
    if (ctx->plan_lent) (void)hipEventSynchronize(ctx->plan_done);
    if (ctx->plan_done) (void)hipEventDestroy(ctx->plan_done);
    delete ctx;
}

tetri_status tetri_set_option(tetri_ctx *ctx, const char *key, int32_t value)
{
    if (!ctx || !key) return fail(ctx, TETRI_ERR_INVALID_ARG, "tetri_set_option: null argument");
    if (std::strcmp(key, "split_keys") == 0) {
        if (value < 0 || value > 1) return fail(ctx, TETRI_ERR_INVALID_ARG, "tetri_set_option: split_keys=%d (0 or 1)", value);
        ctx->split_keys = value;
        ctx->division_set = true;
        return TETRI_OK;
    }
    if (std::strcmp(key, "split_min_stages") == 0) {
        if (value < 2) return fail(ctx, TETRI_ERR_INVALID_ARG, "tetri_set_option: split_min_stages=%d (at least 2)", value);
        ctx->split_min_stages = value;
        ctx->division_set = true;
        return TETRI_OK;
    }
    if (std::strcmp(key, "split_bias_stages") == 0) {
        if (value < 0) return fail(ctx, TETRI_ERR_INVALID_ARG, "tetri_set_option: split_bias_stages=%d (not negative)", value);
        ctx->split_bias_stages = value;
        ctx->division_set = true;
        return TETRI_OK;
    }
    if (std::strcmp(key, "split_share_q8") == 0) {
        if (value < 1 || value > 128) return fail(ctx, TETRI_ERR_INVALID_ARG, "tetri_set_option: split_share_q8=%d (1..128)", value);
        ctx->split_share_q8 = value;
        ctx->division_set = true;
        return TETRI_OK;
    }
    if (std::strcmp(key, "stream_wgs") == 0) {
        if (value < 0 || value > 255) return fail(ctx, TETRI_ERR_INVALID_ARG, "tetri_set_option: stream_wgs=%d (0..255)", value);
        ctx->stream_wgs = value;
        ctx->division_set = true;
        return TETRI_OK;
    }
    if (std::strcmp(key, "decode_parts") == 0) {
        if (value < 0) return fail(ctx, TETRI_ERR_INVALID_ARG, "tetri_set_option: decode_parts=%d (>= 0)", value);
        ctx->decode_parts = value;
        return TETRI_OK;
    }
    if (std::strcmp(key, "decode_ranges") == 0) {
        if (value < 0) return fail(ctx, TETRI_ERR_INVALID_ARG, "tetri_set_option: decode_ranges=%d (>= 0)", value);
        ctx->decode_ranges = value;
        return TETRI_OK;
    }
    if (std::strcmp(key, "transfer_slabs") == 0) {
        if (value < 0) return fail(ctx, TETRI_ERR_INVALID_ARG, "tetri_set_option: transfer_slabs=%d (>= 0)", value);
        ctx->transfer_slabs = value;
        return TETRI_OK;
    }
    if (std::strcmp(key, "attn_variant") == 0) {
        if (value < 0 || value > 5) return fail(ctx, TETRI_ERR_INVALID_ARG, "tetri_set_option: attn_variant=%d unknown", value);
        ctx->attn_variant = value;
        return TETRI_OK;
    }
    return fail(ctx, TETRI_ERR_INVALID_ARG, "tetri_set_option: unknown key '%s'", key);
}

static tetri_status check_common(tetri_ctx *h, const char *fn, const void *const *ptrs, const char *const *names, int n,
                                 int32_t num_segs)
{
    if (!h) return fail(nullptr, TETRI_ERR_INVALID_ARG, "%s: null handle", fn);
    for (int i = 0; i < n; ++i) {
        if (!ptrs[i]) return fail(h, TETRI_ERR_INVALID_ARG, "%s: %s is null", fn, names[i]);
        if (!aligned16(ptrs[i])) return fail(h, TETRI_ERR_INVALID_ARG, "%s: %s is not 16-byte aligned", fn, names[i]);
    }
    if (num_segs < 1 || num_segs > h->cfg.max_segs_per_chunk)
        return fail(h, TETRI_ERR_INVALID_ARG, "%s: num_segs=%d outside 1..%d", fn, num_segs, h->cfg.max_segs_per_chunk);
    return TETRI_OK;
}

tetri_status tetri_kv_append(tetri_ctx *h, const void *k_new, const void *v_new, void *kv_pages,
                             const int32_t *block_table, const int32_t *cu, const int32_t *ctx_lens,
                             int32_t num_segs, void *stream)
{
    const void *ptrs[] = {k_new, v_new, kv_pages};
    const char *names[] = {"k_new", "v_new", "kv_pages"};
    tetri_status st = check_common(h, "tetri_kv_append", ptrs, names, 3, num_segs);
    if (st != TETRI_OK) return st;
    if (!block_table || !cu || !ctx_lens) return fail(h, TETRI_ERR_INVALID_ARG, "tetri_kv_append: null metadata pointer");
    AppendParams p;
    p.k_new = static_cast<const uint16_t *>(k_new);
    p.v_new = static_cast<const uint16_t *>(v_new);
    p.pages = static_cast<uint16_t *>(kv_pages);
    p.bt = block_table; p.cu = cu; p.ctx = ctx_lens;
    p.S = num_segs; p.Hkv = h->cfg.num_kv_heads; p.D = h->cfg.head_dim; p.max_blocks = h->cfg.max_blocks_per_seq;
    hipError_t e = tetri_launch_append(h, p, h->cfg.chunk_size, static_cast<hipStream_t>(stream));
    if (e != hipSuccess) return fail(h, TETRI_ERR_HIP, "tetri_kv_append: launch failed: %s", hipGetErrorString(e));
    return TETRI_OK;
}

// mode 0: 16-bit pool <-> 16-bit buffer; 1: 16-bit pool -> buffer of FP8 codes (quantising);
// 2: FP8 pool <-> buffer of FP8 codes (bytes)
static tetri_status kv_transfer(const char *fn, tetri_ctx *h, void *kv_pages, void *buf, const int32_t *block_table,
                                const int32_t *cu_tokens, const int32_t *first_tokens, int32_t num_reqs,
                                int64_t total_tokens, bool to_pool, void *stream, int mode = 0, float k_scale = 1.f,
                                float v_scale = 1.f)
{
    if (!h) return fail(nullptr, TETRI_ERR_INVALID_ARG, "%s: null handle", fn);
    if (!kv_pages || !aligned16(kv_pages)) return fail(h, TETRI_ERR_INVALID_ARG, "%s: kv_pages is null or not 16-byte aligned", fn);
    if (!block_table || !cu_tokens) return fail(h, TETRI_ERR_INVALID_ARG, "%s: null metadata pointer", fn);
    if (num_reqs < 1 || num_reqs > (1 << 20)) return fail(h, TETRI_ERR_INVALID_ARG, "%s: num_reqs=%d outside 1..%d", fn, num_reqs, 1 << 20);
    const int64_t most = (int64_t)num_reqs * h->cfg.max_blocks_per_seq * h->cfg.page_size;
    if (total_tokens < 0 || total_tokens > most)
        return fail(h, TETRI_ERR_INVALID_ARG, "%s: total_tokens=%lld outside 0..%lld (num_reqs block-table rows)", fn,
                    (long long)total_tokens, (long long)most);
    if (total_tokens == 0) return TETRI_OK;
    if (!buf || !aligned16(buf)) return fail(h, TETRI_ERR_INVALID_ARG, "%s: buf is null or not 16-byte aligned", fn);
    if (mode == 1 && !(std::isfinite(k_scale) && std::isfinite(v_scale) && k_scale > 0.f && v_scale > 0.f))
        return fail(h, TETRI_ERR_INVALID_ARG, "%s: k_scale and v_scale must be positive and finite", fn);
    // 16-bit units of a row as the kernel moves it: an FP8 row of head_dim codes is head_dim / 2 units
    const int32_t row_units = mode == 2 ? h->cfg.head_dim / 2 : h->cfg.head_dim;
    const int64_t tile_tokens = 2048 / row_units;           // a workgroup's tile: 256 lanes of 16 bytes per slab
    const int64_t tiles = total_tokens / tile_tokens + num_reqs;     // >= sum of ceil(n_r / tile_tokens)
    if (tiles > 0x7fffffff) return fail(h, TETRI_ERR_INVALID_ARG, "%s: too many tokens for one launch", fn);
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess || dev != h->device)
        return fail(h, TETRI_ERR_INVALID_ARG, "%s: the handle was created on device %d, the current device is %d", fn, h->device, dev);
    TransferParams p;
    p.pool = static_cast<uint16_t *>(kv_pages);
    p.buf = static_cast<uint16_t *>(buf);
    p.bt = block_table; p.cu = cu_tokens; p.first = first_tokens;
    p.R = num_reqs; p.Hkv = h->cfg.num_kv_heads; p.max_blocks = h->cfg.max_blocks_per_seq;
    // A workgroup per slab while all of them are resident at once (eight per compute unit: a short transfer is bound by the
    // latency of each workgroup's look-ups); beyond that two slabs (quantising export: four, of half the bytes) to a
    // workgroup.  More would amortise the look-ups better, but many small workgroups keep what is read and written
    // at a time closer together and leave no half-empty last round: 20000 tokens of 40x128 with 40 slabs each 203 us, with
    // 2 and 4 191.
    const int64_t slabs = 2 * (int64_t)p.Hkv;
    p.slabs_per_wg = tiles * slabs <= 8 * (int64_t)std::max(h->num_cus, 1) ? 1 : (mode == 1 ? 4 : 2);
    if (h->transfer_slabs > 0) p.slabs_per_wg = h->transfer_slabs;
    p.slabs_per_wg = (int32_t)std::min<int64_t>(slabs, p.slabs_per_wg);
    p.slab_groups = (int32_t)((slabs + p.slabs_per_wg - 1) / p.slabs_per_wg);
    p.groups_magic = p.slab_groups <= 1 ? 0u : (uint32_t)((0x100000000ull + p.slab_groups - 1) / p.slab_groups);
    if ((tiles + 4) * p.slab_groups >= 0x7fffffff || (uint64_t)(tiles + 4) * p.slab_groups / 4 * p.slab_groups >= 0x100000000ull)
        return fail(h, TETRI_ERR_INVALID_ARG, "%s: too many tokens for one launch", fn);
    p.k_inv = 1.0f / k_scale; p.v_inv = 1.0f / v_scale;
    hipError_t e = mode == 1 ? tetri_launch_kv_export_fp8(h, p, (int32_t)tiles, static_cast<hipStream_t>(stream))
                             : tetri_launch_kv_transfer(h, p, row_units, (int32_t)tiles, to_pool, static_cast<hipStream_t>(stream));
    if (e != hipSuccess) return fail(h, TETRI_ERR_HIP, "%s: launch failed: %s", fn, hipGetErrorString(e));
    return TETRI_OK;
}

tetri_status tetri_kv_export_fp8(tetri_ctx *h, const void *kv_pages, const int32_t *block_table, const int32_t *cu_tokens,
                                 const int32_t *first_tokens, int32_t num_reqs, int64_t total_tokens, float k_scale,
                                 float v_scale, void *buf, void *stream)
{
    return kv_transfer("tetri_kv_export_fp8", h, const_cast<void *>(kv_pages), buf, block_table, cu_tokens, first_tokens,
                       num_reqs, total_tokens, false, stream, 1, k_scale, v_scale);
}

tetri_status tetri_kv_import_fp8(tetri_ctx *h, const void *buf, const int32_t *block_table, const int32_t *cu_tokens,
                                 const int32_t *first_tokens, int32_t num_reqs, int64_t total_tokens, void *kv_pages_fp8,
                                 void *stream)
{
    return kv_transfer("tetri_kv_import_fp8", h, kv_pages_fp8, const_cast<void *>(buf), block_table, cu_tokens,
                       first_tokens, num_reqs, total_tokens, true, stream, 2);
}

tetri_status tetri_kv_export(tetri_ctx *h, const void *kv_pages, const int32_t *block_table, const int32_t *cu_tokens,
                             const int32_t *first_tokens, int32_t num_reqs, int64_t total_tokens, void *buf, void *stream)
{
    return kv_transfer("tetri_kv_export", h, const_cast<void *>(kv_pages), buf, block_table, cu_tokens, first_tokens,
                       num_reqs, total_tokens, false, stream);
}

tetri_status tetri_kv_import(tetri_ctx *h, const void *buf, const int32_t *block_table, const int32_t *cu_tokens,
                             const int32_t *first_tokens, int32_t num_reqs, int64_t total_tokens, void *kv_pages, void *stream)
{
    return kv_transfer("tetri_kv_import", h, kv_pages, const_cast<void *>(buf), block_table, cu_tokens, first_tokens,
                       num_reqs, total_tokens, true, stream);
}

static tetri_status decode_common(const char *fn, tetri_ctx *h, const void *q, const void *k_new, const void *v_new,
                                  const void *kv_pages, void *kv_pages_w, const int32_t *block_table,
                                  const int32_t *ctx_lens, int32_t num_reqs, int32_t max_ctx_len, float scale, void *out,
                                  void *stream, bool fp8 = false, float k_scale = 1.f, float v_scale = 1.f,
                                  bool static_scratch = false)
{
    if (!h) return fail(nullptr, TETRI_ERR_INVALID_ARG, "%s: null handle", fn);
    const void *ptrs[] = {q, k_new, v_new, kv_pages, out};
    const char *names[] = {"q", "k_new", "v_new", "kv_pages", "out"};
    for (int i = 0; i < 5; ++i) {
        if (!ptrs[i]) return fail(h, TETRI_ERR_INVALID_ARG, "%s: %s is null", fn, names[i]);
        if (!aligned16(ptrs[i])) return fail(h, TETRI_ERR_INVALID_ARG, "%s: %s is not 16-byte aligned", fn, names[i]);
    }
    if (!block_table || !ctx_lens) return fail(h, TETRI_ERR_INVALID_ARG, "%s: null metadata pointer", fn);
    if (!std::isfinite(scale)) return fail(h, TETRI_ERR_INVALID_ARG, "%s: scale is not finite", fn);
    const tetri_config &cfg = h->cfg;
    if (num_reqs < 1 || (int64_t)num_reqs * cfg.num_kv_heads > (1 << 24))
        return fail(h, TETRI_ERR_INVALID_ARG, "%s: num_reqs=%d outside 1..%d", fn, num_reqs, (1 << 24) / cfg.num_kv_heads);
    // with the fused append the new token itself needs a slot
    const int64_t most = (int64_t)cfg.max_blocks_per_seq * cfg.page_size - (kv_pages_w ? 1 : 0);
    if (max_ctx_len < 0 || max_ctx_len > most)
        return fail(h, TETRI_ERR_INVALID_ARG, "%s: max_ctx_len=%d outside 0..%lld", fn, max_ctx_len, (long long)most);
    if (cfg.num_q_heads / cfg.num_kv_heads > 32)
        return fail(h, TETRI_ERR_UNSUPPORTED, "%s: more than 32 query heads per kv head", fn);
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess || dev != h->device)
        return fail(h, TETRI_ERR_INVALID_ARG, "%s: the handle was created on device %d, the current device is %d", fn, h->device, dev);
    DecodeParams p;
    p.q = static_cast<const uint16_t *>(q);
    p.k_new = static_cast<const uint16_t *>(k_new);
    p.v_new = static_cast<const uint16_t *>(v_new);
    p.pages = static_cast<const uint16_t *>(kv_pages);
    p.bt = block_table; p.ctx = ctx_lens;
    p.out = static_cast<uint16_t *>(out);
    p.pages_w = static_cast<uint16_t *>(kv_pages_w);
    p.partial = static_scratch ? h->decode_static.scratch : reinterpret_cast<float *>(h->scratch);
    p.B = num_reqs; p.Hq = cfg.num_q_heads; p.Hkv = cfg.num_kv_heads; p.g = p.Hq / p.Hkv;
    p.max_blocks = cfg.max_blocks_per_seq;
    p.c = std::fmax(std::fabs(scale) * 1.4426950408889634f, 1e-30f);
    p.neg = scale < 0.f;
    if (fp8 && !(std::isfinite(k_scale) && std::isfinite(v_scale) && k_scale > 0.f && v_scale > 0.f))
        return fail(h, TETRI_ERR_INVALID_ARG, "%s: k_scale and v_scale must be positive and finite", fn);
    p.fp8 = fp8;
    p.k_scale = k_scale; p.v_scale = v_scale;
    p.k_inv = 1.0f / k_scale; p.v_inv = 1.0f / v_scale;
    p.out_scale = fp8 ? v_scale : 1.0f;
    const int64_t n_counters = static_scratch ? kDecodeStaticCounters : h->n_counters;
    const int64_t pairs = (int64_t)num_reqs * p.Hkv;
    const int64_t steps = ((int64_t)max_ctx_len + 32) / 32;
    const int64_t room = static_scratch ? (int64_t)kDecodeStaticScratchBytes : (int64_t)(2 * h->scratch_units * h->unit_bytes);
    if (static_scratch && 2 * (int64_t)num_reqs * p.Hq * (cfg.head_dim + 2) * 4 > room)
        return fail(h, TETRI_ERR_INVALID_ARG, "%s: num_reqs x num_q_heads = %lld exceeds what the static scratch array of %lld bytes "
                    "holds (two parts of head_dim + 2 floats per request and head: at most %lld)", fn,
                    (long long)num_reqs * cfg.num_q_heads, (long long)room, (long long)(room / (2 * (cfg.head_dim + 2) * 4)));
    // How the work is cut (see the kernel).  The host knows the longest context, not the others.
    //  - two (request, kv head) pairs per compute unit or more: a workgroup each, the hardware balances them;
    //  - fewer, and much to read (if all contexts are that long: 200 MB, about 30 us): the steps of the batch in equal
    //    ranges, one workgroup per compute unit (two: up to 15 % slower, there are more partial results).  48 requests of
    //    16 to 8192 tokens, 32/8 heads: 70 us, against 114 with a workgroup per pair and 73 with 3 or 4;
    //  - fewer, and little to read: every pair in as many parts as fill two workgroups per compute unit, of at least three
    //    steps (the ranges' look-up and their cuts through short requests cost more than they balance: 10 us against 14 for
    //    48 requests of up to 1180 tokens, 8/2 heads).
    // All as far as the scratch memory (a partial result per part, two per range) and the counters reach.
    const int64_t part_bytes = (int64_t)4 * (p.g * cfg.head_dim + (2 * p.g + 3) / 4 * 4);
    const int64_t places = room / part_bytes, cus = std::max(h->num_cus, 1);
    p.hkv_magic = p.Hkv <= 1 ? 0u : (uint32_t)((0x100000000ull + p.Hkv - 1) / p.Hkv);
    p.ranges = 0;
    p.min_steps = h->decode_ranges > 0 ? 1 : 4;
    const bool divisible = num_reqs <= kDecodeLookup && num_reqs * ((int64_t)cfg.max_blocks_per_seq * cfg.page_size / 32 + 1) <= 0x7fffffff;
    const int64_t most_bytes = pairs * steps * 32 * 2 * cfg.head_dim * (fp8 ? 1 : 2);
    int64_t parts = h->decode_parts;
    if (parts == 0) {
        parts = std::max<int64_t>(1, std::min(2 * cus / pairs, std::min<int64_t>((steps + 2) / 3, 32)));
        const int64_t most = std::min<int64_t>(places / 2, n_counters) / p.Hkv;
        if (h->decode_ranges > 0 && divisible) p.ranges = (int32_t)std::min<int64_t>(h->decode_ranges, most);
        else if (pairs < 2 * cus && most_bytes >= 200000000 && divisible) p.ranges = (int32_t)std::min(cus / p.Hkv, most);
    }
    if (p.ranges > 1) {
        p.parts = 0;
    } else {
        if (pairs > n_counters) parts = 1;
        p.parts = (int32_t)std::max<int64_t>(1, std::min(std::min(parts, places / pairs), (int64_t)1024));
    }
    if (pairs * std::max(p.parts, 1) * (int64_t)p.Hkv >= 0xffffffffll || pairs * std::max(p.parts, 1) > 0x7fffffff)
        return fail(h, TETRI_ERR_INVALID_ARG, "%s: too many workgroups", fn);
    const bool shares = p.parts != 1;
    p.n_counters = shares ? (int32_t)n_counters : 0;
    CounterSets cs = {nullptr, nullptr};
    if (shares) cs = static_scratch ? counter_sets(h->decode_static.counters, p.n_counters, h->decode_static.turn->fetch_add(1))
                                    : counter_sets(h->counters, p.n_counters, h->counter_turn);
    p.counters = cs.use;
    p.counters_next = cs.clear;
    hipError_t e = tetri_launch_decode(h, p, static_cast<hipStream_t>(stream));
    if (e != hipSuccess) return fail(h, TETRI_ERR_HIP, "%s: launch failed: %s", fn, hipGetErrorString(e));
    if (shares && !static_scratch) ++h->counter_turn;
    return TETRI_OK;
}

tetri_status tetri_decode_attn(tetri_ctx *h, const void *q, const void *k_new, const void *v_new, const void *kv_pages,
                               const int32_t *block_table, const int32_t *ctx_lens, int32_t num_reqs, int32_t max_ctx_len,
                               float scale, void *out, void *stream)
{
    return decode_common("tetri_decode_attn", h, q, k_new, v_new, kv_pages, nullptr, block_table, ctx_lens, num_reqs,
                         max_ctx_len, scale, out, stream);
}

tetri_status tetri_decode_attn_static(tetri_ctx *h, const void *q, const void *k_new, const void *v_new, const void *kv_pages,
                                      const int32_t *block_table, const int32_t *ctx_lens, int32_t num_reqs, int32_t max_ctx_len,
                                      float scale, void *out, void *stream)
{
    return decode_common("tetri_decode_attn_static", h, q, k_new, v_new, kv_pages, nullptr, block_table, ctx_lens, num_reqs,
                         max_ctx_len, scale, out, stream, false, 1.f, 1.f, true);
}

tetri_status tetri_decode_attn_fp8(tetri_ctx *h, const void *q, const void *k_new, const void *v_new, void *kv_pages_fp8,
                                   const int32_t *block_table, const int32_t *ctx_lens, int32_t num_reqs,
                                   int32_t max_ctx_len, float scale, float k_scale, float v_scale, int32_t append,
                                   void *out, void *stream)
{
    if (append != 0 && append != 1) return fail(h, TETRI_ERR_INVALID_ARG, "tetri_decode_attn_fp8: append must be 0 or 1");
    return decode_common("tetri_decode_attn_fp8", h, q, k_new, v_new, kv_pages_fp8, append ? kv_pages_fp8 : nullptr,
                         block_table, ctx_lens, num_reqs, max_ctx_len, scale, out, stream, true, k_scale, v_scale);
}

tetri_status tetri_decode_attn_append(tetri_ctx *h, const void *q, const void *k_new, const void *v_new, void *kv_pages,
                                      const int32_t *block_table, const int32_t *ctx_lens, int32_t num_reqs,
                                      int32_t max_ctx_len, float scale, void *out, void *stream)
{
    return decode_common("tetri_decode_attn_append", h, q, k_new, v_new, kv_pages, kv_pages, block_table, ctx_lens,
                         num_reqs, max_ctx_len, scale, out, stream);
}

// Is the stream being captured into a graph?  (If the question fails: take it that it is.)
static bool stream_captures(hipStream_t hs)
{
    hipStreamCaptureStatus cap = hipStreamCaptureStatusNone;
    return hipStreamIsCapturing(hs, &cap) != hipSuccess || cap != hipStreamCaptureStatusNone;
}

// A prefill launch is about to use the handle's scratch memory and counters: one on another stream must not start before
// the previous one has ended.  (Decode launches are not asked for and do not ask: a decode loop may order its streams by
// events, which a query of the stream cannot tell from an overlap.)  (Asked of the stream, not of an event behind the launch: recording an event per launch costs
// several microseconds of queue time between 20-us kernels.  A stream that is being captured into a graph takes no
// queries: the graph orders its nodes.)
static tetri_status claim_scratch(tetri_ctx *h, const char *fn, hipStream_t hs, bool capturing)
{
    // the scratch memory lives on the device the handle was created on
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess || dev != h->device)
        return fail(h, TETRI_ERR_INVALID_ARG, "%s: the current device is %d, the handle was created on device %d", fn, dev, h->device);
    if (capturing) return TETRI_OK;
    if (h->divide_launched && h->last_divide_stream != hs && hipStreamQuery(h->last_divide_stream) == hipErrorNotReady)
        return fail(h, TETRI_ERR_INVALID_ARG, "%s: the stream of this handle's previous launch that uses its scratch memory still has work "
                    "pending; launches on one handle must not overlap (use one handle per stream)", fn);
    return TETRI_OK;
}
static void scratch_claimed(tetri_ctx *h, hipStream_t hs)
{
    h->last_divide_stream = hs;
    h->divide_launched = true;
}

// Which of the handle's two memories for partial results a launch on a division of the host's may use on stream hs: 0, 1 or, where
// another stream's launch is still at work in the one it would get, -1: none.  No call names another stream than hs: it may
// be capturing by now, or gone.  (hipStreamPerThread is another stream in every thread.)
static int plan_memory(const tetri_ctx *h, hipStream_t hs)
{
    const bool named = hs != hipStreamPerThread;
    if (named && (!h->plan_owned || h->plan_owner == hs)) return 0;
    if (!h->plan_lent || (named && h->plan_borrower == hs) || hipEventQuery(h->plan_done) == hipSuccess) return 1;
    return -1;
}
static void plan_memory_used(tetri_ctx *h, int mem, hipStream_t hs)
{
    ++h->plan_memory[mem].turn;
    (mem == 0 ? h->plan_owned : h->plan_lent) = true;
    (mem == 0 ? h->plan_owner : h->plan_borrower) = hs;
}

struct ShortShape {
    int nwl;                          // log2 of a workgroup's wavefronts
    bool preferred;
};

// The launch of the short kernel for a chunk whose segments the host knows, if it is preferred (or asked for by "attn_variant"): its row
// blocks, most work first, and the shape.  False if the chunk does not fit the kernel's tables.
static bool plan_short(const tetri_ctx *h, const int32_t *cu, const int32_t *ctx_lens, int32_t num_segs, bool fp8, ShortParams &p,
                       ShortShape &shape)
{
    if (num_segs > kShortSegs) return false;
    struct Unit { int32_t steps, seg, t0; } units[kShortUnits];
    int n = 0;
    int64_t steps = 0;                // 32-key steps of all row blocks of one head
    int64_t cached = 0;               // tokens of all contexts
    int32_t most = 0;
    for (int32_t s = 0; s < num_segs; ++s) {
        const int32_t blocks = (cu[s + 1] - cu[s] + 31) / 32, ctx_steps = (ctx_lens[s] + 31) / 32;
        if (n + blocks > kShortUnits) return false;
        for (int32_t b = 0; b < blocks; ++b) {
            units[n++] = {ctx_steps + b + 1, s, 32 * b};
            steps += ctx_steps + b + 1;
        }
        most = std::max(most, ctx_steps + blocks);
        cached += ctx_lens[s];
        if (ctx_lens[s] >= 1 << 26) return false;
    }
    p.units = n;
    p.rows = cu[num_segs];
    // Where Q, K, V and the output fit the L2 caches (8 x 4 MB) together, the output is stored past them: less is left to write back
    // when the launch ends (packed short prompts, 26 MB and below: 640 rows of 40 heads 0.5 %, 512 2.4, 768 of 32/8 6.2, 1280 3.0, 1024 of
    // 24/8 5.7, 1536 of 16 1.9).  Beyond, such stores are the slower ones (31 MB: 768 rows of 40 heads 2.8 %, 1536 of 32/8 7.7; 2048 of 16 3.4, of
    // 40 7.7, of 32/8 11.8).
    const int64_t row_bytes = 2 * h->cfg.head_dim;
    p.out_past_l2 = (int32_t)(2 * row_bytes * p.rows * h->cfg.num_q_heads + 2 * row_bytes * (p.rows + cached / (fp8 ? 2 : 1)) * h->cfg.num_kv_heads <= 28000000);
    const int64_t Hq = h->cfg.num_q_heads, wgs = n * Hq, cus = std::max(h->num_cus, 1);
    const int64_t pad_vectors = (int64_t)(h->cfg.chunk_size - p.rows) * Hq * h->cfg.head_dim / 8;
    p.zero_wgs = (int32_t)std::min<int64_t>(256, (pad_vectors + 1023) / 1024);
    // The measure that the choice below is made by: wavefronts to a row block if all had as many (a compute unit holds 8, at
    // head_dim 64 16).
    const int64_t room = h->cfg.head_dim == 64 ? 2 * cus : cus, total = steps * Hq;
    int wavefronts = wgs <= room ? 8 : (wgs <= 2 * room ? 4 : (2 * wgs <= 9 * room || total > 16 * wgs ? 2 : 1));
    if (most <= 4) wavefronts = std::min(wavefronts, 4);
    // Row blocks for at most half of the compute units: the keys of each are split, down to one step per wavefront.
    // (More workgroups than compute units lose more by the partial results' way through memory than they win.)
    const int64_t units_fit = (int64_t)(2 * h->scratch_units) / wgs;
    p.splits = 1;
    if (h->split_keys && 2 * wgs <= cus && wgs <= h->n_counters)
        p.splits = (int32_t)std::max<int64_t>(1, std::min(std::min<int64_t>(cus / wgs, 16), std::min<int64_t>((most + 7) / 8, units_fit)));
    // Where this kernel is the faster one (both timed on 650 chunks of 40x128, 32/8x128, 24/8x128, 16x128, 16/2x128 and 8/2x128 heads, 32 to
    // 1024 rows in 1 to 10 segments, 0 to 32000 cached tokens; times as a part of the shared-tile kernel's, FP8 codes in brackets):
    //  - exactly a workgroup per compute unit, eight wavefronts to a row block: up to 128 steps to a wavefront (0.4 at the shortest, 1.0
    //    at 17 steps, 1.25 (1.4) at 80);
    //  - fewer: three or more workgroups to a row block, up to 128 steps too (0.5 to 0.99 (1.07) at 31); two, up to 20 (15) steps
    //    (0.93 to 0.98 (0.96 to 1.02) at 16, 1.05 (1.1) at 24, 1.2 (1.3) at 63); one, which leaves compute units without work, up to 16
    //    (12) (0.8 to 0.9 at 9, 1.0 (1.1 to 1.2) at 16, 1.15 (1.3) at 24, 1.4 to 1.9 at 95);
    //  - exactly two workgroups per compute unit: up to 65000 (20000) steps of 32 keys x 32 rows in all (over codes the line is from when a step
    //    of codes took longer: 512 rows of 32/8 heads now 0.78 at 20700, 0.84 at 28400, 0.94 at 52500); between one and two, which leaves
    //    some compute units half empty, also up to 27 (17) steps on a wavefront times the part of the two (256 rows of 40 heads:
    //    1.05 (0.87) at 10 and 14 steps, 1.14 at 22, 1.26 at 32; 512 rows of 24/8 heads: 0.98 at 16, 1.03 at 24; 384 of 40 (0.78) at 11 and 14);
    //  - more: what a launch takes is the chain of steps of its longest row blocks, which the total does not show: up to 30000
    //    steps in all with 22 on a wavefront, at two to a row block, and 22 as laid out (1.08 at 24, 1.07 to 1.16 at 29; one segment over codes 0.66 to 0.98
    //    below these lines, 0.84 to 0.97 right behind them); over codes, several segments, 15000 and 11.  Where the work is even over the row blocks of several segments,
    //    the shared-tile kernel's tiles are ragged and teams keep the chains short: up to 30000 whatever the chain, over codes 20000
    //    unless every query head has K and V of its own (40 heads, 300 rows at 1000 and 212 at 200 cached tokens: 0.75 (0.75); 200 at 2000
    //    and 312 at 600: 0.87 (0.94); 32/8 heads, the same: 1.0 (1.1), 345 at 1353 and 167 at 0: 0.85 (0.95)).
    // head_dim 64: always (1.3 % over 224 chunks of 40x64 and 12/4x64, up to 24 % on single ones; a limit on the chain gains nothing).
    const int Hkv = h->cfg.num_kv_heads;
    const int64_t chain = (most + wavefronts - 1) / wavefronts;
    const bool even = num_segs > 1 && (int64_t)most * n <= 2 * steps;
    if (h->cfg.head_dim == 64) shape.preferred = true;
    else if (wgs <= cus) shape.preferred = chain <= (wgs == cus || p.splits > 2 ? 128 : (p.splits == 2 ? 2 * (fp8 ? 15 : 20) : (fp8 ? 12 : 16)));
    else if (wgs <= 2 * cus) shape.preferred = total <= (fp8 && wgs == 2 * cus ? 20000 : 65000);        // (the steps on a wavefront: below)
    else if (even) shape.preferred = total <= (fp8 && Hq != Hkv ? 20000 : 30000);
    else shape.preferred = total <= (fp8 && num_segs > 1 ? 15000 : 30000) && chain <= (fp8 && num_segs > 1 ? 11 : 22);
    if (!shape.preferred && h->attn_variant != 3) return true;      // (not to be laid out)
    std::sort(units, units + n, [](const Unit &a, const Unit &b) { return a.steps > b.steps; });
    for (int i = 0; i < n; ++i) {
        const int32_t s = units[i].seg;
        const uint32_t row0 = (uint32_t)cu[s], rows = (uint32_t)(cu[s + 1] - cu[s]);
        p.unit[i][0] = (uint32_t)s | (uint32_t)units[i].t0 / 32 << 6 | rows << 13 | row0 << 26;
        p.unit[i][1] = (uint32_t)ctx_lens[s] | (row0 >> 6) << 26;
    }
    // ---- the shape of the launch.  A row block of one head is the work of a team of 1, 2, 4 or 8 wavefronts: as many as leave at
    // most `cap` steps to each, cap the least for which all workgroups of the launch are on the chip at once.  (Teams of one
    // size made the launch as long as its longest row block: the 71 packed chunks of 286 short prompts of 40 heads 16.2 us
    // each, then 14.2.  Counted in wavefronts instead of workgroups, a launch could need a few workgroups more than there is room
    // for: 512 rows of 40 heads at 100 cached tokens 20.3 us (FP8 25.3), now 17.2 (20.3).)
    p.rshift = Hkv % 8 == 0 ? 3 : (Hkv % 4 == 0 ? 2 : (Hkv % 2 == 0 ? 1 : 0));
    p.hpx = (int32_t)Hq >> p.rshift;
    p.hkx = Hkv >> p.rshift;
    p.spread = wgs <= cus;
    // (of a row block of n steps, at most `cap` to a wavefront)
    // head_dim 64, more row blocks than the chip takes with teams of three on average, the work evenly spread or more than one round in any case:
    // teams of two at least, the shortest row blocks in a further round.  (In one round, with single wavefronts for the shorter half: 4096 rows of 16 heads, nothing cached, 81 us
    // (FP8 95), now 66 (84); 4096 of 12/4 62 (79), now 58 (65); 2048 of 32/8 at 2200 113, now 92; 1280 row blocks 0.98 to 1.04.  Uneven work over
    // codes, 1984 row blocks of 15 segments: 78 in one round, 142.)
    const bool twos = h->cfg.head_dim == 64 && 2 * wgs > 5 * room && (2 * wgs <= 9 * room || total > 16 * wgs)
                      && ((int64_t)most * n <= 2 * steps || wgs > 8 * room);
    auto team = [&](int32_t st, int32_t cap, int nwl) {
        int t = 0;
        while (t < nwl && (cap << t) < st) ++t;
        return twos ? std::max(t, 1) : t;
    };
    auto lay_out = [&](int nwl, int32_t cap) -> int32_t {
        int32_t first_wg = 0;
        for (int tl = 3, i = 0; tl >= 0; --tl) {
            const int begin = i;
            p.first_wg[tl] = first_wg;
            p.first_unit[tl] = begin;
            while (i < n && (p.splits > 1 ? nwl : team(units[i].steps, cap, nwl)) == tl) ++i;
            const int64_t per = p.spread ? 1 : ((int64_t)1 << nwl) >> tl;  // teams of a workgroup
            if (i > begin) first_wg += (int32_t)((((int64_t)(i - begin) * p.hpx + per - 1) / per << p.rshift) * p.splits);
        }
        return first_wg;
    };
    // the least cap for which all workgroups are on the chip at once (searched for in steps of a quarter, it was up to a fifth more: 1024
    // rows of 40 heads 32.4 us, now 30.7; 735 and 810 of 24/8 33.3, now 31.3), and the steps on a wavefront
    auto search = [&](int nwl, int32_t &longest) -> int32_t {
        int32_t cap = 1;
        for (int32_t above = most; cap < above;) {
            const int32_t mid = cap + (above - cap) / 2;
            if (lay_out(nwl, mid) > 8 * room >> nwl) cap = mid + 1;
            else above = mid;
        }
        longest = 0;
        for (int i = 0; i < n; ++i) {
            const int t = team(units[i].steps, cap, nwl);
            longest = std::max(longest, (units[i].steps + (1 << t) - 1) >> t);
        }
        return cap;
    };
    // Workgroups of 8 wavefronts, one to a compute unit, where there are no more row blocks than that; else of 4, unless those
    // of 8, whose longest row blocks have teams of 8, leave at most 0.7 times as many steps to a wavefront: timed on 280 chunks of
    // 40, 32/8, 24/8 and 8/2 heads of 128, 224 to 2048 rows, 0 to 2000 cached tokens, 0.79 to 1.0 of the time where they are
    // chosen (384 rows of 32/8 heads in segments at 50, 300 and 700: 14.4 us, now 11.4), 1.03 to 1.2 where they are not; head_dim 64: never
    // (0.86 to 1.16).
    int32_t longest = 0;
    int nwl = p.splits > 1 || (wgs <= room && most > 4) ? 3 : 2;
    int32_t cap = search(nwl, longest);
    if (nwl == 2 && longest > 3 && h->cfg.head_dim == 128) {
        int32_t longest8;
        const int32_t cap8 = search(3, longest8);
        if (10 * longest8 <= 7 * longest) { nwl = 3; cap = cap8; longest = longest8; }
    }
    p.attn_wgs = lay_out(nwl, cap);
    shape.nwl = nwl;
    if (h->cfg.head_dim != 64 && wgs > cus && wgs < 2 * cus) shape.preferred = shape.preferred && 2 * cus * longest <= (fp8 ? 17 : 27) * wgs;
    else if (h->cfg.head_dim != 64 && wgs > 2 * cus && !even && !fp8) shape.preferred = shape.preferred && longest <= 22;
    return (uint64_t)(wgs * p.splits + p.zero_wgs + 8) * (uint64_t)std::max<int64_t>(Hq, p.splits) < 0x100000000ull;   // (the divisions by multiplication)
}

// The division of a launch of the shared-tile kernel over the compute units, for a chunk whose segments the host knows.
// A job is a stretch of stages (128 keys) of one row tile (8 slots of 32 rows); p says how heads and rows share the slots.
// The work of a pool (its head groups' tiles) goes to one workgroup per compute unit so that all end together: a tile longer
// than q stages is cut into pieces of q for a workgroup each, the remainders and the tiles that are shorter are packed, the
// longest first, into the workgroups that are left; q is the smallest for which they fit.  Returns the longest workgroup's stages, 0 if the
// tables do not hold the division.  share: tiles may be cut at all.  average: the stages (with the jobs' costs) of a workgroup if all had as many.
static int32_t plan_tiles(const tetri_ctx *h, const int32_t *cu, const int32_t *ctx_lens, int32_t num_segs, const AttnParams &p, bool share,
                          TilePlan &plan, int32_t &average)
{
    constexpr int kStage = 128;
    // (timed on 120 chunks of 40, 32/8 and 8/2 heads, 256 to 2048 rows, 0 to 13000 cached tokens, both shapes: against pieces of at least
    // 3 stages, 1 for a further job and remainders one stage longer than q 1.0 to 2.0 % on average, 300 rows at 1000 and 212 at 200 cached
    // tokens of 32/8 heads 25 %; 3 or 4 for a further job the same or less)
    constexpr int kMinPiece = 2;      // the shortest pieces a tile is cut into
    constexpr int kJobCost = 2;       // a workgroup's further jobs: what each costs besides its stages, in stages
    const int wgs = (std::max(h->num_cus, 8) / 8) << p.span_shift, pools = 8 >> p.span_shift, rows = 32 * p.rb, gpx = p.gpx;
    if (num_segs > kPlanSegs || p.C > 0xffff || wgs > kPlanJobs || gpx > 1023) return 0;
    // The tiles of a head group, longest first: stages << 8 | 255 - index.  Tile t of the pool's group g is item t * gpx + g.
    uint32_t key[kPlanJobs];
    struct Tile { int32_t n; uint16_t seg, t0; } tile[kPlanJobs], found[kPlanJobs];
    int tiles = 0;
    int64_t total = 0;
    for (int32_t s = 0; s < num_segs; ++s) {
        const int32_t n = cu[s + 1] - cu[s], ctx_stages = (ctx_lens[s] + kStage - 1) / kStage;
        plan.seg[s][0] = cu[s]; plan.seg[s][1] = n; plan.seg[s][2] = ctx_lens[s]; plan.seg[s][3] = 0;
        for (int32_t t0 = 0; t0 < n; t0 += rows) {
            const int32_t stages = ctx_stages + (std::min(n, t0 + rows) + kStage - 1) / kStage;
            if ((tiles + 1) * gpx > kPlanJobs || stages > 0xffff) return 0;
            found[tiles] = {stages, (uint16_t)s, (uint16_t)t0};
            key[tiles] = (uint32_t)stages << 8 | (uint32_t)(255 - tiles);
            ++tiles;
            total += (int64_t)stages * gpx;
        }
    }
    std::sort(key, key + tiles, std::greater<uint32_t>());
    for (int t = 0; t < tiles; ++t) tile[t] = found[255 - (key[t] & 255)];
    const int nt = tiles * gpx;
    const int32_t longest = tile[0].n;
    average = (int32_t)((total + kJobCost * std::max(0, nt - wgs)) / wgs);
    const int64_t places_fit = std::min<int64_t>((int64_t)(2 * h->scratch_units), h->n_counters) / (p.hpw * p.rb * pools);
    // What any division has to meet at pieces of q stages, longer q meeting it too: the whole workgroups' pieces, the remainders
    // and the further jobs' costs fit, at most two pieces to a workgroup, places for all pieces.
    int cut = 0, full = 0;            // (of the q looked at last) tiles of a head group that are cut, and pieces of q of the pool
    auto may_fit = [&](int32_t q) -> bool {
        int64_t cuts = 0;
        for (cut = 0; cut < tiles && tile[cut].n > q; ++cut) {
            const int c = (tile[cut].n - 1) / q;
            cuts += c;
            if (c > 254) return false;
        }
        if (cuts * gpx > wgs) return false;
        full = (int)cuts * gpx;
        const int left = wgs - full;
        return (cuts + cut) * gpx <= places_fit && cut * gpx <= 2 * left && left > 0
               && total + kJobCost * std::max(0, nt - left) <= (int64_t)q * wgs;
    };
    int32_t q = (int32_t)std::min<int64_t>(std::max<int64_t>((total + wgs - 1) / wgs, kMinPiece), longest);
    if (!share) q = longest;
    for (int32_t above = longest; q < above;) {          // the shortest that may fit
        const int32_t mid = q + (above - q) / 2;
        if (may_fit(mid)) above = mid;
        else q = mid + 1;
    }
    struct Bin { int32_t load; int16_t first, last, tail; } bins[kPlanJobs];     // tail: the piece that is its last job
    uint8_t rest[kPlanJobs];          // the items, longest remainder first
    int32_t rem[kPlanJobs];           // remainders of the tiles that are cut
    int16_t link[kPlanJobs];
    for (;; q += std::max(1, q / 64)) {
        q = std::min(q, longest);
        (void)may_fit(q);
        // what remains of the tiles that are cut, in between the whole ones
        for (int t = 0; t < cut; ++t) {
            rem[t] = (tile[t].n - 1) % q + 1;
            key[t] = (uint32_t)rem[t] << 8 | (uint32_t)(255 - t);
        }
        std::sort(key, key + cut, std::greater<uint32_t>());
        int nr = 0;
        for (int x = 0, y = cut; x < cut || y < tiles;) {
            const bool piece = y == tiles || (x < cut && (int32_t)(key[x] >> 8) >= tile[y].n);
            const int t = piece ? 255 - (int)(key[x++] & 255) : y++;
            for (int g = 0; g < gpx; ++g) rest[nr++] = (uint8_t)(t * gpx + g);
        }
        auto stages = [&](int item) -> int32_t { const int t = item / gpx; return t < cut ? rem[t] : tile[t].n; };
        const int left = wgs - full;
        const bool any = q >= longest;                   // nothing is cut: whatever the loads
        // (two of the left + 1 longest meet in a workgroup)
        if (!any && nr > left && stages(rest[left - 1]) + stages(rest[left]) + kJobCost > q) continue;
        // The workgroups that are left: the longest remainder first, to the least loaded one that may take it (a heap of load << 8 |
        // workgroup).  A workgroup does at most two pieces of shared tiles there, the second as its last job (it can leave one
        // hand-over open).
        const int filled = std::min(nr, left);
        uint32_t heap[kPlanJobs];
        int n_heap = 0;
        for (int k = 0; k < left; ++k) {
            bins[k] = {0, -1, -1, -1};
            if (k >= filled) continue;
            bins[k] = {stages(rest[k]), (int16_t)rest[k], (int16_t)rest[k], -1};
            link[rest[k]] = -1;
            if (nr > left) heap[n_heap++] = (uint32_t)bins[k].load << 8 | (uint32_t)k;
        }
        std::make_heap(heap, heap + n_heap, std::greater<uint32_t>());
        bool fits = true;
        for (int r = filled; r < nr; ++r) {
            const int item = rest[r];
            const bool piece = item / gpx < cut;
            uint32_t aside[kPlanJobs];                   // those that have their last job
            int n_aside = 0;
            while (piece && n_heap > 0 && bins[heap[0] & 255].tail >= 0) {
                aside[n_aside++] = heap[0];
                std::pop_heap(heap, heap + n_heap--, std::greater<uint32_t>());
            }
            const int32_t load = n_heap == 0 ? 0 : (int32_t)(heap[0] >> 8) + stages(item) + kJobCost;
            if (n_heap == 0 || (load > q && !any)) { fits = false; break; }
            const int k = (int)(heap[0] & 255);
            Bin &to = bins[k];
            to.load = load;
            const uint32_t moved = (uint32_t)load << 8 | (uint32_t)k;
            int at = 0;                                  // the top sinks to its place
            for (int c; (c = 2 * at + 1) < n_heap; at = c) {
                c += (int)(c + 1 < n_heap && heap[c + 1] < heap[c]);
                if (heap[c] >= moved) break;
                heap[at] = heap[c];
            }
            heap[at] = moved;
            while (n_aside > 0) {
                heap[n_heap++] = aside[--n_aside];
                std::push_heap(heap, heap + n_heap, std::greater<uint32_t>());
            }
            if (piece && to.first / gpx < cut) {
                to.tail = (int16_t)item;
            } else if (piece) {                         // in front of the whole tiles
                link[item] = to.first;
                to.first = (int16_t)item;
            } else {
                link[item] = -1;
                link[to.last] = (int16_t)item;
                to.last = (int16_t)item;
            }
        }
        if (!fits) continue;
        if (nr > left && full + nr > kPlanJobs) return 0;
        // ---- the jobs: the pieces of q stages, then the other workgroups' chains
        int places = 0, jobs = 0;
        uint16_t place[kPlanJobs];                       // of a cut tile's first group
        for (int t = 0; t < cut; ++t) {
            const int cuts = (tile[t].n - rem[t]) / q;
            place[t] = (uint16_t)places;
            for (int g = 0; g < gpx; ++g, places += cuts + 1)
                for (int c = 0; c < cuts; ++c)
                    plan.job[jobs++] = {(uint16_t)(tile[t].seg | g << 6), tile[t].t0, (uint16_t)(c * q), (uint16_t)((c + 1) * q), (uint16_t)places,
                                        (uint8_t)c, (uint8_t)(cuts + 1), 0, 0};
        }
        jobs = wgs;
        int32_t load = full > 0 ? q : 0;
        for (int k = 0; k < left; ++k) {
            load = std::max(load, bins[k].load);
            if (bins[k].tail >= 0) {
                link[bins[k].tail] = -1;
                link[bins[k].last] = bins[k].tail;
            }
            int at = full + k;
            if (bins[k].first < 0) plan.job[at] = {0, 0, 0, 0, 0, 0, 0, 0, 0};
            for (int i = bins[k].first; i >= 0; i = link[i]) {
                const bool more = link[i] >= 0;
                const int t = i / gpx, g = i % gpx, cuts = t < cut ? (tile[t].n - rem[t]) / q : 0;
                plan.job[at] = {(uint16_t)(tile[t].seg | g << 6), tile[t].t0, (uint16_t)(cuts * q), (uint16_t)tile[t].n,
                                (uint16_t)(t < cut ? place[t] + g * (cuts + 1) : 0), (uint8_t)cuts, (uint8_t)(cuts + 1), (uint16_t)(more ? jobs : 0), 0};
                at = jobs;
                jobs += (int)more;
            }
        }
        plan.places = places;
        plan.wgs = wgs;
        plan.rows = cu[num_segs];
        plan.pad = 0;
        return load;
    }
}

// The shared-tile kernel on a division of the host's comes with 8 slots (head, 32-row block) to a workgroup, each a wavefront that
// does all keys, or with 4 and two key parts.  A workgroup of 8 stages a key for 256 rows instead of 128 and waits at half as many
// barriers for the same work (gqa, 16384 rows of 4 x 32 heads at 12000 cached tokens: 3.5 us for 8 blocks per SIMD, with 4 slots 2.1
// us for 4); with 4 the pieces are half as long, which divides short launches better.  Which slots a chunk may have: 4 below 30000 steps of
// 32 keys x 32 rows, 8 from 75000 on; in between both divisions are laid out and their longest workgroups compared: 4 where it has
// fewer stages than 1.7 times those of 8 and half a stage for each piece that the tiles of 8 are cut into (the merge).  Timed on 33 such
// chunks of the 16-bit and the FP8 cache (40x128, 32/8 and 8/2 heads, 256 to 2048 rows, 0 to 13000 cached tokens): 0.4 % on average
// against the better shape each time, 6 % at most (without the merge 2.5 % and 26 %, by the number of steps alone 1.3 % and 21 %).  None: over
// codes, where the launch that divides itself fills the chip with up to four row tiles to a head and their helpers, whose wavefronts walk a head's
// keys side by side (an odd number of query heads to a kv head, evenly spread work, under 50000 steps: the chunks of 512 rows of 40 heads at 1024 and
// 1536 cached tokens 1.3 us less of 83; over 16-bit rows 2.6 us more of 76; with more tiles to a head, 24/8, 20, 16 and 12 heads, prompts of 1500 to
// 3900 tokens take 1.04 to 1.41 times as long).
struct SlotChoice { bool four, eight; };

// Does a full chunk of the handle have five row tiles of 4 slots or more for every four compute units?  Then the launch that divides
// itself runs a workgroup of four wavefronts per tile, two of them to a compute unit.
static bool tiles_fill(const tetri_ctx *h)
{
    int hpw, rb;
    wave_grouping(h->cfg.num_q_heads / h->cfg.num_kv_heads, 4, &hpw, &rb);
    return (int64_t)(h->cfg.chunk_size / (32 * rb)) * (h->cfg.num_q_heads / hpw) * 4 >= 5 * (int64_t)std::max(h->num_cus, 1);
}

// Chunks of short tiles that such a launch takes faster: a job on the host's division costs its loads' and its output's round trips
// over again, with nobody else on the compute unit meanwhile, and there is nothing to balance.  Up to 5 stages to the longest tile, 7
// where the longest is at most 1.35 times a compute unit's share of all stages.  Timed on 900 chunks of 40, 32/8, 24/8, 20, 16, 16/2 and
// 8/2 heads, 512 to 4096 rows, over 16-bit rows and codes: the host's division takes 0.98 to 1.49 times as long at up to 5 stages (packed
// short prompts: 4096 rows of 32/8 heads 34.0 us, with it 47.2), 0.98 to 1.20 at 6 and 7 where that is so, 0.68 to 0.91 at 6 to 8 where it is not.
static bool short_even_tiles(const tetri_ctx *h, const int32_t *cu, const int32_t *ctx_lens, int32_t num_segs)
{
    int hpw, rb;
    wave_grouping(h->cfg.num_q_heads / h->cfg.num_kv_heads, 4, &hpw, &rb);
    const int64_t groups = h->cfg.num_q_heads / hpw, rows = 32 * rb, cus = std::max(h->num_cus, 1);
    int64_t tiles = 0, stages = 0, longest = 0;
    for (int32_t s = 0; s < num_segs; ++s) {
        const int64_t n = cu[s + 1] - cu[s], ctx_stages = (ctx_lens[s] + 127) / 128;
        longest = std::max(longest, ctx_stages + (n + 127) / 128);
        if (longest > 7) return false;
        for (int64_t t0 = 0; t0 < n; t0 += rows, ++tiles) stages += ctx_stages + (std::min(n, t0 + rows) + 127) / 128;
    }
    return 4 * tiles * groups >= 5 * cus && (longest <= 5 || 20 * longest * cus <= 27 * stages * groups);
}

static SlotChoice planned_slots(const tetri_ctx *h, const int32_t *cu, const int32_t *ctx_lens, int32_t num_segs, bool fp8)
{
    if (h->cfg.head_dim != 128) return {false, false};
    if (h->attn_variant == 4) return {false, true};
    if (h->attn_variant == 5) return {true, false};
    if (h->attn_variant != 0 || h->division_set) return {false, false};
    if (tiles_fill(h) && short_even_tiles(h, cu, ctx_lens, num_segs)) return {false, false};
    int64_t steps = 0, all = 0, tiles = 0, most = 0;  // of one head: steps, row blocks, row tiles, steps of the longest block
    for (int32_t s = 0; s < num_segs; ++s) {
        const int64_t blocks = (cu[s + 1] - cu[s] + 31) / 32, ctx_steps = (ctx_lens[s] + 31) / 32;
        steps += blocks * ctx_steps + blocks * (blocks + 1) / 2;
        all += blocks;
        tiles += (blocks + 3) / 4;
        most = std::max(most, ctx_steps + blocks);
    }
    const int64_t Hq = h->cfg.num_q_heads, self = (tiles + tiles / 2) * Hq;
    if (fp8 && tiles <= 4 && Hq / h->cfg.num_kv_heads % 2 != 0 && steps * Hq < 50000 && most * all <= 2 * steps && self <= h->num_cus && 8 * self > 7 * h->num_cus)
        return {false, false};
    return {steps * Hq < 75000, steps * Hq >= 30000};
}

// A batch's metadata that has not been sent yet, in the arguments of a kernel of its own.
static tetri_status send_metadata(tetri_ctx *h, const char *fn, MetaUpload &m, hipStream_t hs)
{
    if (!m.host) return TETRI_OK;
    const hipError_t e = tetri_launch_upload_inline(m.host, m.dev, m.len, hs);
    m.host = nullptr;
    return e == hipSuccess ? TETRI_OK : fail(h, TETRI_ERR_HIP, "%s: launch failed: %s", fn, hipGetErrorString(e));
}

// What a launch of the short kernel asks for of the next chunk's rows: K first, then V and Q, by workgroups in the places that its row blocks
// leave free.  Not for rows of less than 4 MB, nor for head_dim 64, which gain little (chunks of 256 rows of 16 and 24/8 heads, 3.1 and 2.6 MB, 2 to 3 %, 512 of
// 8/2 heads, 1.5 MB, nothing; head_dim 64, 512 rows of 40 heads 3 % more to 1 % less).  Nor with
// places for less: a prompt of 2048 tokens, 16 places in the first chunk's launch, gains nothing.  All free places share what there is to read:
// with up to kFetchKB a wavefront wherever there is as much, launches of few row blocks, short and with many places, ended later than without
// (chunks of short prompts of 16 heads, 384 rows: 112 us without, 120 so, 115 shared; 40 heads, 160 rows: 110, 115, 111; 32 heads, 192 rows: 107, 113,
// 105; prompts of 600 tokens, 16 heads, 384 rows: 144, 137, 138).  Nor with more than 4 row blocks of a head to a compute unit, whose own first reads go
// on for longer than the others wait (without and with: 40 heads, 896 rows, 204 and 214, 640 rows, 3.7 row blocks, 170 and 165; 32 heads, 1024 rows, 191 and
// 197, 768 rows, 3.5, 167 and 154; 24/8 heads, 1536 rows, 161 and 165; 20 heads, 1536 rows, 190 and 193).
static void fetch_ahead(const tetri_ctx *h, const NextRows *next, int wavefronts, ShortParams &p)
{
    p.fetch_wgs = 0;
    const int64_t cus = std::max(h->num_cus, 1);
    if (!next || next->rows == 0 || h->cfg.head_dim != 128 || (int64_t)p.units * h->cfg.num_q_heads > 4 * cus) return;
    const int64_t row = 2 * (int64_t)h->cfg.head_dim, kv = next->rows * row * h->cfg.num_kv_heads, q = next->rows * row * h->cfg.num_q_heads;
    const int64_t places = cus * 8 / wavefronts - p.attn_wgs - (p.carry ? 1 : 0);     // (one copies the metadata)
    const int64_t sizes[3] = {kv, kv, q};
    if (places * wavefronts * kFetchKB < 4096 || 2 * kv + q < 4 << 20 || 2 * kv + q > INT32_MAX) return;
    const int64_t share = (2 * kv + q + 1024 * places * wavefronts - 1) / (1024 * places * wavefronts), each = wavefronts * std::min<int64_t>(share, kFetchKB);
    const void *from[3] = {next->k_new, next->v_new, next->q};
    int64_t left = places * each;
    for (int i = 0; i < 3; ++i) {
        const int64_t kb = std::min((sizes[i] + 1023) / 1024, left);
        p.next[i] = static_cast<const uint16_t *>(from[i]);
        p.next_kb[i] = (uint32_t)kb;
        left -= kb;
    }
    p.next_bytes[0] = (uint32_t)kv;
    p.next_bytes[1] = (uint32_t)q;
    p.fetch_wgs = (int32_t)(places - left / each);
}

// How a launch of the short kernel stores its new rows of K and V (head_dim 64: ordinarily, nothing gained otherwise).  Ordinary stores leave them in the
// L2s, which are written back when the launch ends.  Written through they are in the cache in front of the memory by then, where the next chunk, the
// transfer or the decode iteration that reads them finds them; past the caches, costs least where none of them will be there any more: in calls whose rows
// do not fit that cache, 256 MB.  In launches of more than 28 MB of Q, K, V and output ordinary stores are the best or as good.  Prompts of 16 to 512
// tokens, stored ordinarily, through and past, the step alone, with the export of its requests and with a decode iteration behind it, us: 40 heads, chunks
// of 512, 4175 tokens 118, 114, 109; 138, 136, 139; 133, 131, 134; 36320 tokens 954, 908, 894; 1229, 1184, 1178; 1110, 1067, 1044 (16485 tokens, 338 MB:
// through and past 415, 410; 524, 522; 486, 481); 32/8 heads, chunks of 1024, 12496 tokens 173, 170, 171; 188, 186, 192; 187, 184, 189; 40 heads, 1024, 4175
// tokens (42 MB) 102, 99, 100; 123, 120, 131; 120, 117, 125; 24/8 heads, 2048 (34 MB) 236, 239, 238; 269, 272, 277; 261, 264, 267.  Through against
// ordinarily, over 8 head shapes and the step alone, repeated over the same buffers, with export and with decode: 0.92 to 1.02 up to 25 MB, 0.93 to 1.05 at 31 to
// 34, 0.98 to 1.04 beyond.  One prompt: 40 heads, chunks of 256, 512 tokens 23.5, 22.6; 16 heads, chunks of 512, 1024 tokens 25.0, 24.1; 8/2 heads, chunks of
// 1024, 2048 tokens 33.9, 33.2 (prompts of 700 to 4000 tokens, chunks of 1024 of 16 heads: 396, 399).
static int32_t new_row_stores(const tetri_ctx *h, int32_t num_segs, bool fp8, int64_t rows, int64_t call_rows)
{
    if (h->cfg.head_dim != 128) return kRowsCached;
    const int64_t row = 4 * h->cfg.head_dim;
    if (!fp8 && num_segs > 1 && call_rows * row * h->cfg.num_kv_heads > 256 << 20) return kRowsPast;
    return rows * row * (h->cfg.num_q_heads + h->cfg.num_kv_heads) <= 28 << 20 ? kRowsThrough : kRowsCached;
}

static tetri_status attn_common(const char *fn, tetri_ctx *h, const void *q, const void *k_new, const void *v_new,
                                const void *kv_pages, void *kv_pages_w, const int32_t *block_table, const int32_t *cu,
                                const int32_t *ctx_lens, int32_t num_segs, float scale, void *out, void *stream,
                                bool fp8 = false, float k_scale = 1.f, float v_scale = 1.f,
                                const int32_t *host_cu = nullptr, const int32_t *host_ctx = nullptr, MetaUpload *carry = nullptr,
                                const NextRows *next = nullptr)
{
    const void *ptrs[] = {q, k_new, v_new, kv_pages, out};
    const char *names[] = {"q", "k_new", "v_new", "kv_pages", "out"};
    tetri_status st = check_common(h, fn, ptrs, names, 5, num_segs);
    if (st != TETRI_OK) return st;
    if (!block_table || !cu || !ctx_lens) return fail(h, TETRI_ERR_INVALID_ARG, "%s: null metadata pointer", fn);
    if (!std::isfinite(scale)) return fail(h, TETRI_ERR_INVALID_ARG, "%s: scale is not finite", fn);
    if (fp8 && !(std::isfinite(k_scale) && std::isfinite(v_scale) && k_scale > 0.f && v_scale > 0.f))
        return fail(h, TETRI_ERR_INVALID_ARG, "%s: k_scale and v_scale must be positive and finite", fn);
    AttnParams p;
    p.plan = nullptr;
    p.k_scale = k_scale; p.v_scale = v_scale;
    p.k_inv = 1.0f / k_scale; p.v_inv = 1.0f / v_scale;
    p.q = static_cast<const uint16_t *>(q);
    p.k_new = static_cast<const uint16_t *>(k_new);
    p.v_new = static_cast<const uint16_t *>(v_new);
    p.pages = static_cast<const uint16_t *>(kv_pages);
    p.pages_w = static_cast<uint16_t *>(kv_pages_w);
    p.bt = block_table; p.cu = cu; p.ctx = ctx_lens;
    p.out = static_cast<uint16_t *>(out);
    p.S = num_segs; p.C = h->cfg.chunk_size; p.Hq = h->cfg.num_q_heads; p.Hkv = h->cfg.num_kv_heads;
    p.g = p.Hq / p.Hkv;
    p.max_blocks = h->cfg.max_blocks_per_seq;
    // scale == 0 is run as a tiny positive scale: every finite score then maps to weight 1 exactly,
    // while masked scores (-inf) still map to weight 0
    p.c = std::fmax(std::fabs(scale) * 1.4426950408889634f, 1e-30f);
    p.neg = scale < 0.f;
    hipStream_t hs = static_cast<hipStream_t>(stream);
    // divisions the kernels do by launch constants, as multiplications
    auto magic = [](uint32_t d) -> uint32_t { return d <= 1 ? 0u : (uint32_t)((0x100000000ull + d - 1) / d); };
    const int cus = std::max(h->num_cus, 1);
    // ---- a chunk with little work, its segments known on the host.  (What is captured into a graph is replayed for other
    // metadata in the same device arrays: a launch that carries the segments along is not the one to capture.)
    ShortParams sp;
    ShortShape shape = {0, false};
    // A caller who has set one of the shared-tile kernel's ways of dividing its work gets that kernel.
    if (host_cu && (h->attn_variant == 3 || (h->attn_variant == 0 && !h->division_set)) && !stream_captures(hs) &&
        plan_short(h, host_cu, host_ctx, num_segs, fp8, sp, shape) && (shape.preferred || h->attn_variant == 3)) {
        sp.q = p.q; sp.k_new = p.k_new; sp.v_new = p.v_new; sp.pages = p.pages; sp.bt = p.bt; sp.out = p.out; sp.pages_w = p.pages_w;
        sp.C = p.C; sp.Hq = p.Hq; sp.Hkv = p.Hkv; sp.g = p.g; sp.max_blocks = p.max_blocks;
        sp.hpx_magic = magic((uint32_t)sp.hpx); sp.hkx_magic = magic((uint32_t)sp.hkx); sp.splits_magic = magic((uint32_t)sp.splits);
        sp.c = p.c; sp.neg = p.neg; sp.k_scale = p.k_scale; sp.v_scale = p.v_scale; sp.k_inv = p.k_inv; sp.v_inv = p.v_inv;
        sp.zero = h->counters + kCounterSets * (size_t)h->n_counters;
        sp.scratch = reinterpret_cast<float *>(h->scratch);
        const CounterSets cs = counter_sets(h->counters, h->n_counters, h->counter_turn);
        sp.counters = cs.use;
        sp.counters_next = cs.clear;
        sp.n_counters = h->n_counters;
        if (sp.splits > 1 && (st = claim_scratch(h, fn, hs, false)) != TETRI_OK) return st;
        // (metadata that has not been sent yet goes with this launch, if it fits)
        const bool takes = carry && carry->host && !fp8 && carry->len <= kShortCarry;
        if (carry && !takes && (st = send_metadata(h, fn, *carry, hs)) != TETRI_OK) return st;
        sp.carry = takes ? carry : nullptr;
        sp.new_rows = new_row_stores(h, num_segs, fp8, host_cu[num_segs], next ? next->call_rows : 0);
        fetch_ahead(h, next, 1 << shape.nwl, sp);
        hipError_t e = tetri_launch_short(h->cfg.head_dim, fp8, sp, 1 << shape.nwl, hs);
        if (e != hipSuccess) return fail(h, TETRI_ERR_HIP, "%s: launch failed: %s", fn, hipGetErrorString(e));
        if (takes) carry->host = nullptr;
        if (sp.splits > 1) {
            ++h->counter_turn;
            scratch_claimed(h, hs);
        }
        return TETRI_OK;
    }
    if (carry && (st = send_metadata(h, fn, *carry, hs)) != TETRI_OK) return st;
    auto log2i = [](int v) { int s = 0; while ((1 << s) < v) ++s; return s; };
    // ---- the other chunks whose segments the host knows: the shared-tile kernel on a division made here
    if (host_cu && !stream_captures(hs)) {
        TilePlan plans[2];
        AttnParams shapes[2];                          // 4 and 8 slots
        int32_t load[2] = {0, 0}, average[2] = {0, 0};
        const SlotChoice may = planned_slots(h, host_cu, host_ctx, num_segs, fp8);
        const int mem = may.four || may.eight ? plan_memory(h, hs) : -1;
        for (int i = 1; i >= 0; --i) {
            // (a few more tiles of 8 than workgroups, too long to be cut: one workgroup has two, most have one.  40 heads, 609 and 779 rows at
            // 11600 cached tokens with five short segments: 626 us, on 4 slots 510)
            const bool uneven = h->attn_variant == 0 && load[1] != 0 && 20 * (int64_t)load[1] > 29 * (int64_t)average[1];
            if (!(i == 0 ? may.four || uneven : may.eight)) continue;
            AttnParams &x = shapes[i] = p;
            wave_grouping(x.g, 4 << i, &x.hpw, &x.rb);
            x.groups = x.Hq / x.hpw;
            x.hpw_shift = log2i(x.hpw);
            x.rb_shift = log2i(x.rb);
            x.span_shift = x.groups <= 1 ? 3 : (x.groups <= 2 ? 2 : (x.groups <= 4 ? 1 : 0));
            x.gpx = (x.groups + (8 >> x.span_shift) - 1) / (8 >> x.span_shift);
            load[i] = plan_tiles(h, host_cu, host_ctx, num_segs, x, h->split_keys && mem >= 0, plans[i], average[i]);
        }
        if (load[0] + load[1] != 0) {
            int32_t pieces = 0;                        // of a tile of the second
            for (int w = 0; load[1] != 0 && w < plans[1].wgs; ++w) pieces = std::max<int32_t>(pieces, plans[1].job[w].npieces);
            const int pick = load[1] == 0 || (load[0] != 0 && 10 * load[0] < 17 * load[1] + 5 * pieces) ? 0 : 1;
            TilePlan &plan = plans[pick];
            p = shapes[pick];
            int dev = -1;
            if (plan.places != 0 && (hipGetDevice(&dev) != hipSuccess || dev != h->device))
                return fail(h, TETRI_ERR_INVALID_ARG, "%s: the current device is %d, the handle was created on device %d", fn, dev, h->device);
            p.plan = &plan;
            p.gpx_magic = magic((uint32_t)p.gpx);
            p.kv_magic = magic((uint32_t)(p.g / p.hpw));
            p.tiles = p.stream_wgs = p.helpers = p.tail_q8 = p.split_min = p.split_bias = 0;
            p.attn_grid = 8 * ((plan.wgs + (1 << p.span_shift) - 1) >> p.span_shift);
            p.attn_first = p.attn_grid;
            p.append_blocks = 0;                    // (the workgroups cache the rows of their tiles)
            PlanMemory &memory = h->plan_memory[std::max(mem, 0)];
            p.scratch = memory.scratch;
            p.n_counters = h->n_counters;
            const CounterSets cs = counter_sets(memory.counters, h->n_counters, memory.turn);
            p.counters = cs.use;
            p.counters_next = cs.clear;
            plan.done = plan.places != 0 && mem == 1 ? h->plan_done : nullptr;
            hipError_t e = tetri_launch_attn(h, p, 2, fp8, hs);
            if (e != hipSuccess) return fail(h, TETRI_ERR_HIP, "%s: launch failed: %s", fn, hipGetErrorString(e));
            if (plan.places != 0) plan_memory_used(h, mem, hs);
            return TETRI_OK;
        }
    }
    wave_grouping(p.g, 4, &p.hpw, &p.rb);
    const int groups = p.Hq / p.hpw;
    // Workgroup size of the shared-tile kernel.  A full chunk has at least C / (rows of a tile) tiles per head
    // group; when that alone gives five workgroups per four compute units or more, four-wavefront workgroups (two
    // to a CU, their barriers independent of each other), one per tile, do best: with two per CU everywhere they run
    // the block loop 4-15 % faster than eight-wavefront ones, and at 1.25 per CU (ChunkSize 1024 at 40 heads)
    // still 4 % faster than eight-wavefront workgroups that divide the stages of a head among them.  On smaller
    // launches the eight-wavefront workgroup, which puts twice the wavefronts on its tile's CU, is the better one.
    int key_parts = h->attn_variant == 1 ? 1 : 2;
    if (h->attn_variant == 0 && h->stream_wgs == 0 && tiles_fill(h)) key_parts = 1;
    p.tiles = tile_bound(p.C, p.S, 32 * p.rb);
    p.gpx = (groups + 7) / 8;
    // How the work of a head group is handed out (see the kernel):
    //  - tail mode: a launch whose row tiles would occupy at most two thirds of the compute units gets one more
    //    workgroup per two tiles, which takes the tails of their key ranges; all tiles of a head start together and
    //    walk the keys side by side, so K and V come out of L2 for all but the first of them;
    //  - stream mode: a launch with more tiles than that but fewer than five per four compute units gives every head
    //    group G workgroups that share the stages of all its tiles evenly (measured: better than a second, mostly
    //    empty round of eight-wavefront workgroups, worse than tail mode where that applies: workgroups of a head
    //    then read different parts of K and V at any one time);
    //  - tile mode: one workgroup per row tile (launches with more tiles than that: four-wavefront workgroups).
    // The divisions are worked out on the device from the segment lengths; the host only has to know that
    // the numbers fit: scratch memory and arrival counters for every (tile, slot) resp. (workgroup, slot), and for
    // stream mode at most 64 segments (one lane each) and positions times G in 31 bits.
    int G = 0;
    p.helpers = 0;
    const bool counters_fit = (int64_t)groups * p.tiles * 4 <= h->n_counters;
    if (h->stream_wgs > 0) {
        G = h->stream_wgs;
    } else if (h->split_keys) {
        const int helpers = p.tiles / 2 + 1;
        // (the last tile of the bound and its helper exist only in chunks with ragged segments and are not counted)
        if (p.tiles >= 2 && (int64_t)(p.tiles - 1 + helpers - 1) * groups <= cus && (size_t)p.tiles * groups * 4 <= h->scratch_units)
            p.helpers = helpers;
        // (segments of under 256 rows on average are a batch of short prompts: a handful of stages per tile, which
        // the division would only cut into smaller pieces)
        else if ((key_parts == 2 || h->attn_variant == 1) && (int64_t)p.tiles * groups < 2 * (int64_t)cus && (int64_t)p.C >= 256 * (int64_t)p.S)
            G = std::min(255, (cus - (kv_pages_w ? 8 : 0)) / groups);
    }
    const int stage = 64 * key_parts;
    const int64_t stage_bound = (int64_t)p.tiles * (((int64_t)p.max_blocks * 16 + p.C) / stage + 2);
    if (G > 0 && (p.S > 64 || stage_bound * (G + 1) >= 0x7fffffffll || (size_t)groups * G * 4 > h->scratch_units || !counters_fit))
        G = 0;
    if (!counters_fit) p.helpers = 0;
    const bool shares = G > 0 || p.helpers > 0;         // the launch uses the handle's scratch memory and counters
    const bool capturing = shares && stream_captures(hs);
    if (shares && (st = claim_scratch(h, fn, hs, capturing)) != TETRI_OK) return st;
    p.stream_wgs = G;
    // (in tail mode the bound's last tile and its helper are extra jobs of existing workgroups)
    p.span_shift = groups <= 1 ? 3 : (groups <= 2 ? 2 : (groups <= 4 ? 1 : 0));
    const int per_group = G > 0 ? G : (p.helpers > 0 ? p.tiles + p.helpers - 2 : p.tiles);
    p.attn_grid = 8 * p.gpx * ((per_group + (1 << p.span_shift) - 1) >> p.span_shift);
    p.attn_first = p.attn_grid;
    // fused append: a few dozen workgroups, each copying every 64th row of the chunk
    // (every eight-wavefront workgroup of this kernel occupies a whole CU: in stream mode only the CUs the
    // attention workgroups leave free take append workgroups right away)
    int append_wgs = 64;
    if (shares) {
        const int idle = cus - p.attn_first;
        append_wgs = idle >= 8 ? (idle < 64 ? idle / 8 * 8 : 64) : 8;
    }
    p.append_blocks = kv_pages_w ? (p.C < append_wgs ? p.C : append_wgs) : 0;
    p.hpw_shift = log2i(p.hpw);
    p.rb_shift = log2i(p.rb);
    p.groups = groups;
    p.gpx_magic = magic((uint32_t)p.gpx);
    p.tail_q8 = h->split_share_q8;
    p.split_min = h->split_min_stages;
    p.split_bias = h->split_bias_stages;
    p.scratch = h->scratch;
    p.n_counters = h->n_counters;
    const CounterSets cs = counter_sets(h->counters, h->n_counters, h->counter_turn);
    p.counters = cs.use;
    p.counters_next = cs.clear;
    p.kv_magic = magic((uint32_t)(p.g / p.hpw));
    if ((uint64_t)p.attn_grid * (uint64_t)(p.tiles + G + 1) >= 0x100000000ull)
        return fail(h, TETRI_ERR_UNSUPPORTED, "%s: chunk_size x heads too large for one launch", fn);
    hipError_t e = tetri_launch_attn(h, p, key_parts, fp8, hs);
    if (e != hipSuccess) return fail(h, TETRI_ERR_HIP, "%s: launch failed: %s", fn, hipGetErrorString(e));
    if (shares) {
        ++h->counter_turn;
        if (!capturing) scratch_claimed(h, hs);
    }
    return TETRI_OK;
}

tetri_status tetri_chunk_prefill_attn(tetri_ctx *h, const void *q, const void *k_new, const void *v_new,
                                      const void *kv_pages, const int32_t *block_table, const int32_t *cu,
                                      const int32_t *ctx_lens, int32_t num_segs, float scale, void *out, void *stream)
{
    return attn_common("tetri_chunk_prefill_attn", h, q, k_new, v_new, kv_pages, nullptr, block_table, cu, ctx_lens,
                       num_segs, scale, out, stream);
}

tetri_status tetri_chunk_prefill_attn_append(tetri_ctx *h, const void *q, const void *k_new, const void *v_new,
                                             void *kv_pages, const int32_t *block_table, const int32_t *cu,
                                             const int32_t *ctx_lens, int32_t num_segs, float scale, void *out,
                                             void *stream)
{
    return attn_common("tetri_chunk_prefill_attn_append", h, q, k_new, v_new, kv_pages, kv_pages, block_table, cu,
                       ctx_lens, num_segs, scale, out, stream);
}

tetri_status tetri_chunk_prefill_attn_fp8(tetri_ctx *h, const void *q, const void *k_new, const void *v_new,
                                          void *kv_pages_fp8, const int32_t *block_table, const int32_t *cu,
                                          const int32_t *ctx_lens, int32_t num_segs, float scale, float k_scale,
                                          float v_scale, int32_t append, void *out, void *stream)
{
    if (append != 0 && append != 1) return fail(h, TETRI_ERR_INVALID_ARG, "tetri_chunk_prefill_attn_fp8: append must be 0 or 1");
    return attn_common("tetri_chunk_prefill_attn_fp8", h, q, k_new, v_new, kv_pages_fp8, append ? kv_pages_fp8 : nullptr,
                       block_table, cu, ctx_lens, num_segs, scale, out, stream, true, k_scale, v_scale);
}

// Host copies of a chunk's metadata: are they a chunk of this handle?
static tetri_status check_host_chunk(tetri_ctx *h, const char *fn, const int32_t *cu, const int32_t *ctx_lens, int32_t num_segs)
{
    if (!cu || !ctx_lens) return fail(h, TETRI_ERR_INVALID_ARG, "%s: null host metadata", fn);
    const int64_t most = (int64_t)h->cfg.max_blocks_per_seq * h->cfg.page_size;
    bool ok = cu[0] == 0 && cu[num_segs] <= h->cfg.chunk_size;
    for (int32_t s = 0; s < num_segs && ok; ++s)
        ok = cu[s + 1] > cu[s] && ctx_lens[s] >= 0 && (int64_t)ctx_lens[s] + (cu[s + 1] - cu[s]) <= most;
    if (!ok) return fail(h, TETRI_ERR_INVALID_ARG, "%s: the host metadata is not a chunk of this handle", fn);
    return TETRI_OK;
}

tetri_status tetri_chunk_prefill_planned(tetri_ctx *h, const void *q, const void *k_new, const void *v_new, void *kv_pages,
                                         const int32_t *block_table, const int32_t *cu, const int32_t *ctx_lens, int32_t num_segs,
                                         float scale, int32_t append, int32_t fp8, float k_scale, float v_scale,
                                         const int32_t *host_cu, const int32_t *host_ctx, void *out, void *stream)
{
    const char *fn = "tetri_chunk_prefill_planned";
    if (!h) return fail(nullptr, TETRI_ERR_INVALID_ARG, "%s: null handle", fn);
    if ((append != 0 && append != 1) || (fp8 != 0 && fp8 != 1)) return fail(h, TETRI_ERR_INVALID_ARG, "%s: append and fp8 must be 0 or 1", fn);
    if (num_segs < 1 || num_segs > h->cfg.max_segs_per_chunk)
        return fail(h, TETRI_ERR_INVALID_ARG, "%s: num_segs=%d outside 1..%d", fn, num_segs, h->cfg.max_segs_per_chunk);
    tetri_status st = check_host_chunk(h, fn, host_cu, host_ctx, num_segs);
    if (st != TETRI_OK) return st;
    return attn_common(fn, h, q, k_new, v_new, kv_pages, append ? kv_pages : nullptr, block_table, cu, ctx_lens, num_segs, scale,
                       out, stream, fp8 != 0, fp8 ? k_scale : 1.f, fp8 ? v_scale : 1.f, host_cu, host_ctx);
}

}  // extern "C"

// A ring of pinned staging buffers.  A buffer may be written again when the upload that read it is done: at once where the
// plan travelled in the kernel's arguments, otherwise the kernel's own completion signals an event (tetri_launch_upload), in
// the call that launches it, so that no stream is named again later.
struct tetri_batch {
    static constexpr int kSlots = 8;
    tetri_ctx *h = nullptr;
    int32_t *host = nullptr, *dev = nullptr;
    int64_t len = 0;                  // int32 per buffer, a multiple of 4
    hipEvent_t done[kSlots] = {};     // the buffer's last upload
    bool pending[kSlots] = {};        // ... has not been waited for
    uint64_t turn = 0;
    int slot = 0;                     // the buffer of the last upload
};

extern "C" {

int32_t tetri_batch_slots(void) { return tetri_batch::kSlots; }

void tetri_batch_destroy(tetri_batch *b)
{
    if (!b) return;
    // the caller may free the staging buffers next: no upload reads them any more
    for (int i = 0; i < tetri_batch::kSlots; ++i) {
        if (b->pending[i]) (void)hipEventSynchronize(b->done[i]);
        if (b->done[i]) (void)hipEventDestroy(b->done[i]);
    }
    delete b;
}

tetri_status tetri_batch_create(tetri_ctx *h, int64_t meta_len, int32_t *staging, int32_t *meta_dev, tetri_batch **out)
{
    const char *fn = "tetri_batch_create";
    if (!h || !out) return fail(h, TETRI_ERR_INVALID_ARG, "%s: null argument", fn);
    *out = nullptr;
    if (!staging || !aligned16(staging)) return fail(h, TETRI_ERR_INVALID_ARG, "%s: staging is null or not 16-byte aligned", fn);
    if (!meta_dev || !aligned16(meta_dev)) return fail(h, TETRI_ERR_INVALID_ARG, "%s: meta_dev is null or not 16-byte aligned", fn);
    if (meta_len < 4 || meta_len % 4 != 0 || meta_len > INT32_MAX - 3)
        return fail(h, TETRI_ERR_INVALID_ARG, "%s: meta_len=%lld (a positive multiple of 4)", fn, (long long)meta_len);
    // (the upload kernel reads the staging buffers: memory the device cannot reach would fault)
    for (const int32_t *at : {(const int32_t *)staging, (const int32_t *)staging + tetri_batch::kSlots * meta_len - 1}) {
        hipPointerAttribute_t a;
        if (hipPointerGetAttributes(&a, at) != hipSuccess || a.type != hipMemoryTypeHost) {
            (void)hipGetLastError();
            return fail(h, TETRI_ERR_INVALID_ARG, "%s: staging is not pinned host memory", fn);
        }
    }
    tetri_batch *b = new (std::nothrow) tetri_batch;
    if (!b) return fail(h, TETRI_ERR_NOMEM, "%s: out of host memory", fn);
    b->h = h; b->len = meta_len; b->host = staging; b->dev = meta_dev;
    for (hipEvent_t &ev : b->done)
        if (hipError_t e = hipEventCreateWithFlags(&ev, hipEventDisableTiming)) {
            tetri_batch_destroy(b);
            return fail(h, TETRI_ERR_HIP, "%s: %s", fn, hipGetErrorString(e));
        }
    *out = b;
    return TETRI_OK;
}

}  // extern "C"

// The plan of a batch in the next staging buffer and on its way to the device.  later (null: now): a plan that fits a kernel's arguments is
// left to be sent by the caller's next launch.
static tetri_status batch_plan(const char *fn, tetri_batch *b, const int32_t *prompt_lens, int32_t n_prompts, const int32_t *order, int32_t n_order,
                               const int32_t *req_block_tables, int32_t *layout_out, int32_t n_chunks, void *stream, MetaUpload *later)
{
    if (!b) return fail(nullptr, TETRI_ERR_INVALID_ARG, "%s: null batch", fn);
    tetri_ctx *h = b->h;
    if (!layout_out || n_chunks < 0) return fail(h, TETRI_ERR_INVALID_ARG, "%s: null layout_out or negative n_chunks", fn);
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess || dev != h->device)
        return fail(h, TETRI_ERR_INVALID_ARG, "%s: the handle was created on device %d, the current device is %d", fn, h->device, dev);
    hipStream_t hs = static_cast<hipStream_t>(stream);
    const int slot = (int)(b->turn % tetri_batch::kSlots);
    hipError_t e = hipSuccess;
    if (b->pending[slot] && hipEventQuery(b->done[slot]) == hipErrorNotReady) e = hipEventSynchronize(b->done[slot]);
    if (e != hipSuccess) return fail(h, TETRI_ERR_HIP, "%s: %s", fn, hipGetErrorString(e));
    b->pending[slot] = false;
    int32_t *host = b->host + (size_t)slot * b->len;
    int64_t len = 0;
    const int32_t got = tetri_plan_metadata(prompt_lens, n_prompts, order, n_order, h->cfg.chunk_size, req_block_tables,
                                            h->cfg.max_blocks_per_seq, host, b->len, layout_out, n_chunks, &len);
    if (got < 0) return fail(h, (tetri_status)got, "%s: %s", fn, tetri_thread_error());
    if (got != n_chunks) return fail(h, TETRI_ERR_INVALID_ARG, "%s: the plan has %d chunks, expected %d", fn, got, n_chunks);
    if (len > 0) {
        // Small plans travel in the kernel's arguments.  (Captured into a graph, the upload runs in replays: they read the staging
        // buffer, whatever it holds by then, and no event tells of them.)
        const bool capturing = stream_captures(hs), inside = len <= kUploadInline && !capturing;
        if (inside && later) {
            *later = {host, b->dev, len};
        } else {
            e = inside ? tetri_launch_upload_inline(host, b->dev, len, hs)
                       : tetri_launch_upload(host, b->dev, len, hs, capturing ? nullptr : b->done[slot]);
            if (e != hipSuccess) return fail(h, TETRI_ERR_HIP, "%s: launch failed: %s", fn, hipGetErrorString(e));
        }
        b->pending[slot] = !capturing && !inside;
    }
    b->slot = slot;
    ++b->turn;
    return TETRI_OK;
}

static tetri_status batch_launch(const char *fn, tetri_batch *b, const int32_t *layout, int32_t first_chunk, int32_t n, const void *const *q,
                                 const void *const *k_new, const void *const *v_new, void *kv_pages, void *const *out, float scale,
                                 int32_t mode, void *stream, MetaUpload *carry)
{
    if (!b) return fail(nullptr, TETRI_ERR_INVALID_ARG, "%s: null batch", fn);
    tetri_ctx *h = b->h;
    if (mode < 0 || mode > 2) return fail(h, TETRI_ERR_INVALID_ARG, "%s: mode=%d (0, 1 or 2)", fn, mode);
    if (!layout || !q || !k_new || !v_new || !out || first_chunk < 0 || n < 0)
        return fail(h, TETRI_ERR_INVALID_ARG, "%s: null argument or negative count", fn);
    const int32_t *host = b->host + (size_t)b->slot * b->len;
    // chunk c of the layout: does it fit the batch, and is its metadata a chunk of the handle?
    auto check = [&](int32_t c) -> tetri_status {
        const int32_t o_cu = layout[4 * c], o_ctx = layout[4 * c + 1], o_bt = layout[4 * c + 2], S = layout[4 * c + 3];
        if (S < 1 || S > h->cfg.max_segs_per_chunk || o_cu < 0 || o_ctx < o_cu + S + 1 || o_bt < o_ctx + S ||
            o_bt + (int64_t)S * h->cfg.max_blocks_per_seq > b->len)
            return fail(h, TETRI_ERR_INVALID_ARG, "%s: the layout of chunk %d does not fit the batch", fn, c);
        return check_host_chunk(h, fn, host + o_cu, host + o_ctx, S);
    };
    int32_t known = first_chunk;      // chunks in front of this one will not be refused for their layout or metadata
    int64_t call_rows = 0;
    for (; known < first_chunk + n && check(known) == TETRI_OK; ++known) call_rows += host[layout[4 * known] + layout[4 * known + 3]];
    for (int32_t c = first_chunk; c < first_chunk + n; ++c) {
        const int32_t o_cu = layout[4 * c], o_ctx = layout[4 * c + 1], o_bt = layout[4 * c + 2], S = layout[4 * c + 3];
        tetri_status st = c < known ? TETRI_OK : check(c);
        if (st != TETRI_OK) return st;
        // the next chunk's rows, where its launch follows this one here
        NextRows next = {nullptr, nullptr, nullptr, 0, call_rows};
        if (c + 1 < known && q[c + 1] && k_new[c + 1] && v_new[c + 1] && aligned16(q[c + 1]) && aligned16(k_new[c + 1]) && aligned16(v_new[c + 1]))
            next = {q[c + 1], k_new[c + 1], v_new[c + 1], host[layout[4 * c + 4] + layout[4 * c + 7]], call_rows};
        st = attn_common(fn, h, q[c], k_new[c], v_new[c], kv_pages, mode == 1 ? kv_pages : nullptr, b->dev + o_bt, b->dev + o_cu,
                         b->dev + o_ctx, S, scale, out[c], stream, false, 1.f, 1.f, host + o_cu, host + o_ctx, carry, &next);
        if (st == TETRI_OK && mode == 0)
            st = tetri_kv_append(h, k_new[c], v_new[c], kv_pages, b->dev + o_bt, b->dev + o_cu, b->dev + o_ctx, S, stream);
        if (st != TETRI_OK) return st;
    }
    return TETRI_OK;
}

extern "C" {

tetri_status tetri_batch_upload(tetri_batch *b, const int32_t *prompt_lens, int32_t n_prompts, const int32_t *order, int32_t n_order,
                                const int32_t *req_block_tables, int32_t *layout_out, int32_t n_chunks, void *stream)
{
    return batch_plan("tetri_batch_upload", b, prompt_lens, n_prompts, order, n_order, req_block_tables, layout_out, n_chunks, stream, nullptr);
}

tetri_status tetri_batch_launch(tetri_batch *b, const int32_t *layout, int32_t first_chunk, int32_t n, const void *const *q,
                                const void *const *k_new, const void *const *v_new, void *kv_pages, void *const *out, float scale,
                                int32_t mode, void *stream)
{
    return batch_launch("tetri_batch_launch", b, layout, first_chunk, n, q, k_new, v_new, kv_pages, out, scale, mode, stream, nullptr);
}

tetri_status tetri_batch_step(tetri_batch *b, const int32_t *prompt_lens, int32_t n_prompts, const int32_t *order, int32_t n_order,
                              const int32_t *req_block_tables, int32_t *layout_out, int32_t n_chunks, const void *const *q,
                              const void *const *k_new, const void *const *v_new, void *kv_pages, void *const *out, float scale, int32_t mode,
                              void *stream)
{
    const char *fn = "tetri_batch_step";
    MetaUpload meta = {nullptr, nullptr, 0};
    tetri_status st = batch_plan(fn, b, prompt_lens, n_prompts, order, n_order, req_block_tables, layout_out, n_chunks, stream, &meta);
    if (st != TETRI_OK) return st;
    st = batch_launch(fn, b, layout_out, 0, n_chunks, q, k_new, v_new, kv_pages, out, scale, mode, stream, &meta);
    // (no chunk, or an error before the first launch: the metadata is sent all the same, as by tetri_batch_upload; the first error counts)
    const hipError_t e = meta.host ? tetri_launch_upload_inline(meta.host, meta.dev, meta.len, static_cast<hipStream_t>(stream)) : hipSuccess;
    return st != TETRI_OK || e == hipSuccess ? st : fail(b->h, TETRI_ERR_HIP, "%s: launch failed: %s", fn, hipGetErrorString(e));
}

tetri_status tetri_validate_chunk(tetri_ctx *h, const int32_t *block_table, const int32_t *cu, const int32_t *ctx_lens,
                                  int32_t num_segs, void *stream)
{
    if (!h) return fail(nullptr, TETRI_ERR_INVALID_ARG, "tetri_validate_chunk: null handle");
    if (!block_table || !cu || !ctx_lens) return fail(h, TETRI_ERR_INVALID_ARG, "tetri_validate_chunk: null metadata pointer");
    if (num_segs < 1 || num_segs > h->cfg.max_segs_per_chunk)
        return fail(h, TETRI_ERR_INVALID_ARG, "tetri_validate_chunk: num_segs=%d outside 1..%d", num_segs, h->cfg.max_segs_per_chunk);
    const tetri_config &c = h->cfg;
    std::vector<int32_t> hcu((size_t)num_segs + 1), hctx((size_t)num_segs), hbt((size_t)num_segs * c.max_blocks_per_seq);
    hipStream_t st = static_cast<hipStream_t>(stream);
    hipError_t e = hipStreamSynchronize(st);
    if (e == hipSuccess) e = hipMemcpy(hcu.data(), cu, hcu.size() * 4, hipMemcpyDeviceToHost);
    if (e == hipSuccess) e = hipMemcpy(hctx.data(), ctx_lens, hctx.size() * 4, hipMemcpyDeviceToHost);
    if (e == hipSuccess) e = hipMemcpy(hbt.data(), block_table, hbt.size() * 4, hipMemcpyDeviceToHost);
    if (e != hipSuccess) return fail(h, TETRI_ERR_HIP, "tetri_validate_chunk: %s", hipGetErrorString(e));
    if (hcu[0] != 0) return fail(h, TETRI_ERR_INVALID_ARG, "tetri_validate_chunk: cu[0]=%d, expected 0", hcu[0]);
    std::vector<int32_t> writer((size_t)c.num_pages, -1);
    for (int32_t s = 0; s < num_segs; ++s) {
        const int32_t n = hcu[s + 1] - hcu[s];
        if (n <= 0) return fail(h, TETRI_ERR_INVALID_ARG, "tetri_validate_chunk: segment %d has length %d", s, n);
        if (hctx[s] < 0) return fail(h, TETRI_ERR_INVALID_ARG, "tetri_validate_chunk: ctx_lens[%d]=%d", s, hctx[s]);
        const int64_t end = (int64_t)hctx[s] + n;
        const int64_t blocks = (end + c.page_size - 1) / c.page_size;
        if (blocks > c.max_blocks_per_seq)
            return fail(h, TETRI_ERR_INVALID_ARG, "tetri_validate_chunk: segment %d needs %lld pages, block_table rows hold %d",
                        s, (long long)blocks, c.max_blocks_per_seq);
        for (int64_t b = 0; b < blocks; ++b) {
            const int32_t page = hbt[(size_t)s * c.max_blocks_per_seq + b];
            if (page < 0 || page >= c.num_pages)
                return fail(h, TETRI_ERR_INVALID_ARG, "tetri_validate_chunk: block_table[%d][%lld]=%d outside the pool of %d pages",
                            s, (long long)b, page, c.num_pages);
            if (b >= hctx[s] / c.page_size) {      // a page this segment writes to
                if (writer[page] >= 0 && writer[page] != s)
                    return fail(h, TETRI_ERR_INVALID_ARG, "tetri_validate_chunk: page %d is written by segments %d and %d", page, writer[page], s);
                writer[page] = s;
            }
        }
    }
    if (hcu[num_segs] > c.chunk_size)
        return fail(h, TETRI_ERR_INVALID_ARG, "tetri_validate_chunk: cu[num_segs]=%d exceeds chunk_size=%d", hcu[num_segs], c.chunk_size);
    return TETRI_OK;
}

}  // extern "C"
