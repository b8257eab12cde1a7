// Driver of the host-layer tests (built and run by tests/test_host_launches.py): the library's host layer
// (tetri_host.cpp, tetri_plan.cpp) linked with a HIP runtime and kernel launchers that only write down what
// they are asked for.  So what a call hands to a kernel, and which streams and events it touches, can be checked
// without a GPU, also where the real thing would be a race.  argv[1] names the check.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <string>
#include <vector>

#include "tetri_internal.h"

#define CHECK(cond)                                                                       \
    do {                                                                                  \
        if (!(cond)) {                                                                    \
            std::fprintf(stderr, "%s:%d: check failed: %s\n", __FILE__, __LINE__, #cond); \
            std::exit(1);                                                                 \
        }                                                                                 \
    } while (0)

namespace {

struct Block { char *p; size_t n; };
std::vector<Block> g_blocks;                  // what hipMalloc has given out
int g_device = 0;                             // the current device

bool in_handle_memory(const void *p)
{
    for (const Block &b : g_blocks)
        if (static_cast<const char *>(p) >= b.p && static_cast<const char *>(p) < b.p + b.n) return true;
    return false;
}

// The arrival counters of every launch that shares results, in order: the set it uses and the one it zeroes.
struct Counters {
    const int32_t *use, *clear;
    int32_t n;
};
std::vector<Counters> g_counters;
int g_parts = 0, g_ranges = 0;                // how the last decode was cut
std::string g_kernel;                         // the attention kernel launched last
const char *g_partials = nullptr;             // where the last attention or decode launch keeps partial results
ShortParams g_short;                          // the last launch of the short kernel
int g_short_wavefronts = 0;
std::vector<int64_t> g_carried;               // of each: int32 of metadata that it takes along
int g_out_past_l2 = -1;                       // how the last launch of the short kernel stores its output
int g_longest = 0, g_short_wgs = 0;           // the steps of its longest wavefront, and its workgroups (of the attention)
int g_places = 0;                             // of the last division made by the host: tiles' pieces there

struct Event { bool pending = false; };       // pending: work in front of it that nobody has waited for
Event &event(hipEvent_t e) { return *reinterpret_cast<Event *>(e); }
hipStream_t g_destroyed = nullptr;            // a stream that no longer exists
bool g_busy = false;                          // every stream has work pending
struct Upload {
    const int32_t *pinned;
    hipEvent_t done;
};
std::vector<Upload> g_uploads;

float g_static_scratch[kDecodeStaticScratchBytes / 4];
int32_t g_static_counters[kCounterSets * kDecodeStaticCounters];
std::atomic<uint32_t> g_static_turn;

}  // namespace

// ---- the HIP runtime, as far as the host layer uses it
extern "C" {
hipError_t hipGetDeviceCount(int *n) { *n = 2; return hipSuccess; }
hipError_t hipGetDevice(int *d) { *d = g_device; return hipSuccess; }
hipError_t hipGetDeviceProperties(hipDeviceProp_t *p, int)    // (the header renames it and the type to their current versions)
{
    std::memset(p, 0, sizeof *p);
    p->multiProcessorCount = 256;
    return hipSuccess;
}
const char *hipGetErrorString(hipError_t) { return "stub"; }
hipError_t hipGetLastError() { return hipSuccess; }
hipError_t hipMalloc(void **p, size_t n)
{
    *p = std::aligned_alloc(256, (n + 255) / 256 * 256);
    g_blocks.push_back({static_cast<char *>(*p), n});
    return hipSuccess;
}
hipError_t hipFree(void *p)
{
    for (size_t i = 0; i < g_blocks.size(); ++i)
        if (g_blocks[i].p == p) { g_blocks.erase(g_blocks.begin() + i); std::free(p); return hipSuccess; }
    return hipErrorInvalidValue;
}
hipError_t hipMemset(void *p, int v, size_t n) { std::memset(p, v, n); return hipSuccess; }
hipError_t hipMemcpy(void *d, const void *s, size_t n, hipMemcpyKind) { std::memcpy(d, s, n); return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipStreamQuery(hipStream_t s) { CHECK(s == nullptr || s != g_destroyed); return g_busy ? hipErrorNotReady : hipSuccess; }
hipError_t hipStreamIsCapturing(hipStream_t, hipStreamCaptureStatus *s) { *s = hipStreamCaptureStatusNone; return hipSuccess; }
hipError_t hipEventCreateWithFlags(hipEvent_t *e, unsigned)
{
    *e = reinterpret_cast<hipEvent_t>(new Event);
    return hipSuccess;
}
hipError_t hipEventRecord(hipEvent_t e, hipStream_t s)
{
    CHECK(s != g_destroyed);
    event(e).pending = true;
    return hipSuccess;
}
hipError_t hipEventQuery(hipEvent_t e) { return event(e).pending ? hipErrorNotReady : hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t e) { event(e).pending = false; return hipSuccess; }
hipError_t hipEventDestroy(hipEvent_t e)
{
    CHECK(!event(e).pending);                 // (somebody has waited for the work in front of it)
    delete &event(e);
    return hipSuccess;
}
hipError_t hipPointerGetAttributes(hipPointerAttribute_t *a, const void *) { a->type = hipMemoryTypeHost; return hipSuccess; }
}

// ---- the kernel launchers
hipError_t tetri_launch_attn(const tetri_ctx *, const AttnParams &p, int, bool, hipStream_t)
{
    g_kernel = "shared";
    g_partials = p.scratch;
    if (p.plan != nullptr) {
        g_places = p.plan->places;
        if (g_places != 0) g_counters.push_back({p.counters, p.counters_next, p.n_counters});
        if (p.plan->done != nullptr) event(p.plan->done).pending = true;
    } else if (p.stream_wgs > 0 || p.helpers > 0) g_counters.push_back({p.counters, p.counters_next, p.n_counters});
    return hipSuccess;
}
hipError_t tetri_launch_short(int, bool, const ShortParams &p, int wavefronts, hipStream_t)
{
    g_kernel = "short";
    g_short = p;
    g_short_wavefronts = wavefronts;
    g_carried.push_back(p.carry ? p.carry->len : 0);
    g_out_past_l2 = p.out_past_l2;
    g_longest = 0;
    g_short_wgs = p.attn_wgs;
    for (int tl = 0; tl < 4; ++tl)
        for (int u = p.first_unit[tl]; u < (tl == 0 ? p.units : p.first_unit[tl - 1]); ++u) {
            const int steps = (int)((p.unit[u][1] & 0x3ffffff) + 31) / 32 + (int)(p.unit[u][0] >> 6 & 127) + 1;
            g_longest = std::max(g_longest, (steps + (1 << tl) - 1) >> tl);
        }
    if (p.splits > 1) g_counters.push_back({p.counters, p.counters_next, p.n_counters});
    return hipSuccess;
}
hipError_t tetri_launch_decode(const tetri_ctx *, const DecodeParams &p, hipStream_t)
{
    CHECK((p.parts != 1) == (p.n_counters != 0));
    g_partials = reinterpret_cast<const char *>(p.partial);
    g_parts = p.parts;
    g_ranges = p.ranges;
    if (p.parts != 1) g_counters.push_back({p.counters, p.counters_next, p.n_counters});
    return hipSuccess;
}
hipError_t tetri_decode_static_memory(DecodeStatic *out)
{
    *out = {g_static_scratch, g_static_counters, &g_static_turn};
    return hipSuccess;
}
hipError_t tetri_launch_kv_transfer(const tetri_ctx *, const TransferParams &, int32_t, int32_t, bool, hipStream_t) { return hipSuccess; }
hipError_t tetri_launch_kv_export_fp8(const tetri_ctx *, const TransferParams &, int32_t, hipStream_t) { return hipSuccess; }
hipError_t tetri_launch_append(const tetri_ctx *, const AppendParams &, int32_t, hipStream_t) { return hipSuccess; }
hipError_t tetri_launch_upload(const int32_t *pinned, int32_t *, int64_t, hipStream_t, hipEvent_t done)
{
    if (done) {
        // the upload that read this buffer before has been waited for
        for (const Upload &u : g_uploads) CHECK(u.pinned != pinned || !event(u.done).pending);
        event(done).pending = true;
        g_uploads.push_back({pinned, done});
    } else {
        g_uploads.push_back({pinned, nullptr});
    }
    return hipSuccess;
}
hipError_t tetri_launch_upload_inline(const int32_t *, int32_t *, int64_t len, hipStream_t)
{
    CHECK(len > 0 && len <= kUploadInline);
    g_uploads.push_back({nullptr, nullptr});
    return hipSuccess;
}

namespace {

alignas(16) char g_any[64];                   // stands for every device array: nothing is read

tetri_ctx *handle(int hq, int hkv, int d, int max_blocks = 256)
{
    const tetri_config c = {hq, hkv, d, 16, 256, 1024, max_blocks, 8, TETRI_BF16};
    tetri_ctx *h = nullptr;
    CHECK(tetri_create(&c, &h) == TETRI_OK);
    return h;
}

void decode(tetri_ctx *h, bool is_static, int requests = 4)
{
    const int32_t *meta = reinterpret_cast<const int32_t *>(g_any);
    auto fn = is_static ? tetri_decode_attn_static : tetri_decode_attn;
    CHECK(fn(h, g_any, g_any, g_any, g_any, meta, meta, requests, 3000, 0.1f, g_any, nullptr) == TETRI_OK);
}

// tetri_decode_attn_static shares nothing with other launches of its handle: its counters are not the handle's.
void static_decode_counters()
{
    tetri_ctx *h = handle(2, 2, 64);
    tetri_set_option(h, "decode_parts", 5);
    decode(h, false);
    CHECK(g_counters.size() == 1 && in_handle_memory(g_counters[0].use));
    decode(h, true);
    CHECK(g_counters.size() == 2 && !in_handle_memory(g_counters[1].use) && !in_handle_memory(g_counters[1].clear));
    // as many (request, kv head)s as there are counters: a counter each, and not one more
    decode(h, true, kDecodeStaticCounters / 2);
    CHECK(g_counters.size() == 3);
    decode(h, true, kDecodeStaticCounters / 2 + 1);
    CHECK(g_counters.size() == 3);
    tetri_destroy(h);
}

// A chunk of one request: with 32 rows the short kernel splits its keys, with 256 the shared-tile kernel divides its stages, with 250
// they are divided by the host.
void prefill(tetri_ctx *h, int32_t rows)
{
    const int32_t cu[2] = {0, rows}, ctx[1] = {2000};
    const int32_t *meta = reinterpret_cast<const int32_t *>(g_any);
    tetri_set_option(h, "attn_variant", rows == 32 ? 3 : (rows == 250 ? 5 : 0));
    CHECK(tetri_chunk_prefill_planned(h, g_any, g_any, g_any, g_any, meta, meta, meta, 1, 0.1f, 0, 0, 1.f, 1.f, cu, ctx, g_any,
                                      nullptr) == TETRI_OK);
}

// Whatever a launch leaves in its counters is zeroed before they are used again, and a launch zeroes neither its own set nor
// that of the launch before or after it: decode, split short launches and divided ones in any order on one handle, and
// static decodes of two handles.
void counters_are_cleared()
{
    tetri_ctx *h = handle(8, 2, 128), *other = handle(8, 2, 128);
    tetri_set_option(h, "decode_parts", 5);
    tetri_set_option(other, "decode_parts", 5);
    const char *sequences[] = {"dddddddddd", "ssssssssss", "pppppppppp", "dspdpsddsspdpdssdpppd", "tututtuutuut", "hhhhhhhhhh", "hdhhphsdpsdhhhhdps"};
    for (const char *seq : sequences) {
        g_counters.clear();
        tetri_set_option(h, "stream_wgs", seq[0] == 's' ? 0 : 5);        // (a divided launch, whatever the shape would get)
        for (const char *c = seq; *c; ++c) {
            if (*c == 'd') decode(h, false);
            else if (*c == 's') prefill(h, 32);
            else if (*c == 'p') prefill(h, 256);
            else if (*c == 'h') prefill(h, 250);
            else decode(*c == 't' ? h : other, true);
        }
        const size_t n = g_counters.size();
        CHECK(n == std::strlen(seq));
        for (size_t i = 0; i < n; ++i) {
            const Counters &x = g_counters[i];
            CHECK(x.n > 0 && x.clear != nullptr && x.clear != x.use);
            if (i > 0) CHECK(x.clear != g_counters[i - 1].use && x.use != g_counters[i - 1].use && x.use != g_counters[i - 1].clear);
            for (size_t j = i + 1; j < n; ++j)
                if (g_counters[j].use == x.use) {                        // the set's next use: zeroed in between, all of it
                    bool cleared = false;
                    for (size_t k = i + 1; k < j; ++k) cleared = cleared || (g_counters[k].clear == x.use && g_counters[k].n == x.n);
                    CHECK(cleared);
                    break;
                }
        }
    }
    tetri_destroy(h);
    tetri_destroy(other);
}

// Launches on a division of the host's cut tiles of launches of any size.  On several streams at once they disturb neither decode nor
// launches that divide themselves nor each other, are not refused, and name no stream but their own; where there is no memory left
// for their pieces, they cut nothing.
void planned_launches_overlap()
{
    tetri_config c = {40, 40, 128, 16, 2048, 8192, 512, 8, TETRI_BF16};
    tetri_ctx *h = nullptr;
    CHECK(tetri_create(&c, &h) == TETRI_OK);
    const int32_t *meta = reinterpret_cast<const int32_t *>(g_any);
    const size_t bytes = 2 * h->scratch_units * h->unit_bytes;
    auto stream = [](uintptr_t i) { return reinterpret_cast<hipStream_t>(64 * i); };
    struct Memory { const char *partials; Counters counters; };
    auto last = [&]() { return Memory{g_partials, g_counters.back()}; };
    auto apart = [&](const Memory &a, const Memory &b) {
        CHECK(in_handle_memory(a.partials) && in_handle_memory(a.partials + bytes - 1) && in_handle_memory(a.counters.use + a.counters.n - 1));
        CHECK(a.partials + bytes <= b.partials || b.partials + bytes <= a.partials);
        for (const int32_t *x : {a.counters.use, a.counters.clear})
            for (const int32_t *y : {b.counters.use, b.counters.clear}) CHECK(x + a.counters.n <= y || y + b.counters.n <= x);
    };
    auto prefill = [&](int32_t rows, int32_t ctx, hipStream_t s) {
        const int32_t cu[2] = {0, rows};
        return tetri_chunk_prefill_planned(h, g_any, g_any, g_any, g_any, meta, meta, meta, 1, 0.1f, 1, 0, 1.f, 1.f, cu, &ctx, g_any, s);
    };
    auto split_decode = [&](hipStream_t s) {
        CHECK(tetri_decode_attn(h, g_any, g_any, g_any, g_any, meta, meta, 2, 3000, 0.1f, g_any, s) == TETRI_OK && g_parts > 1);
    };
    g_busy = true;
    CHECK(prefill(2048, 0, stream(1)) == TETRI_OK && g_places > 0);
    const Memory first = last();
    for (int i = 0; i < 5; ++i) {                  // (five take all turns of the counters)
        split_decode(stream(2));
        apart(first, last());
    }
    CHECK(prefill(1024, 4096, stream(2)) == TETRI_OK && g_places > 0);
    const Memory second = last();
    apart(first, second);
    split_decode(stream(3));
    apart(second, last());
    // a third stream beside the second's launch, and when that has ended
    const size_t n = g_counters.size();
    CHECK(prefill(2048, 0, stream(3)) == TETRI_OK && g_places == 0 && g_counters.size() == n);
    CHECK(prefill(2048, 0, hipStreamPerThread) == TETRI_OK && g_places == 0);
    CHECK(event(h->plan_done).pending);
    event(h->plan_done).pending = false;
    CHECK(prefill(2048, 0, stream(3)) == TETRI_OK && g_places > 0 && last().partials == second.partials);
    // the streams of earlier launches are gone
    g_destroyed = stream(3);
    CHECK(prefill(2048, 0, stream(4)) == TETRI_OK && g_places == 0);
    event(h->plan_done).pending = false;
    CHECK(prefill(2048, 0, stream(4)) == TETRI_OK && g_places > 0 && last().partials == second.partials);
    CHECK(prefill(2048, 0, stream(4)) == TETRI_OK && g_places > 0);
    // hipStreamPerThread is another stream in every thread: no launch on it follows another
    event(h->plan_done).pending = false;
    CHECK(prefill(2048, 0, hipStreamPerThread) == TETRI_OK && g_places > 0);
    CHECK(prefill(2048, 0, hipStreamPerThread) == TETRI_OK && g_places == 0);
    // the first stream's launches follow each other
    g_destroyed = stream(4);
    CHECK(prefill(2048, 0, stream(1)) == TETRI_OK && g_places > 0 && last().partials == first.partials);
    event(h->plan_done).pending = false;
    tetri_destroy(h);
    // launches that divide themselves beside them; two of those are held apart as ever
    c.chunk_size = 512;
    CHECK(tetri_create(&c, &h) == TETRI_OK);
    CHECK(prefill(512, 4000, stream(1)) == TETRI_OK && g_places > 0);
    const Memory planned = last();
    CHECK(tetri_set_option(h, "stream_wgs", 5) == TETRI_OK);
    CHECK(prefill(512, 4000, stream(5)) == TETRI_OK);
    apart(planned, last());
    CHECK(prefill(512, 4000, stream(6)) == TETRI_ERR_INVALID_ARG && std::strstr(tetri_last_error(h), "overlap"));
    g_busy = false;
    tetri_destroy(h);
}

// A batch of one prompt, staged in ordinary memory (which the stub takes for pinned).
struct BatchOfOne {
    tetri_ctx *h;
    const int64_t len;                        // a plan's int32: the two small arrays and the block table
    int32_t *staging;
    alignas(16) int32_t dev[4] = {};
    tetri_batch *b = nullptr;
    std::vector<int32_t> pages;
    explicit BatchOfOne(int max_blocks)
        : h(handle(8, 2, 128, max_blocks)), len(8 + max_blocks), staging(static_cast<int32_t *>(std::aligned_alloc(16, tetri_batch_slots() * len * 4))),
          pages(max_blocks)
    {
        CHECK(tetri_batch_create(h, len, staging, dev, &b) == TETRI_OK);
    }
    tetri_status upload(hipStream_t stream)
    {
        const int32_t len = 100;
        int32_t layout[4];
        return tetri_batch_upload(b, &len, 1, nullptr, 1, pages.data(), layout, 1, stream);
    }
    ~BatchOfOne()
    {
        tetri_batch_destroy(b);
        tetri_destroy(h);
        std::free(staging);
    }
};

// The upload is a kernel: with another device current it would run there.
void upload_checks_the_device()
{
    BatchOfOne x(256);
    CHECK(x.upload(nullptr) == TETRI_OK && g_uploads.size() == 1);
    g_device = 1;
    CHECK(x.upload(nullptr) == TETRI_ERR_INVALID_ARG && std::strstr(tetri_last_error(x.h), "device") && g_uploads.size() == 1);
    g_device = 0;
    CHECK(x.upload(nullptr) == TETRI_OK && g_uploads.size() == 2);
}

// Every upload that reads a staging buffer leaves an event behind itself in its own call: the buffer is waited for before it
// is written again and before the batch ends, and no stream is named in a later call (its owner may have destroyed it).
// Plans that fit the kernel's arguments are not read from the staging buffer at all.
void uploads_name_no_stream_later()
{
    for (int rounds : {1, 5, 8, 21}) {
        g_uploads.clear();
        g_destroyed = nullptr;
        BatchOfOne x(kUploadInline - 4), y(kUploadInline - 8);
        CHECK(y.upload(nullptr) == TETRI_OK && g_uploads.size() == 1 && g_uploads[0].pinned == nullptr);
        g_uploads.clear();
        for (int i = 0; i < rounds; ++i) {
            const hipStream_t s = reinterpret_cast<hipStream_t>(uintptr_t(64 + i / 3));
            CHECK(x.upload(s) == TETRI_OK && g_uploads.size() == size_t(i + 1));
            CHECK(g_uploads.back().done != nullptr && event(g_uploads.back().done).pending);
            if (i % 3 == 2) g_destroyed = s;
        }
        g_destroyed = reinterpret_cast<hipStream_t>(uintptr_t(64 + (rounds - 1) / 3));
    }
}

// Which kernel takes a chunk: what its longest row block leaves to one wavefront counts, not the total alone.
void choice_of_kernel()
{
    const tetri_config c = {32, 8, 128, 16, 512, 4096, 2100, 8, TETRI_BF16};
    tetri_ctx *h = nullptr;
    CHECK(tetri_create(&c, &h) == TETRI_OK);
    const int32_t *meta = reinterpret_cast<const int32_t *>(g_any);
    auto taken = [&](std::vector<int32_t> cu, std::vector<int32_t> ctx, int fp8) {
        CHECK(tetri_chunk_prefill_planned(h, g_any, g_any, g_any, g_any, meta, meta, meta, (int32_t)ctx.size(), 0.1f, 0, fp8, 1.f, 1.f,
                                          cu.data(), ctx.data(), g_any, nullptr) == TETRI_OK);
        return g_kernel;
    };
    // 544 workgroups of two wavefronts, the longest block alone: 40 steps, 22, 44, 45
    CHECK(taken({0, 36, 512}, {1191, 0}, 1) == "shared" && taken({0, 36, 512}, {1191, 0}, 0) == "short");
    CHECK(taken({0, 36, 512}, {640, 0}, 1) == "short" && taken({0, 36, 512}, {641, 0}, 1) == "shared");
    CHECK(taken({0, 36, 512}, {1344, 0}, 0) == "short" && taken({0, 36, 512}, {1345, 0}, 0) == "shared");
    // 512 workgroups: the total counts (32 x (16 x context steps + 136))
    CHECK(taken({0, 512}, {960}, 1) == "short" && taken({0, 512}, {992}, 1) == "shared");
    CHECK(taken({0, 512}, {3776}, 0) == "short" && taken({0, 512}, {3808}, 0) == "shared");
    // 256 workgroups of eight: whatever the total, up to 128 steps on a wavefront
    CHECK(taken({0, 256}, {32000}, 1) == "short" && taken({0, 256}, {32500}, 0) == "short" && taken({0, 256}, {32513}, 0) == "shared");
    tetri_destroy(h);
}

// The short kernel's output goes past the caches where Q, K, V and the output fit them together (28 MB), not in larger launches.
void short_output_stores()
{
    const tetri_config c = {40, 40, 128, 16, 2048, 8192, 512, 40, TETRI_BF16};
    tetri_ctx *h = nullptr;
    CHECK(tetri_create(&c, &h) == TETRI_OK && tetri_set_option(h, "attn_variant", 3) == TETRI_OK);
    const int32_t *meta = reinterpret_cast<const int32_t *>(g_any);
    auto past = [&](int32_t rows, int32_t ctx, int fp8) {
        const int32_t cu[2] = {0, rows};
        CHECK(tetri_chunk_prefill_planned(h, g_any, g_any, g_any, g_any, meta, meta, meta, 1, 0.1f, 1, fp8, 1.f, 1.f, cu, &ctx, g_any, nullptr) == TETRI_OK);
        CHECK(g_kernel == "short");
        return g_out_past_l2;
    };
    // 40 heads: 40 KB a row, 20 a cached token (codes: 10)
    CHECK(past(683, 0, 0) == 1 && past(684, 0, 0) == 0 && past(2048, 0, 1) == 0 && past(1, 0, 1) == 1);
    CHECK(past(512, 343, 0) == 1 && past(512, 344, 0) == 0 && past(512, 686, 1) == 1 && past(512, 688, 1) == 0);
    tetri_destroy(h);
}

// A launch of the short kernel that the next chunk's follows asks for rows of that chunk and for nothing outside them, with the places
// that its row blocks leave free; the last chunk's launch, one with no place left, one for small rows and head_dim 64 do not.
void next_chunk_rows()
{
    auto batch = [&](int hq, int hkv, int d, int chunk, std::vector<int32_t> lens, int32_t first, int32_t n) {
        const int max_blocks = 128, prompts = (int)lens.size();
        const tetri_config c = {hq, hkv, d, 16, chunk, 8192, max_blocks, 40, TETRI_BF16};
        tetri_ctx *h = nullptr;
        CHECK(tetri_create(&c, &h) == TETRI_OK && tetri_set_option(h, "attn_variant", 3) == TETRI_OK);
        std::vector<int32_t> pages((size_t)prompts * max_blocks), layout(4 * 64);
        const int64_t len = 1 << 14;
        int32_t *staging = static_cast<int32_t *>(std::aligned_alloc(16, tetri_batch_slots() * len * 4));
        alignas(16) static int32_t dev[4];
        tetri_batch *b = nullptr;
        g_uploads.clear();
        CHECK(tetri_batch_create(h, len, staging, dev, &b) == TETRI_OK);
        int32_t rows = 0;
        for (int32_t x : lens) rows += x;
        const int32_t chunks = (rows + chunk - 1) / chunk;
        CHECK(tetri_batch_upload(b, lens.data(), prompts, nullptr, prompts, pages.data(), layout.data(), chunks, nullptr) == TETRI_OK);
        std::vector<const void *> q, k, v;
        std::vector<void *> out;
        for (uintptr_t i = 0; i < (uintptr_t)chunks; ++i) {
            q.push_back(reinterpret_cast<void *>((4 * i + 1) << 32));
            k.push_back(reinterpret_cast<void *>((4 * i + 2) << 32));
            v.push_back(reinterpret_cast<void *>((4 * i + 3) << 32));
            out.push_back(reinterpret_cast<void *>((4 * i + 4) << 32));
        }
        CHECK(tetri_batch_launch(b, layout.data(), first, n, q.data(), k.data(), v.data(), g_any, out.data(), 0.1f, 1, nullptr) == TETRI_OK);
        CHECK(g_kernel == "short");
        const ShortParams &p = g_short;
        uint64_t asked = 0;
        CHECK(p.fetch_wgs == 0);                     // (of the last chunk)
        // the launch before it: the last chunk is refused
        if (n > 1) {
            std::vector<const void *> none(q);
            none[first + n - 1] = nullptr;
            CHECK(tetri_batch_launch(b, layout.data(), first, n, none.data(), k.data(), v.data(), g_any, out.data(), 0.1f, 1, nullptr) != TETRI_OK);
            CHECK(p.fetch_wgs == 0);                 // (and its rows are not known)
            int32_t wider[4 * 64];
            std::copy(layout.begin(), layout.end(), wider);
            wider[4 * (first + n - 1) + 3] = 0;      // no segments: refused too
            CHECK(tetri_batch_launch(b, wider, first, n, q.data(), k.data(), v.data(), g_any, out.data(), 0.1f, 1, nullptr) != TETRI_OK);
            CHECK(p.fetch_wgs == 0);
            std::copy(layout.begin(), layout.end(), wider);
            int32_t *const l = wider + 4 * (first + n - 1);
            l[0] = l[1] - l[3];                      // refused; where its number of rows would be stands that of its cached tokens
            CHECK(tetri_batch_launch(b, wider, first, n, q.data(), k.data(), v.data(), g_any, out.data(), 0.1f, 1, nullptr) != TETRI_OK);
            CHECK(p.fetch_wgs == 0);
            std::vector<void *> bad(out);
            bad[first + n - 1] = nullptr;            // refused, its rows known
            CHECK(tetri_batch_launch(b, layout.data(), first, n, q.data(), k.data(), v.data(), g_any, bad.data(), 0.1f, 1, nullptr) != TETRI_OK);
            const int32_t next = first + n - 1;
            const uint64_t have = (uint64_t)std::min(chunk, rows - next * chunk), row = 2 * (uint64_t)d;
            if (p.fetch_wgs != 0) {
                const void *from[3] = {k[next], v[next], q[next]};
                CHECK(p.attn_wgs + p.fetch_wgs <= 256 * 8 / g_short_wavefronts);
                CHECK(p.next_bytes[0] == have * row * hkv && p.next_bytes[1] == have * row * hq);
                for (int i = 0; i < 3; ++i) {
                    CHECK(p.next[i] == from[i] && 1024 * (uint64_t)p.next_kb[i] < p.next_bytes[i == 2] + 1024);
                    asked += p.next_kb[i];
                }
                // (all free places share what there is, up to kFetchKB to a wavefront)
                const uint64_t all = (2 * p.next_bytes[0] + p.next_bytes[1] + 1023) / 1024, waves = (uint64_t)(256 * 8 / g_short_wavefronts - p.attn_wgs) * g_short_wavefronts;
                const uint64_t each = std::min<uint64_t>(kFetchKB, (all + waves - 1) / waves) * g_short_wavefronts;
                CHECK(asked <= p.fetch_wgs * each && asked > (p.fetch_wgs - 1) * each);
                // what the kernel's lanes make of that: every 16 bytes of that much of a matrix, none outside its rows
                for (int m = 0; m < 3; ++m) {
                    std::vector<char> seen(p.next_bytes[m == 2] / 16, 0);
                    for (uint32_t i = 0; i < (uint32_t)asked; ++i)
                        for (uint32_t lane = 0; lane < 64; ++lane) {
                            const FetchAt f = fetch_at(i, lane, p.next_kb[0], p.next_kb[1], p.next_bytes[0], p.next_bytes[1]);
                            CHECK(f.byte % 16 == 0 && f.byte + 16 <= p.next_bytes[f.matrix == 2]);
                            if (f.matrix == m) seen[f.byte / 16] = 1;
                        }
                    const size_t want = std::min<size_t>(seen.size(), (size_t)p.next_kb[m] * 64);
                    CHECK(std::count(seen.begin(), seen.begin() + want, 1) == (ptrdiff_t)want);
                }
            }
        }
        // the same with the metadata in the first launch: it leaves a place for the workgroup that copies it (the second chunk's launch refused)
        if (first == 0 && n > 1) {
            const int32_t fetched = p.fetch_wgs;
            CHECK(fetched == 0 || p.carry == nullptr);
            std::vector<void *> bad(out);
            bad[1] = nullptr;
            CHECK(tetri_batch_step(b, lens.data(), prompts, nullptr, prompts, pages.data(), layout.data(), chunks, q.data(), k.data(), v.data(), g_any,
                                   bad.data(), 0.1f, 1, nullptr) != TETRI_OK);
            CHECK(p.fetch_wgs <= fetched && (p.fetch_wgs == 0 || p.attn_wgs + p.fetch_wgs + (p.carry != nullptr) <= 256 * 8 / g_short_wavefronts));
        }
        tetri_batch_destroy(b);
        tetri_destroy(h);
        std::free(staging);
        return asked;
    };
    CHECK(batch(40, 40, 128, 512, {1024}, 0, 1) == 0);
    CHECK(batch(40, 40, 128, 512, {1024}, 0, 2) == 0);                                // 496 places taken
    CHECK(batch(40, 40, 128, 512, {512, 512, 512}, 1, 2) == 0);
    CHECK(batch(40, 40, 128, 512, {1536}, 1, 2) == 32 * 4 * kFetchKB);                // 480
    CHECK(batch(40, 40, 128, 512, {200, 312, 139}, 0, 2) != 0);                       // 139 rows: 4.27 MB, not a multiple of 1 KB per head
    CHECK(batch(40, 40, 128, 512, {200, 312, 136}, 0, 2) == 0);                       // 4.18 MB: below 4 MiB
    CHECK(batch(32, 8, 128, 512, {100, 412, 511}, 0, 2) != 0);
    CHECK(batch(8, 2, 128, 512, {1024}, 0, 2) == 0);
    CHECK(batch(32, 8, 128, 512, {100, 611}, 0, 2) == 0);                             // 199 rows at 412 cached tokens
    CHECK(batch(40, 40, 64, 512, {1024}, 0, 2) == 0);
    // up to four row blocks of a head to a compute unit: 1024 of them, not 1280 or 1056
    CHECK(batch(40, 40, 128, 1024, {2048}, 0, 2) == 0);
    CHECK(batch(32, 32, 128, 1020, {64, 64, 64, 64, 64, 64, 64, 64, 64, 64, 380, 1020}, 0, 2) != 0);
    CHECK(batch(32, 32, 128, 1052, {64, 64, 64, 64, 64, 64, 64, 64, 64, 64, 412, 1052}, 0, 2) == 0);
    CHECK(batch(16, 16, 128, 384, {200, 184, 384}, 0, 2) == 3 * 384 * 4);             // 1300 places for wavefronts: 4 KB each
    // (those that tests/test_gpu_batch_step.py runs)
    CHECK(batch(36, 9, 128, 512, {150, 362, 301, 211, 333}, 0, 2) != 0 && batch(36, 9, 128, 512, {150, 362, 301, 211, 333}, 1, 2) != 0);
    CHECK(batch(40, 40, 128, 512, {60, 60, 60, 60, 60, 60, 60, 60, 32, 200, 200, 200, 200, 200}, 0, 2) != 0);
    CHECK(batch(40, 40, 128, 160, {480}, 0, 2) != 0 && g_short_wavefronts == 8);
    CHECK(batch(40, 40, 128, 512, {200, 312, 300, 500, 77}, 1, 2) != 0);
}

// How new rows are stored: through the L2 in launches of up to 28 MB of rows, past the caches in calls of more than 256 MB of new ones.
void new_row_stores()
{
    auto launch = [&](int hq, int hkv, int d, std::vector<int32_t> rows, int fp8) {
        const tetri_config c = {hq, hkv, d, 16, 2048, 8192, 512, 40, TETRI_BF16};
        tetri_ctx *h = nullptr;
        CHECK(tetri_create(&c, &h) == TETRI_OK && tetri_set_option(h, "attn_variant", 3) == TETRI_OK);
        const int32_t *meta = reinterpret_cast<const int32_t *>(g_any);
        std::vector<int32_t> cu{0}, ctx(rows.size());
        for (int32_t n : rows) cu.push_back(cu.back() + n);
        CHECK(tetri_chunk_prefill_planned(h, g_any, g_any, g_any, g_any, meta, meta, meta, (int32_t)ctx.size(), 0.1f, 1, fp8, 1.f, 1.f, cu.data(), ctx.data(), g_any,
                                          nullptr) == TETRI_OK);
        CHECK(g_kernel == "short");
        tetri_destroy(h);
        return g_short.new_rows;
    };
    CHECK(launch(40, 40, 128, {716}, 0) == kRowsThrough && launch(40, 40, 128, {717}, 0) == kRowsCached && launch(40, 40, 128, {200, 312}, 0) == kRowsThrough && launch(40, 40, 128, {200, 312}, 1) == kRowsThrough);
    CHECK(launch(40, 40, 128, {200, 516}, 0) == kRowsThrough && launch(40, 40, 128, {200, 517}, 1) == kRowsCached);      // (40 KB a row)
    CHECK(launch(40, 40, 64, {200, 312}, 0) == kRowsCached);
    // 40 heads: 20 KB a token, 13107 tokens are not quite 256 MB
    auto batch = [&](int32_t tokens, int32_t first, int32_t n) {
        const int max_blocks = 32;
        const tetri_config c = {40, 40, 128, 16, 512, 8192, max_blocks, 40, TETRI_BF16};
        tetri_ctx *h = nullptr;
        CHECK(tetri_create(&c, &h) == TETRI_OK && tetri_set_option(h, "attn_variant", 3) == TETRI_OK);
        std::vector<int32_t> lens(51, 256);
        lens.push_back(tokens - 51 * 256);
        const int64_t len = 1 << 14;
        std::vector<int32_t> pages(52 * max_blocks), layout(4 * 26);
        int32_t *staging = static_cast<int32_t *>(std::aligned_alloc(16, tetri_batch_slots() * len * 4));
        alignas(16) static int32_t dev[4];
        tetri_batch *b = nullptr;
        g_uploads.clear();
        CHECK(tetri_batch_create(h, len, staging, dev, &b) == TETRI_OK);
        CHECK(tetri_batch_upload(b, lens.data(), 52, nullptr, 52, pages.data(), layout.data(), 26, nullptr) == TETRI_OK);
        std::vector<const void *> in(26, g_any);
        std::vector<void *> out(26, g_any);
        CHECK(tetri_batch_launch(b, layout.data(), first, n, in.data(), in.data(), in.data(), g_any, out.data(), 0.1f, 1, nullptr) == TETRI_OK);
        CHECK(g_kernel == "short");
        if (!g_uploads.empty() && g_uploads[0].done) event(g_uploads[0].done).pending = false;
        tetri_batch_destroy(b);
        tetri_destroy(h);
        std::free(staging);
        return g_short.new_rows;
    };
    CHECK(batch(13107, 0, 26) == kRowsThrough && batch(13108, 0, 26) == kRowsPast);
    CHECK(batch(13108, 1, 25) == kRowsThrough && batch(13108, 25, 1) == kRowsThrough);
}

// Where a step's metadata travels: with the first launch up to kShortCarry int32 if that is one of the short kernel; else in one upload in front
// of it; once, whatever the launch comes to.
void carried_metadata()
{
    auto step = [&](int max_blocks, int variant, float scale, int32_t chunks_expected, int64_t expected_len, bool refused_later = false) {
        const tetri_config c = {8, 2, 128, 16, 128, 8192, max_blocks, 40, TETRI_BF16};
        tetri_ctx *h = nullptr;
        CHECK(tetri_create(&c, &h) == TETRI_OK && tetri_set_option(h, "attn_variant", variant) == TETRI_OK);
        const int32_t lens[1] = {chunks_expected * 128};
        const int64_t len = 1 << 12;
        int32_t *staging = static_cast<int32_t *>(std::aligned_alloc(16, tetri_batch_slots() * len * 4));
        std::vector<int32_t> pages(max_blocks), layout(4 * chunks_expected + 4);
        alignas(16) static int32_t dev[4];
        tetri_batch *b = nullptr;
        CHECK(tetri_batch_create(h, len, staging, dev, &b) == TETRI_OK);
        std::vector<const void *> in(chunks_expected, g_any);
        std::vector<void *> out(chunks_expected, g_any);
        if (refused_later) out.back() = nullptr;
        g_uploads.clear();
        g_carried.clear();
        const tetri_status st = tetri_batch_step(b, lens, 1, nullptr, 1, pages.data(), layout.data(), chunks_expected, in.data(), in.data(), in.data(), g_any,
                                                 out.data(), scale, 1, nullptr);
        CHECK((st == TETRI_OK) == (std::isfinite(scale) && !refused_later));
        int64_t carried = 0;
        for (size_t i = 0; i < g_carried.size(); ++i) {
            CHECK(i == 0 || g_carried[i] == 0);          // (the first launch, no other)
            carried += g_carried[i];
        }
        if (carried != 0) CHECK(carried == expected_len && g_short.bt >= dev);
        CHECK(g_uploads.size() == (carried == 0));
        const bool inside = !g_uploads.empty() && g_uploads[0].pinned == nullptr;
        if (!g_uploads.empty() && !inside) event(g_uploads[0].done).pending = false;
        tetri_batch_destroy(b);
        tetri_destroy(h);
        std::free(staging);
        return carried != 0 ? "carried" : (inside ? "inline" : "staged");
    };
    // 4 chunks of a segment: 8 int32 and a table of 160 to 224 (a multiple of 4) each
    CHECK(step(160, 3, 0.1f, 4, 672) == std::string("carried"));
    CHECK(step(164, 3, 0.1f, 4, 688) == std::string("inline"));
    CHECK(step(216, 3, 0.1f, 4, 896) == std::string("inline"));
    CHECK(step(220, 3, 0.1f, 4, 912) == std::string("staged"));
    CHECK(step(32, 3, 0.1f, 1, 40) == std::string("carried") && step(664, 3, 0.1f, 1, 672) == std::string("carried"));
    CHECK(step(668, 3, 0.1f, 1, 676) == std::string("inline"));
    CHECK(step(160, 2, 0.1f, 4, 672) == std::string("inline"));                      // no launch of the short kernel
    CHECK(step(160, 3, NAN, 4, 672) == std::string("inline"));                       // refused before the first launch
    CHECK(step(160, 3, 0.1f, 4, 672, true) == std::string("carried"));               // ... and behind it
}

// Teams are as small as leaves all workgroups on the chip at once and no smaller: 32 row blocks of 1 to 32 steps and 40 heads, 512 places
// for workgroups of four wavefronts, take 480 with up to 16 steps to a wavefront (15 would take 530).
void short_teams()
{
    const tetri_config c = {40, 40, 128, 16, 1024, 8192, 512, 40, TETRI_BF16};
    tetri_ctx *h = nullptr;
    CHECK(tetri_create(&c, &h) == TETRI_OK);
    const int32_t *meta = reinterpret_cast<const int32_t *>(g_any);
    const int32_t cu[2] = {0, 1024}, ctx = 0;
    CHECK(tetri_chunk_prefill_planned(h, g_any, g_any, g_any, g_any, meta, meta, meta, 1, 0.1f, 1, 0, 1.f, 1.f, cu, &ctx, g_any, nullptr) == TETRI_OK);
    CHECK(g_kernel == "short" && g_longest == 16 && g_short_wgs == 480);
    tetri_destroy(h);
    // head_dim 64, 128 row blocks of 1 to 128 steps and 16 heads: two wavefronts to each in two rounds, not one round with up to 52 steps to
    // single ones; a long context beside them: one round
    const tetri_config c64 = {16, 16, 64, 16, 4096, 8192, 1024, 40, TETRI_BF16};
    CHECK(tetri_create(&c64, &h) == TETRI_OK);
    const int32_t cu64[2] = {0, 4096}, ragged[3] = {0, 96, 4096}, contexts[2] = {9000, 0};
    CHECK(tetri_chunk_prefill_planned(h, g_any, g_any, g_any, g_any, meta, meta, meta, 1, 0.1f, 1, 0, 1.f, 1.f, cu64, &ctx, g_any, nullptr) == TETRI_OK);
    CHECK(g_longest == 64 && g_short_wgs == 128 * 16 / 2);
    CHECK(tetri_chunk_prefill_planned(h, g_any, g_any, g_any, g_any, meta, meta, meta, 2, 0.1f, 1, 0, 1.f, 1.f, ragged, contexts, g_any, nullptr) == TETRI_OK);
    CHECK(g_longest >= 71 && g_short_wgs <= 1024);
    tetri_destroy(h);
}

// How the host cuts a decode batch: equal ranges where there is much to read and fewer than two pairs per compute unit
// (the batches of test_gpu_decode_ranges.py's default rule are among these), equal parts or whole pairs otherwise.
void decode_division()
{
    const tetri_config c = {16, 8, 128, 16, 64, 64, 300, 8, TETRI_BF16};
    tetri_ctx *h = nullptr;
    CHECK(tetri_create(&c, &h) == TETRI_OK);
    const int32_t *meta = reinterpret_cast<const int32_t *>(g_any);
    auto cut = [&](int requests, int max_ctx, int fp8) {
        const tetri_status st = fp8 ? tetri_decode_attn_fp8(h, g_any, g_any, g_any, g_any, meta, meta, requests, max_ctx, 0.1f, 1.f, 1.f, 0, g_any, nullptr)
                                    : tetri_decode_attn(h, g_any, g_any, g_any, g_any, meta, meta, requests, max_ctx, 0.1f, g_any, nullptr);
        CHECK(st == TETRI_OK);
    };
    cut(12, 4700, 0);                             // 96 pairs x 147 steps x 16 KB = 231 MB
    CHECK(g_ranges == 32 && g_parts == 0);
    cut(12, 4000, 0);                             // 126 steps: 198 MB
    CHECK(g_ranges == 0 && g_parts == 5);
    cut(22, 4700, 1);                             // codes: 176 pairs x 147 x 8 KB = 212 MB
    CHECK(g_ranges == 32 && g_parts == 0);
    cut(12, 4700, 1);
    CHECK(g_ranges == 0 && g_parts == 5);
    cut(64, 4700, 0);                             // two pairs per compute unit
    CHECK(g_ranges == 0 && g_parts == 1);
    tetri_destroy(h);
}

}  // namespace

int main(int argc, char **argv)
{
    const std::string name = argc > 1 ? argv[1] : "";
    if (name == "static_decode_counters") static_decode_counters();
    else if (name == "counters_are_cleared") counters_are_cleared();
    else if (name == "planned_launches_overlap") planned_launches_overlap();
    else if (name == "upload_checks_the_device") upload_checks_the_device();
    else if (name == "uploads_name_no_stream_later") uploads_name_no_stream_later();
    else if (name == "choice_of_kernel") choice_of_kernel();
    else if (name == "short_output_stores") short_output_stores();
    else if (name == "next_chunk_rows") next_chunk_rows();
    else if (name == "new_row_stores") new_row_stores();
    else if (name == "carried_metadata") carried_metadata();
    else if (name == "short_teams") short_teams();
    else if (name == "decode_division") decode_division();
    else return 2;
    std::printf("%s: ok\n", name.c_str());
    return 0;
}
