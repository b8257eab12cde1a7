// Driver of the host-layer tests (built and run by tests/test_host_launches.py): the library's host layer
// (tetri_host.cpp, tetri_plan.cpp) linked with a HIP runtime and kernel launchers that only write down what
// they are asked for.  So what a call hands to a kernel, and which streams and events it touches, can be checked
// without a GPU, also where the real thing would be a race.  argv[1] names the check.
#include <hip/hip_runtime.h>

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

std::vector<const int32_t *> g_counters;      // the arrival counters of every launch that shares results, in order

float g_static_scratch[kDecodeStaticScratchBytes / 4];
int32_t g_static_counters[kDecodeStaticCounters];

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
hipError_t hipStreamQuery(hipStream_t) { return hipSuccess; }
hipError_t hipStreamIsCapturing(hipStream_t, hipStreamCaptureStatus *s) { *s = hipStreamCaptureStatusNone; return hipSuccess; }
hipError_t hipEventCreateWithFlags(hipEvent_t *, unsigned) { return hipErrorUnknown; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipErrorUnknown; }
hipError_t hipEventQuery(hipEvent_t) { return hipErrorUnknown; }
hipError_t hipEventSynchronize(hipEvent_t) { return hipErrorUnknown; }
hipError_t hipEventDestroy(hipEvent_t) { return hipErrorUnknown; }
hipError_t hipPointerGetAttributes(hipPointerAttribute_t *a, const void *) { a->type = hipMemoryTypeHost; return hipSuccess; }
}

// ---- the kernel launchers
hipError_t tetri_launch_attn(const tetri_ctx *, const AttnParams &p, int, bool, hipStream_t)
{
    if (p.stream_wgs > 0 || p.helpers > 0) g_counters.push_back(p.counters);
    return hipSuccess;
}
hipError_t tetri_launch_short(int, bool, const ShortParams &p, int, hipStream_t)
{
    if (p.splits > 1) g_counters.push_back(p.counters);
    return hipSuccess;
}
hipError_t tetri_launch_decode(const tetri_ctx *, const DecodeParams &p, hipStream_t)
{
    if (p.parts != 1) g_counters.push_back(p.counters);
    return hipSuccess;
}
hipError_t tetri_decode_static_memory(DecodeStatic *out)
{
    *out = {g_static_scratch, g_static_counters};
    return hipSuccess;
}
hipError_t tetri_launch_kv_transfer(const tetri_ctx *, const TransferParams &, int32_t, int32_t, bool, hipStream_t) { return hipSuccess; }
hipError_t tetri_launch_kv_export_fp8(const tetri_ctx *, const TransferParams &, int32_t, hipStream_t) { return hipSuccess; }
hipError_t tetri_launch_append(const tetri_ctx *, const AppendParams &, int32_t, hipStream_t) { return hipSuccess; }
hipError_t tetri_launch_upload(const int32_t *, int32_t *, int64_t, hipStream_t) { return hipSuccess; }

namespace {

alignas(16) char g_any[64];                   // stands for every device array: nothing is read

tetri_ctx *handle(int hq, int hkv, int d)
{
    const tetri_config c = {hq, hkv, d, 16, 256, 1024, 256, 8, TETRI_BF16};
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
    CHECK(g_counters.size() == 1 && in_handle_memory(g_counters[0]));
    decode(h, true);
    CHECK(g_counters.size() == 2 && !in_handle_memory(g_counters[1]));
    // as many (request, kv head)s as there are counters: a counter each, and not one more
    decode(h, true, kDecodeStaticCounters / 2);
    CHECK(g_counters.size() == 3);
    decode(h, true, kDecodeStaticCounters / 2 + 1);
    CHECK(g_counters.size() == 3);
    tetri_destroy(h);
}

}  // namespace

int main(int argc, char **argv)
{
    const std::string name = argc > 1 ? argv[1] : "";
    if (name == "static_decode_counters") static_decode_counters();
    else return 2;
    std::printf("%s: ok\n", name.c_str());
    return 0;
}
