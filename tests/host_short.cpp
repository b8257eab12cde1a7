// Driver of tests/test_host_short.py and tests/test_host_choice.py: the host layer (tetri_host.cpp, tetri_plan.cpp) with a launcher that walks the grid of the
// kernel for chunks with little work as its wavefronts do, instead of running it.  Draws chunks (argv: seed, number of draws, heads, kv
// heads, head dim, chunk size) and fails if a 32-key step of a row block is missing or done twice, a row block is not the
// chunk's, or a partial result lies outside the handle's memory.  Prints how many row blocks had teams of 1, 2, 4 and 8 wavefronts
// and how many had their keys split over workgroups.  With the heads alone (argv: heads, kv heads) it reads chunks from the standard input (FP8
// or not, number of segments, rows and cached tokens of each) and prints the kernel the library's own rule gives each of them.  Without arguments: the
// packed words of a launch at the edges of their fields.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <random>
#include <set>
#include <vector>

#include "tetri_internal.h"

#define CHECK(cond)                                                                       \
    do {                                                                                  \
        if (!(cond)) {                                                                    \
            std::fprintf(stderr, "%s:%d: check failed: %s\n", __FILE__, __LINE__, #cond); \
            std::exit(1);                                                                 \
        }                                                                                 \
    } while (0)

extern "C" {
hipError_t hipGetDeviceCount(int *n) { *n = 1; return hipSuccess; }
hipError_t hipGetDevice(int *d) { *d = 0; return hipSuccess; }
hipError_t hipGetDeviceProperties(hipDeviceProp_t *p, int) { std::memset(p, 0, sizeof *p); p->multiProcessorCount = 256; return hipSuccess; }
const char *hipGetErrorString(hipError_t) { return "stub"; }
hipError_t hipGetLastError() { return hipSuccess; }
hipError_t hipMalloc(void **p, size_t n) { *p = std::malloc(n); return hipSuccess; }
hipError_t hipFree(void *p) { std::free(p); return hipSuccess; }
hipError_t hipMemset(void *, int, size_t) { return hipSuccess; }
hipError_t hipMemcpy(void *, const void *, size_t, hipMemcpyKind) { return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipStreamQuery(hipStream_t) { return hipSuccess; }
hipError_t hipStreamIsCapturing(hipStream_t, hipStreamCaptureStatus *s) { *s = hipStreamCaptureStatusNone; return hipSuccess; }
hipError_t hipEventCreateWithFlags(hipEvent_t *, unsigned) { return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipEventQuery(hipEvent_t) { return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
hipError_t hipPointerGetAttributes(hipPointerAttribute_t *a, const void *) { a->type = hipMemoryTypeHost; return hipSuccess; }
}

hipError_t tetri_launch_decode(const tetri_ctx *, const DecodeParams &, hipStream_t) { return hipSuccess; }
hipError_t tetri_decode_static_memory(DecodeStatic *out) { *out = {}; return hipSuccess; }
hipError_t tetri_launch_kv_transfer(const tetri_ctx *, const TransferParams &, int32_t, int32_t, bool, hipStream_t) { return hipSuccess; }
hipError_t tetri_launch_kv_export_fp8(const tetri_ctx *, const TransferParams &, int32_t, hipStream_t) { return hipSuccess; }
hipError_t tetri_launch_append(const tetri_ctx *, const AppendParams &, int32_t, hipStream_t) { return hipSuccess; }
hipError_t tetri_launch_upload(const int32_t *, int32_t *, int64_t, hipStream_t, hipEvent_t) { return hipSuccess; }
hipError_t tetri_launch_upload_inline(const int32_t *, int32_t *, int64_t, hipStream_t) { return hipSuccess; }

namespace {

std::vector<int32_t> g_cu, g_ctx;
const char *g_taken = "";
const tetri_ctx *g_h = nullptr;
int g_launches = 0, g_teams[4] = {0, 0, 0, 0}, g_split = 0, g_most_units = 0, g_most_splits = 0;

uint32_t div_by(uint32_t n, uint32_t magic) { return magic == 0 ? n : (uint32_t)(((uint64_t)n * magic) >> 32); }

// The words that the kernel gets of a launch say what the host laid out.
void check_words(const ShortParams &p)
{
    const ShortShapeWords s = short_unpack(short_pack(p));
    CHECK(p.first_wg[3] == 0 && p.first_unit[3] == 0);                 // (neither travels)
    for (int tl = 0; tl < 3; ++tl) CHECK(s.first_unit[tl] == p.first_unit[tl]);
    CHECK(s.units == p.units && s.splits == p.splits && s.rshift == p.rshift && s.spread == p.spread && s.hpx == p.hpx && s.hkx == p.hkx);
}

// ... at the edges of what plan_short lays out, every field at its largest and smallest beside the others
int words()
{
    int n = 0;
    for (int units : {1, 2, 127, kShortUnits})
        for (int f0 : {0, 1, units - 1, units})
            for (int f1 : {0, f0 / 2, f0})
                for (int f2 : {0, f1 / 2, f1})
                    for (int splits : {1, 2, 15, 16})
                        for (int rshift : {0, 1, 2, 3})
                            for (int spread : {0, 1})
                                for (int hpx : {1, 40, 0xffff})
                                    for (int hkx : {1, 5, hpx}) {
                                        ShortParams p = {};
                                        p.units = units; p.first_unit[0] = f0; p.first_unit[1] = f1; p.first_unit[2] = f2;
                                        p.splits = splits; p.rshift = rshift; p.spread = spread; p.hpx = hpx; p.hkx = hkx;
                                        check_words(p);
                                        ++n;
                                    }
    std::printf("%d launches\n", n);
    return 0;
}

int choices(int hq, int hkv)
{
    alignas(16) static char any[64];
    const int32_t *meta = reinterpret_cast<const int32_t *>(any);
    int fp8, segs;
    while (std::scanf("%d %d", &fp8, &segs) == 2) {
        std::vector<int32_t> cu(1, 0), ctx;
        for (int i = 0; i < segs; ++i) {
            int rows, cached;
            CHECK(std::scanf("%d %d", &rows, &cached) == 2);
            cu.push_back(cu.back() + rows);
            ctx.push_back(cached);
        }
        const tetri_config c = {hq, hkv, 128, 16, cu.back(), 1 << 20, 4096, std::min(cu.back(), 64), TETRI_BF16};
        tetri_ctx *h = nullptr;
        CHECK(tetri_create(&c, &h) == TETRI_OK);
        g_cu = cu;
        g_ctx = ctx;
        CHECK(tetri_chunk_prefill_planned(h, any, any, any, any, meta, meta, meta, segs, 0.1f, 0, fp8, 1.f, 1.f, cu.data(), ctx.data(), any, nullptr) == TETRI_OK);
        std::printf("%s\n", g_taken);
        tetri_destroy(h);
    }
    return 0;
}

}  // namespace

hipError_t tetri_launch_attn(const tetri_ctx *, const AttnParams &p, int, bool, hipStream_t)
{
    g_taken = p.plan == nullptr ? "self" : (p.hpw * p.rb == 8 ? "eight" : "four");
    return hipSuccess;
}

hipError_t tetri_launch_short(int D, bool, const ShortParams &p, int wavefronts, hipStream_t)
{
    ++g_launches;
    g_taken = "short";
    if (g_h == nullptr) return hipSuccess;
    CHECK(wavefronts == 4 || wavefronts == 8);
    check_words(p);
    g_most_units = std::max(g_most_units, p.units);
    g_most_splits = std::max(g_most_splits, p.splits);
    const int nwl = wavefronts == 8 ? 3 : 2;
    CHECK(p.units >= 1 && p.units <= kShortUnits && p.rows == g_cu.back() && p.hpx << p.rshift == p.Hq && p.hkx << p.rshift == p.Hkv);
    std::vector<std::vector<int>> done((size_t)p.units * p.Hq);          // how often each step ran
    for (int w = 0; w < p.attn_wgs; ++w) {
        int tl = 0;
        while (tl < 3 && w < p.first_wg[tl]) ++tl;
        CHECK(tl <= nwl && w >= p.first_wg[tl] && (p.splits == 1 || tl == nwl));
        const int T = 1 << tl, u_end = tl == 0 ? p.units : p.first_unit[tl - 1], pack = p.spread ? 0 : nwl - tl;
        const uint32_t r = (uint32_t)(w - p.first_wg[tl]), j = p.splits > 1 ? div_by(r, p.splits_magic) : r;
        const int part = p.splits > 1 ? (int)(r - j * p.splits) : 0;
        CHECK(part >= 0 && part < p.splits);
        const int x = j & ((1 << p.rshift) - 1);
        for (int wave = 0; wave < wavefronts; ++wave) {
            const int team = wave >> tl, item = (int)(((j >> p.rshift) << pack) + (uint32_t)team), rank = wave & (T - 1);
            const int ul = (int)div_by((uint32_t)item, p.hpx_magic), hh = item - ul * p.hpx;
            const int grp = (int)div_by((uint32_t)hh, p.hkx_magic), kh = x + ((hh - grp * p.hkx) << p.rshift);
            const int u = p.first_unit[tl] + ul;
            if (u >= u_end || team >> pack != 0) continue;
            CHECK(hh >= 0 && hh < p.hpx && kh >= 0 && kh < p.Hkv && grp < p.g);
            const int head = kh * p.g + grp;
            const uint32_t lo = p.unit[u][0], hi = p.unit[u][1];
            const int seg = lo & 63, t0 = (lo >> 6 & 127) * 32, n = lo >> 13 & 8191, row0 = (int)(lo >> 26 | (hi >> 26) << 6), L = hi & 0x3ffffff;
            CHECK(seg < (int)g_ctx.size() && row0 == g_cu[seg] && n == g_cu[seg + 1] - g_cu[seg] && t0 < n && L == g_ctx[seg]);
            const int steps = (L + 31) / 32 + t0 / 32 + 1, spp = (steps + p.splits - 1) / p.splits;
            if (p.splits > 1) CHECK((int64_t)p.units * p.Hq <= p.n_counters && (int64_t)p.units * p.Hq * p.splits * (32 * D + 64) * 4 <=
                                    (int64_t)(2 * g_h->scratch_units * g_h->unit_bytes));
            std::vector<int> &d = done[(size_t)u * p.Hq + head];
            d.resize(steps);
            for (int s = part * spp + rank; s < std::min(steps, (part + 1) * spp); s += T) ++d[s];
            if (rank == 0 && part == 0 && head == 0) {
                ++g_teams[tl];
                g_split += p.splits > 1;
            }
        }
    }
    std::set<std::pair<int, int>> blocks;
    for (int u = 0; u < p.units; ++u) {
        blocks.insert({p.unit[u][0] & 63, p.unit[u][0] >> 6 & 127});
        for (int head = 0; head < p.Hq; ++head) {
            const std::vector<int> &d = done[(size_t)u * p.Hq + head];
            CHECK(!d.empty());
            for (int times : d) CHECK(times == 1);
        }
    }
    size_t want = 0;
    for (size_t s = 0; s < g_ctx.size(); ++s) want += (g_cu[s + 1] - g_cu[s] + 31) / 32;
    CHECK(blocks.size() == want);
    return hipSuccess;
}

int main(int argc, char **argv)
{
    if (argc == 1) return words();
    if (argc == 3) return choices(std::atoi(argv[1]), std::atoi(argv[2]));
    CHECK(argc == 7);
    std::mt19937 rng((unsigned)std::atoi(argv[1]));
    const int draws = std::atoi(argv[2]), hq = std::atoi(argv[3]), hkv = std::atoi(argv[4]), d = std::atoi(argv[5]), chunk = std::atoi(argv[6]);
    alignas(16) static char any[64];
    const int32_t *meta = reinterpret_cast<const int32_t *>(any);
    const tetri_config c = {hq, hkv, d, 16, chunk, 1 << 20, 4096, std::min(chunk, 64), TETRI_BF16};
    tetri_ctx *h = nullptr;
    CHECK(tetri_create(&c, &h) == TETRI_OK);
    CHECK(tetri_set_option(h, "attn_variant", 3) == TETRI_OK);
    g_h = h;
    auto upto = [&](int n) { return (int)(rng() % (unsigned)n); };
    for (int i = 0; i < draws; ++i) {
        const int segs = 1 + (upto(3) == 0 ? upto(std::min(44, chunk)) : upto(std::min(4, chunk)));
        std::set<int> cuts;
        while ((int)cuts.size() < segs) cuts.insert(1 + upto(chunk));
        g_cu.assign(1, 0);
        g_cu.insert(g_cu.end(), cuts.begin(), cuts.end());
        g_ctx.clear();
        for (size_t s = 0; s + 1 < g_cu.size(); ++s) g_ctx.push_back(upto(3) == 0 ? 0 : upto(1 << (3 + upto(11))));
        CHECK(tetri_chunk_prefill_planned(h, any, any, any, any, meta, meta, meta, (int32_t)g_ctx.size(), 0.1f, upto(2), upto(2), 1.f, 1.f,
                                          g_cu.data(), g_ctx.data(), any, nullptr) == TETRI_OK);
    }
    tetri_destroy(h);
    std::printf("%d launches, row blocks by team %d %d %d %d, split %d, at most %d row blocks, %d parts\n", g_launches, g_teams[0], g_teams[1], g_teams[2], g_teams[3],
                g_split, g_most_units, g_most_splits);
    return 0;
}
