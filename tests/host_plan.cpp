// Driver of tests/test_host_plan.py: the host layer (tetri_host.cpp, tetri_plan.cpp) with launchers that check the division of
// a launch of the shared-tile kernel instead of running it.  Draws chunks (argv: seed, number of draws, heads, kv heads, chunk size,
// "attn_variant" (4), "split_keys" (1)) and fails if a stage of a row tile is missing or done twice, a partial result or an arrival counter lies outside the handle's
// memory or belongs to two tiles, a workgroup's chain of jobs does not end, or a tile is shared in spite of split_keys = 0.  With "time" in
// place of the last two: chunks of packed short prompts, some behind a carried-over one, by the library's own choice of kernel;
// prints what a call takes of the host.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdio>
#include <cmath>
#include <cstdlib>
#include <cstring>
#include <ctime>
#include <map>
#include <random>
#include <set>
#include <tuple>
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

hipError_t tetri_launch_short(int, bool, const ShortParams &, int, hipStream_t) { return hipSuccess; }
hipError_t tetri_launch_decode(const tetri_ctx *, const DecodeParams &, hipStream_t) { return hipSuccess; }
hipError_t tetri_decode_static_memory(DecodeStatic *out) { *out = {}; return hipSuccess; }
hipError_t tetri_launch_kv_transfer(const tetri_ctx *, const TransferParams &, int32_t, int32_t, bool, hipStream_t) { return hipSuccess; }
hipError_t tetri_launch_kv_export_fp8(const tetri_ctx *, const TransferParams &, int32_t, hipStream_t) { return hipSuccess; }
hipError_t tetri_launch_append(const tetri_ctx *, const AppendParams &, int32_t, hipStream_t) { return hipSuccess; }
hipError_t tetri_launch_upload(const int32_t *, int32_t *, int64_t, hipStream_t, hipEvent_t) { return hipSuccess; }
hipError_t tetri_launch_upload_inline(const int32_t *, int32_t *, int64_t, hipStream_t) { return hipSuccess; }

namespace {

std::vector<int32_t> g_cu, g_ctx;
int g_planned = 0, g_shared = 0, g_eight = 0, g_variant = 0;
bool g_timed = false;

void check_plan(const tetri_ctx *h, const AttnParams &p)
{
    const TilePlan &plan = *p.plan;
    const int pools = 8 >> p.span_shift, rows = 32 * p.rb, slots = p.hpw * p.rb;
    CHECK((g_variant == 0 ? slots == 4 || slots == 8 : slots == (g_variant == 4 ? 8 : 4)) && p.groups * p.hpw == p.Hq && p.g % p.hpw == 0 && (1 << p.hpw_shift) == p.hpw && (1 << p.rb_shift) == p.rb);
    CHECK(pools * p.gpx >= p.groups && p.attn_grid % 8 == 0 && (p.attn_grid / 8) << p.span_shift >= plan.wgs && plan.wgs <= kPlanJobs);
    CHECK((int64_t)pools * plan.places * slots <= (int64_t)(2 * h->scratch_units) && (int64_t)pools * plan.places * slots <= p.n_counters);
    CHECK(plan.places == 0 || h->split_keys != 0);
    g_eight += slots == 8;
    CHECK(plan.rows == g_cu.back());
    struct Piece { int begin, end, piece, npieces, place; };
    std::map<std::tuple<int, int, int>, std::vector<Piece>> tiles;       // (group, segment, first row)
    std::set<int> seen;
    for (int w = 0; w < plan.wgs; ++w) {
        int open = 0;                             // hand-overs the workgroup leaves open behind it
        for (int i = w, last = -1;; i = plan.job[i].next) {
            CHECK(i > last && i < kPlanJobs && (last < 0 || i >= plan.wgs) && seen.insert(i).second);
            const PlanJob &j = plan.job[i];
            if (j.begin < j.end) tiles[{j.seg_grp >> 6, j.seg_grp & 63, j.t0}].push_back({j.begin, j.end, j.piece, j.npieces, j.place});
            last = i;
            if (j.next == 0) break;
            open += j.npieces > 1;
            CHECK(open <= 1);
        }
    }
    size_t want = 0;
    std::set<int> places;
    bool shared = false;
    for (size_t s = 0; s < g_ctx.size(); ++s) {
        const int n = g_cu[s + 1] - g_cu[s];
        CHECK(plan.seg[s][0] == g_cu[s] && plan.seg[s][1] == n && plan.seg[s][2] == g_ctx[s]);
        for (int t0 = 0; t0 < n; t0 += rows)
            for (int g = 0; g < p.gpx; ++g, ++want) {
                auto at = tiles.find({g, (int)s, t0});
                CHECK(at != tiles.end());
                std::vector<Piece> &v = at->second;
                std::sort(v.begin(), v.end(), [](const Piece &a, const Piece &b) { return a.piece < b.piece; });
                int pos = 0;
                for (size_t i = 0; i < v.size(); ++i) {
                    CHECK(v[i].begin == pos && v[i].piece == (int)i && v[i].npieces == (int)v.size() && v[i].place == v[0].place);
                    pos = v[i].end;
                    if (v.size() > 1) CHECK(v[0].place + (int)i < plan.places && places.insert(v[0].place + (int)i).second);
                }
                shared = shared || v.size() > 1;
                CHECK(pos == (g_ctx[s] + 127) / 128 + (std::min(n, t0 + rows) + 127) / 128);
            }
    }
    CHECK(want == tiles.size() && shared == (plan.places != 0));
}

}  // namespace

hipError_t tetri_launch_attn(const tetri_ctx *h, const AttnParams &p, int, bool, hipStream_t)
{
    ++g_shared;
    if (p.plan != nullptr) {
        ++g_planned;
        if (!g_timed) check_plan(h, p);
    }
    return hipSuccess;
}

int main(int argc, char **argv)
{
    g_timed = argc == 7 && std::strcmp(argv[6], "time") == 0;
    CHECK(argc == 6 || argc == 8 || g_timed);
    g_variant = g_timed ? 0 : (argc == 8 ? std::atoi(argv[6]) : 4);
    std::mt19937 rng((unsigned)std::atoi(argv[1]));
    const int draws = std::atoi(argv[2]), hq = std::atoi(argv[3]), hkv = std::atoi(argv[4]), chunk = std::atoi(argv[5]);
    alignas(16) static char any[64];
    const int32_t *meta = reinterpret_cast<const int32_t *>(any);
    const tetri_config c = {hq, hkv, 128, 16, chunk, 1 << 20, 4096, std::min(chunk, 64), TETRI_BF16};
    tetri_ctx *h = nullptr;
    CHECK(tetri_create(&c, &h) == TETRI_OK);
    CHECK(tetri_set_option(h, "attn_variant", g_variant) == TETRI_OK);
    if (argc == 8 && std::atoi(argv[7]) == 0) CHECK(tetri_set_option(h, "split_keys", 0) == TETRI_OK);
    auto upto = [&](int n) { return (int)(rng() % (unsigned)n); };
    std::vector<double> us;
    for (int d = 0; d < draws && g_timed; ++d) {
        g_cu.assign(1, 0);
        g_ctx.clear();
        while (g_cu.back() < chunk && g_ctx.size() < 40) {
            const int n = (int)std::exp(4.5 + 0.8 * (upto(1000) + upto(1000) + upto(1000) - 1500) / 500.0);
            g_cu.push_back(std::min(chunk, g_cu.back() + std::min(std::max(n, 16), 512)));
            g_ctx.push_back(g_ctx.empty() ? upto(2) * upto(3000) : 0);
        }
        double best = 1e9;
        for (int i = 0; i < 5; ++i) {
            timespec a, b;
            clock_gettime(CLOCK_THREAD_CPUTIME_ID, &a);
            CHECK(tetri_chunk_prefill_planned(h, any, any, any, any, meta, meta, meta, (int32_t)g_ctx.size(), 0.1f, 1, 0, 1.f, 1.f, g_cu.data(),
                                              g_ctx.data(), any, nullptr) == TETRI_OK);
            clock_gettime(CLOCK_THREAD_CPUTIME_ID, &b);
            best = std::min(best, 1e6 * (double)(b.tv_sec - a.tv_sec) + 1e-3 * (double)(b.tv_nsec - a.tv_nsec));
        }
        us.push_back(best);
    }
    if (g_timed) {
        std::sort(us.begin(), us.end());
        std::printf("%.2f %.2f\n", us[us.size() / 2], us[us.size() * 9 / 10]);
        tetri_destroy(h);
        return 0;
    }
    for (int d = 0; d < draws; ++d) {
        const int segs = 1 + (upto(3) == 0 ? upto(std::min(44, chunk)) : upto(std::min(4, chunk)));
        std::set<int> cuts;
        while ((int)cuts.size() < segs) cuts.insert(1 + upto(chunk));
        if (upto(2)) { cuts.erase(*cuts.rbegin()); cuts.insert(chunk); }
        g_cu.assign(1, 0);
        g_cu.insert(g_cu.end(), cuts.begin(), cuts.end());
        g_ctx.clear();
        for (size_t s = 0; s + 1 < g_cu.size(); ++s) g_ctx.push_back(upto(3) == 0 ? 0 : upto(1 << (4 + upto(12))));
        CHECK(tetri_chunk_prefill_planned(h, any, any, any, any, meta, meta, meta, (int32_t)g_ctx.size(), 0.1f, upto(2), upto(2), 1.f, 1.f,
                                          g_cu.data(), g_ctx.data(), any, nullptr) == TETRI_OK);
    }
    tetri_destroy(h);
    std::printf("%d launches, %d on a division of the host\n", g_shared, g_planned);
    if (argc == 8) std::printf("with eight slots: %d\n", g_eight);
    return 0;
}
