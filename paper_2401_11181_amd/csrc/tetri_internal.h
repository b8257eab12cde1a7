// Internal declarations shared by the host layer and the kernel launchers of libtetri.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>
#include <atomic>
#include <string>

#include "tetri.h"

// Arrival counters of launches whose workgroups share results: kCounterSets sets, used in turn.  A launch leaves the
// set it used at zero and also zeroes the set after the next: so whatever a launch left behind is gone before its set's turn
// comes again, and launches that follow each other never touch each other's set, not even if they wrongly overlap.
constexpr int kCounterSets = 4;
struct CounterSets {
    int32_t *use, *clear;
};
inline CounterSets counter_sets(int32_t *first, int32_t n, uint32_t turn)
{
    return {first + (size_t)(turn % kCounterSets) * n, first + (size_t)((turn + 2) % kCounterSets) * n};
}

// The static device memory behind tetri_decode_attn_static: the parts of split requests, and arrival counters of their own,
// so that such a call shares nothing with the other launches of its handle.
constexpr size_t kDecodeStaticScratchBytes = (size_t)8 << 20;
constexpr int32_t kDecodeStaticCounters = 2048;
struct DecodeStatic {
    float *scratch = nullptr;
    int32_t *counters = nullptr;        // sets of kDecodeStaticCounters, zero when the library is loaded
    std::atomic<uint32_t> *turn = nullptr;  // the set of the device's next such call
};

// Partial results and arrival counters of launches on a division of the host's, which cuts tiles of launches of any size: apart
// from the handle's other scratch memory (decode, launches that divide themselves), whose users such launches may overlap.
struct PlanMemory {
    char *scratch = nullptr;        // 2 x scratch_units units
    int32_t *counters = nullptr;    // kCounterSets sets of n_counters
    uint32_t turn = 0;
};

struct tetri_ctx {
    tetri_config cfg;
    std::string err;
    int attn_variant = 0;   // 0 = library's choice, 1 / 2 = shared-tile kernel with 1 / 2 key parts, 3 = short kernel, 4 / 5 = host's division with 8 / 4 slots
    int split_keys = 1;     // 1 = launches with fewer than two row tiles per CU divide the stages of every head group evenly over the CUs
    int stream_wgs = 0;     // workgroups per head group of such a launch (0: as many as the device has CUs for); > 0 forces the mode
    int split_min_stages = 8;   // tail mode: the shortest key range that hands its tail to a helper workgroup
    int split_bias_stages = 6;  // a helper's overhead, in stages (see the kernel)
    int split_share_q8 = 85;    // the share of the remaining stages a tile hands over, in 1/256 (a third)
    bool division_set = false;  // one of the five options above has been set: the caller wants the shared-tile kernel
    int decode_parts = 0;       // key parts per (request, kv head) of the decode kernel (0: the library chooses)
    int decode_ranges = 0;      // equal ranges of a decode batch's steps per kv head (0: the library chooses)
    int transfer_slabs = 0;     // (K / V, head) slabs per workgroup of the export / import kernels (0: the library chooses)
    int device = 0;         // the device the handle was created on; its scratch memory lives there
    int num_cus = 0;
    char *scratch = nullptr;        // partial results of tiles shared by workgroups: 2 x scratch_units units
    int32_t *counters = nullptr;    // sets of n_counters arrival counters, and behind them a row of zeros
    size_t scratch_units = 0, unit_bytes = 0;
    int32_t n_counters = 0;
    uint32_t counter_turn = 0;      // the set of the next launch that uses one
    bool divide_launched = false;       // a prefill launch has used scratch and counters ...
    hipStream_t last_divide_stream = nullptr;   // ... the last one on this stream
    DecodeStatic decode_static;         // this device's memory of tetri_decode_attn_static
    // The first stream with such a launch owns the first of these for good (its launches follow each other: no event, which costs
    // a launch 0.5 to 0.9 us); all others take turns with the second, each launch signalling an event.
    PlanMemory plan_memory[2];
    bool plan_owned = false, plan_lent = false;     // the first has an owner, the second a last user
    hipStream_t plan_owner = nullptr, plan_borrower = nullptr;     // (compared, never named to the runtime: they may be gone)
    hipEvent_t plan_done = nullptr;     // the second's last launch
};

// The shared-tile kernel on a division made by the host (tetri_planned.hip): the jobs travel in the kernel arguments.  The eight
// XCDs form pools (one XCD each, or 2, 4 or 8 where there are few head groups); every pool has the same jobs, for its own
// head groups.
constexpr int kPlanSegs = 40, kPlanJobs = 160;
struct PlanJob {
    uint16_t seg_grp;             // segment | head group within the pool << 6
    uint16_t t0;                  // first row of the tile in its segment
    uint16_t begin, end;          // stages of the tile's key range (begin == end: none)
    uint16_t place;               // where in the pool the partial result of the tile's first piece goes
    uint8_t piece, npieces;
    uint16_t next;                // the workgroup's next job (always a later one), 0: none
    uint16_t pad;
};
struct __attribute__((aligned(16))) TilePlan {
    PlanJob job[kPlanJobs];       // workgroup w of a pool starts with job w
    int32_t seg[kPlanSegs][4];    // first row, rows, cached tokens of a segment
    int32_t rows;                 // chunk rows that belong to a request
    int32_t places;               // partial results of a pool (0: no tile is shared)
    int32_t wgs;                  // workgroups of a pool
    int32_t pad;
    hipEvent_t done;              // for the host: signalled when the launch has ended (null: none)
};

// Launch parameters of the attention kernels (passed by value).
struct AttnParams {
    const uint16_t *q, *k_new, *v_new, *pages;   // bf16 bit patterns
    const int32_t *bt, *cu, *ctx;
    uint16_t *out;
    uint16_t *pages_w;    // pool for the fused append (null when append_blocks == 0)
    int32_t S, C, Hq, Hkv, g;
    int32_t hpw;          // query heads handled by one workgroup (they share one kv head)
    int32_t rb;           // 32-row blocks handled by one workgroup
    int32_t hpw_shift, rb_shift;   // log2 of the two
    int32_t groups;       // Hq / hpw: head groups, one workgroup column each
    int32_t stream_wgs;   // workgroups per head group that share its stages evenly (0: one workgroup per row tile ...)
    int32_t helpers;      // ... plus, per head group, this many that take the tails of two tiles' key ranges each (0: none)
    int32_t tail_q8;      // the share of a tile's stages that goes to its helper, in 1/256
    int32_t split_min;    // only key ranges of at least this many stages hand a tail over
    int32_t split_bias;   // stages not counted when a key range's tail is measured
    int32_t n_counters;   // size of a set of arrival counters
    int32_t gpx;          // head groups per XCD
    uint32_t gpx_magic;   // ceil(2^32 / gpx), 0 for 1
    int32_t span_shift;   // a head group runs on 1 << span_shift XCDs (more than one only with gpx = 1)
    char *scratch;        // partial results of tiles shared by several workgroups
    int32_t *counters;    // one per (group, tile, slot), all zero when the launch begins
    int32_t *counters_next;   // the set of a later launch: zeroed by this one
    uint32_t kv_magic;    // the same for g / hpw: head group -> kv head
    int32_t max_blocks;
    int32_t tiles;        // upper bound of the number of row tiles of the chunk
    int32_t attn_grid;    // workgroups of the attention grid (a multiple of 8)
    int32_t append_blocks; // extra workgroups that do the fused KV append (0: none)
    int32_t attn_first;   // attention workgroups that precede them in the grid (a multiple of 8)
    float c;              // |scale| * log2(e)
    int32_t neg;          // 1 if scale < 0
    // FP8 cache (the kernel variant that reads a pool of E4M3 codes): cached K / V = value(code) * scale
    float k_scale, v_scale;
    float k_inv, v_inv;   // fl32(1 / scale): the fused append quantises with them
    const TilePlan *plan; // host memory: the host's division of the launch (null: none)
};

// The attention kernel for chunks with little work (tetri_short.hip).  What it reads of its arguments, behind the words that find a
// wavefront's row block: the chunk's row blocks travel in it.
constexpr int kShortSegs = 40, kShortUnits = 128;
// How the fused append stores new rows: by ordinary stores; written through the L2; past the caches, but for the last segment's, which may go on
// in the next chunk.
enum { kRowsCached, kRowsThrough, kRowsPast };
struct __attribute__((aligned(64))) ShortArgs {
    // (read together with the row block at the kernel's start: a cache line ...)
    const uint16_t *q, *k_new, *v_new, *pages;
    uint16_t *out, *pages_w;      // pages_w: pool for the fused append (null: none)
    const void *zero;             // a row of zeros
    int32_t Hq, Hkv;
    // (... and two words)
    int32_t g;
    int32_t out_past_l2;          // 1: the output rows are stored past the caches
    // (read where they are used)
    float c;                      // |scale| * log2(e)
    int32_t neg;                  // 1 if scale < 0
    float k_scale, v_scale, k_inv, v_inv;
    int32_t C, rows;              // chunk rows, and those that belong to a request
    float *scratch;               // splits > 1: partial results, [(unit * Hq + head) * splits + part][32 * D + 64] floats
    int32_t *counters;            // ... and arrival counters, one per (unit, head), zero before and after the launch
    int32_t *counters_next;       // the set of a later launch: zeroed by this one
    int32_t n_counters;           // size of a set
    int32_t fetch_wgs;            // workgroups that ask for rows of the next chunk (0: none)
    const uint16_t *next[3];      // ... of K, V and Q, and how many instructions of 1 KB go to each
    uint32_t next_kb[3];
    uint32_t next_bytes[2];       // what the rows take: K or V, and Q
    int32_t new_rows;             // how the fused append stores the chunk's K and V: kRowsCached ...
    // most work first, 64 bits each: segment (6), row block in it (7), the segment's rows (13) and first row (12), cached tokens (26)
    uint32_t unit[kShortUnits][2];
};

// A batch's metadata on its way to the device: len int32 of host memory for dev (16-byte aligned); host is null once it has been sent.
struct MetaUpload {
    const int32_t *host;
    int32_t *dev;
    int64_t len;
};

// The rows of the chunk that the caller's next launch is for (rows 0: not known), those of all chunks of the call, and how many KB of the
// former a wavefront of a launch asks for at most.
struct NextRows {
    const void *q, *k_new, *v_new;
    int32_t rows;
    int64_t call_rows;
};
constexpr int kFetchKB = 32;
// What a lane of instruction i of those asks for: 16 bytes of K (0), V (1) or Q (2), lanes past the end of the rows the last ones.
struct FetchAt {
    int32_t matrix;
    uint32_t byte;
};
__host__ __device__ inline FetchAt fetch_at(uint32_t i, uint32_t lane, uint32_t k_kb, uint32_t v_kb, uint32_t kv_bytes, uint32_t q_bytes)
{
    const int32_t matrix = i < k_kb ? 0 : (i < k_kb + v_kb ? 1 : 2);
    const uint32_t at = (i - (matrix == 0 ? 0 : (matrix == 1 ? k_kb : k_kb + v_kb))) * 1024 + lane * 16;
    const uint32_t last = (matrix == 2 ? q_bytes : kv_bytes) - 16;
    return {matrix, at < last ? at : last};
}

// The same with the metadata of the whole batch: the launch finds its page ids there and copies it to the device, for the launches
// behind it.  At most kShortCarry int32.
constexpr int64_t kShortCarry = 672;
struct __attribute__((aligned(64))) ShortCarry : ShortArgs {
    int32_t *meta_dev;
    int32_t meta_vectors;         // of 16 bytes
    int32_t pad2;
    uint32_t meta[kShortCarry];
};

// The launch as the host lays it out; what it adds goes to the kernel as leading scalars, some of them packed.
struct ShortParams : ShortArgs {
    const MetaUpload *carry;      // metadata that this launch takes along (null: none); bt lies in its dev then
    const int32_t *bt;
    int32_t max_blocks;
    int32_t first_wg[4];          // of the row blocks of 1, 2, 4 and 8 wavefronts: the classes follow each other from 8 down ...
    int32_t first_unit[4];        // ... and their first row blocks
    int32_t units;                // row blocks of 32 rows
    int32_t attn_wgs;             // workgroups but for those that write the padding rows
    int32_t zero_wgs;             // ... and those
    int32_t splits;               // workgroups that share the keys of a row block of one head (> 1: one class, the whole workgroup)
    uint32_t splits_magic;        // ceil(2^32 / d), 0 for 1
    int32_t hpx;                  // query heads whose kv head is x modulo 1 << rshift: as many for every x
    uint32_t hpx_magic;
    int32_t hkx;                  // ... and such kv heads
    uint32_t hkx_magic;
    int32_t rshift;
    int32_t spread;               // 1: one team to a workgroup
};

// Row blocks of the classes and the shape of the launch, in three words.  (The class of the largest teams starts at workgroup 0 and row
// block 0: neither travels.)  Row blocks <= kShortUnits, splits <= 16, rshift <= 3, heads below 65536: plan_short refuses what is
// not below 2^32 as row blocks x heads x heads.
struct ShortWords {
    uint32_t first_units, shape, per_x;
};
struct ShortShapeWords {
    int32_t first_unit[3], units, splits, rshift, spread, hpx, hkx;
};
__host__ __device__ inline ShortWords short_pack(const ShortParams &p)
{
    static_assert(kShortUnits <= 255, "row blocks in a byte");
    return {(uint32_t)p.first_unit[0] | (uint32_t)p.first_unit[1] << 8 | (uint32_t)p.first_unit[2] << 16 | (uint32_t)p.units << 24,
            (uint32_t)p.splits | (uint32_t)p.rshift << 8 | (uint32_t)p.spread << 10, (uint32_t)p.hpx | (uint32_t)p.hkx << 16};
}
__host__ __device__ inline ShortShapeWords short_unpack(const ShortWords &w)
{
    return {{(int32_t)(w.first_units & 255), (int32_t)(w.first_units >> 8 & 255), (int32_t)(w.first_units >> 16 & 255)}, (int32_t)(w.first_units >> 24),
            (int32_t)(w.shape & 255), (int32_t)(w.shape >> 8 & 3), (int32_t)(w.shape >> 10), (int32_t)(w.per_x & 0xffff), (int32_t)(w.per_x >> 16)};
}

struct AppendParams {
    const uint16_t *k_new, *v_new;
    uint16_t *pages;
    const int32_t *bt, *cu, *ctx;
    int32_t S, Hkv, D, max_blocks;
};

// Launch parameters of the KV export / import kernels.
struct TransferParams {
    uint16_t *pool;       // the paged pool (read by export, written by import)
    uint16_t *buf;        // the dense transfer buffer (written by export, read by import)
    const int32_t *bt, *cu, *first;   // first may be null: every range starts at token 0
    int32_t R, Hkv, max_blocks;
    int32_t slabs_per_wg; // (K / V, head) slabs one workgroup moves
    int32_t slab_groups;  // runs of that many slabs
    uint32_t groups_magic; // ceil(2^32 / slab_groups), 0 for 1
    float k_inv, v_inv;   // quantising export: fl32(1 / scale) of the K and of the V half
};

// Most requests of a decode batch whose steps are divided evenly (a lane of a wavefront looks at up to 16 of them).
constexpr int kDecodeLookup = 1024;

// What the decode-iteration kernel reads of its arguments behind the leading scalars: what it needs up to the end of its loop in
// one cache line (the structure starts 8 bytes before one), the others behind.  (Heads of 4 x 64, 6 requests of up to 184 tokens
// over codes: 6.14 us with Hq and g in the line before c and k_scale, this way 6.07.)
struct DecodeArgs {
    uint16_t *out;
    const uint16_t *k_new, *v_new;
    int32_t Hq, g;
    float c;              // |scale| * log2(e)
    int32_t neg;          // 1 if scale < 0
    float k_scale, v_inv; // FP8 pool: the scales and fl32(1 / scale)
    int32_t ranges;       // parts == 0: the steps of the batch in that many equal ranges, a workgroup each per kv head
    int32_t min_steps;    // ... of at least this many steps
    int32_t *counters_next;   // the set of a later launch: zeroed by this one
    int32_t n_counters;   // size of a set; 0: no (request, kv head) is shared, the launch touches no counters
    float out_scale;      // factor on the finished output: v_scale for an FP8 pool, else 1
    uint16_t *pages_w;    // pool for the fused append of the new token (null: no append)
    float *partial;       // scratch: partial results of (request, kv head)s shared by workgroups
    int32_t *counters;    // ... and their arrival counters, zero before and after the launch
    float v_scale, k_inv;
};

// The launch as the host lays it out: what it adds goes to the kernel as leading scalars, but for the choice of the kernel.
struct DecodeParams : DecodeArgs {
    const int32_t *ctx, *bt;
    const uint16_t *pages, *q;
    int32_t max_blocks, Hkv;
    uint32_t hkv_magic;   // ceil(2^32 / Hkv), 0 for 1
    int32_t parts;        // > 0: each (request, kv head)'s keys in that many equal parts, a workgroup each
    int32_t B;
    int32_t fp8;          // 1: the pool holds E4M3 codes (one byte per element) with per-tensor scales
};

hipError_t tetri_launch_attn(const tetri_ctx *h, const AttnParams &p, int key_parts, bool fp8_pool, hipStream_t stream);
hipError_t tetri_launch_planned(const AttnParams &p, bool fp8_pool, hipStream_t stream);      // (tetri_launch_attn's, for p.plan)
hipError_t tetri_launch_short(int head_dim, bool fp8_pool, const ShortParams &p, int wavefronts, hipStream_t stream);
hipError_t tetri_launch_kv_transfer(const tetri_ctx *h, const TransferParams &p, int32_t row_units, int32_t tiles,
                                    bool to_pool, hipStream_t stream);
hipError_t tetri_launch_kv_export_fp8(const tetri_ctx *h, const TransferParams &p, int32_t tiles, hipStream_t stream);
hipError_t tetri_launch_decode(const tetri_ctx *h, const DecodeParams &p, hipStream_t stream);
// Device addresses (on the current device) of the static memory of tetri_decode_attn_static.
hipError_t tetri_decode_static_memory(DecodeStatic *out);
hipError_t tetri_launch_append(const tetri_ctx *h, const AppendParams &p, int32_t chunk_rows, hipStream_t stream);

// Copies len int32 (rounded up to a multiple of 4) from pinned host memory to the device, both 16-byte aligned; `done` (null:
// none) is signalled when that has ended.
hipError_t tetri_launch_upload(const int32_t *pinned, int32_t *dev, int64_t len, hipStream_t stream, hipEvent_t done);
// The same for at most kUploadInline int32, which travel in the kernel's arguments: host memory is read before this returns.
constexpr int64_t kUploadInline = 896;
hipError_t tetri_launch_upload_inline(const int32_t *host, int32_t *dev, int64_t len, hipStream_t stream);
