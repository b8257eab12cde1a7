// One decode iteration over the paged KV cache for gfx950: the counterpart, on the decode instance, of
// the chunked-prefill kernel (TetriInfer Sec. 2.1: the decode phase produces one token per iteration
// and its query attends to the request's cached keys and values; Sec. 3.4: the decode instance batches
// the steps of many requests over a paged cache).
//
// The work is reading every cached K and V byte once: HBM-bound (per request and kv head 4 * D bytes
// per cached token against 4 * D * g flops).  Design:
//   * the g query heads that share a kv head are the columns of one matrix product, so K and V are read once for
//     all of them; a step is 32 keys of one (request, kv head);
//   * a batch is cut in one of three ways, which the host chooses (tetri_host.cpp, decode_common): a workgroup per
//     (request, kv head); every (request, kv head) in equal parts, a workgroup each, where there are few of them and little to
//     read; or, where there are few and much to read, the steps of the whole batch, request after request, in equal ranges,
//     for every kv head the same ones: a workgroup has one range of one kv head, so that all of them have the same number
//     of steps however the context lengths fall.  That division is worked out on the device from the context lengths.
//     (Equal parts left a batch of 16 to 8192 tokens waiting for its longest: 4.2 TB/s.)  Neighbouring workgroups take
//     different kv heads of the same range or part: what they read at a time lies in the same pages (ranges cut across the
//     heads instead had 2048 pages in use at once and were 10 % slower);
//   * the wavefronts of a workgroup take its steps in turn, each with K and V tiles of its own; the loads of a
//     wavefront's next step are in flight while it computes, across requests, and no barrier stands between steps.  Eight
//     wavefronts to a compute unit keep about 100 KB of loads in flight there;
//   * K and V go straight from global memory into the tiles (16 bytes per lane per instruction, swizzled so that the
//     fragment reads are conflict-free); scores and the PV product run on the matrix cores (S^T = K Q^T, O^T += V^T P^T
//     with 32x32x16 bf16 MFMA; only g of the 32 columns are real, which costs nothing on a kernel that waits for
//     memory), V is transposed on the way out of LDS by ds_read_b64_tr_b16;
//   * at the end of a request the wavefronts merge in LDS; a request cut between workgroups is finished by the one that
//     arrives last, from the partial results in scratch memory, in the order of the parts (the result does not
//     depend on who that is).  Nobody waits; there is no second kernel.
// Keys past the end of a request's cache are loaded from a row of zeros and masked, so that stale
// page contents (which may be NaN bit patterns) never reach an MFMA.
//
// FP8 cache (template flag FP8; this build's extension, not the paper's): the pool holds E4M3 codes with one scale per
// tensor.  The tiles hold codes, half the bytes, so that two steps fit and a wavefront has as many bytes in flight as with
// the 16-bit cache.  K fragments are read as 8 codes per lane, V fragments by ds_read_b64_tr_b8 (8 keys of one d per lane),
// and become bf16 in registers (v_cvt_scalef32_pk_bf16_fp8, exact: a code has four significant bits).  (Codes that went
// through registers into bf16 tiles cost as many conversions, a second trip through LDS and 32 registers.)  The
// scales are not applied per element: the K scale multiplies the scores of cached keys, the V scale the finished output;
// the new token, which is not quantised, is a step of its own (one key in a matrix product) with its weight divided by the
// V scale.
#include <mutex>

#include "attn_common.h"

namespace {

using namespace tetri_dev;

constexpr int kMergeCols = 4;     // query heads whose partial O the merge area in LDS holds at a time

// A workgroup's partial result: g rows of D floats (unnormalised O), then g of m and g of the row sum.
template <int D> __device__ __forceinline__ int part_floats(int g) { return g * D + ((2 * g + 3) & ~3); }

__device__ __forceinline__ float load_coherent(const float *p)
{
    return __hip_atomic_load(reinterpret_cast<const __attribute__((address_space(1))) float *>((uintptr_t)p), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ float2 load_coherent2(const float *p)
{
    const uint64_t v = __hip_atomic_load(reinterpret_cast<const __attribute__((address_space(1))) uint64_t *>((uintptr_t)p), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    return make_float2(__builtin_bit_cast(float, (uint32_t)v), __builtin_bit_cast(float, (uint32_t)(v >> 32)));
}

__device__ __forceinline__ void store_coherent2(float *p, float x, float y)
{
    const uint64_t v = (uint64_t)__builtin_bit_cast(uint32_t, x) | (uint64_t)__builtin_bit_cast(uint32_t, y) << 32;
    __hip_atomic_store(reinterpret_cast<__attribute__((address_space(1))) uint64_t *>((uintptr_t)p), v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// How rows of K and V lie in a tile: RB bytes per row, 16-byte chunks XOR-ed by the row so that 16-lane groups of a fragment
// read meet no bank twice.
template <int D, bool FP8> struct Tile {
    static constexpr int RB = FP8 ? D : 2 * D, BYTES = 32 * RB, CH = RB / 16;
    static constexpr int NI = BYTES / 1024, RPI = 1024 / RB;      // load instructions of a tile, rows of one
    static constexpr int PI = 16 / RPI;                           // ... of a page's 16 rows
    static __device__ __forceinline__ constexpr int swizzle(int row, bool is_v)
    {
        return FP8 ? (D == 128 ? row & 7 : (row >> 2) & 3) : (is_v ? v_swizzle<D>(row) : k_swizzle<D>(row));
    }
};

// A page's 16 rows of one head, K or V, into a tile.
template <int D, bool FP8>
__device__ __forceinline__ void issue_page(const char *base, uint32_t off, bool is_v, uint32_t lds)
{
    typedef Tile<D, FP8> T;
    uint32_t v[T::PI];
#pragma unroll
    for (int i = 0; i < T::PI; ++i) v[i] = FP8 ? off : off ^ (uint32_t)(T::swizzle(T::RPI * i, is_v) * 16);
    dma16_stream<T::PI>(base, v, lds);
}
// The last step of a request: key L comes from new_row (null: from the row of zeros), keys past it from a row of zeros.
template <int D, bool FP8>
__device__ __forceinline__ void issue_last(const char *page_lo, const char *page_hi, const char *new_row, int first_key, int L,
                                           bool is_v, int lane, uint32_t lds_base)
{
    typedef Tile<D, FP8> T;
    asm volatile("" : "+v"(lane));                       // (per-lane values worked out here, not kept across the caller's loop)
    const char *zero = reinterpret_cast<const char *>(g_zero_row);
#pragma unroll
    for (int i = 0; i < T::NI; ++i) {
        const int r = T::RPI * i + lane / T::CH;             // this lane's row and 16-byte chunk
        const int chunk = (lane % T::CH) ^ T::swizzle(r, is_v);
        const int key = first_key + r;
        const char *src = (r < kPage ? page_lo : page_hi) + (r % kPage) * T::RB;
        if (key == L) src = new_row != nullptr ? new_row : zero;
        if (key > L) src = zero;
        dma16(src + chunk * 16, lds_base + i * 1024);
    }
}

typedef __attribute__((address_space(4))) const DecodeArgs const_decode_args;

// A stretch of steps of one request; wave-uniform.
struct Job {
    int b;                      // request
    int begin, end;             // steps [begin, end)
    int L;                      // cached tokens of the request
    __device__ __forceinline__ int steps() const { return (L + 32) >> 5; }    // over keys 0..L (key L is the new token)
};

// Bytes of the kernel's arguments in front of its structure.  What the first addresses are made of comes first and by itself: those
// words are in scalar registers when a wavefront starts, the structure is a memory read of 0.4 us away (one request of 1000
// tokens, 40 heads: 9.32 us before, 8.96 now).
constexpr int kDecodeLead = 56;
static_assert((kDecodeLead + offsetof(DecodeArgs, k_new)) % 64 == 0 && offsetof(DecodeArgs, pages_w) == offsetof(DecodeArgs, k_new) + 64, "a cache line");

// RANGES: `ranges` equal ranges of the batch's steps, a workgroup each per kv head; otherwise every (request, kv head) in
// `parts` equal parts, a workgroup each.  Grid: kv head fastest.
template <int D, bool FP8, int NW, bool RANGES>
__global__ __launch_bounds__(NW * 64, 2) void decode_attn_kernel(const int32_t *ctx_lens, const int32_t *bt, const uint16_t *pages, int max_blocks, int Hkv,
                                                                  uint32_t hkv_magic, int parts, const uint16_t *q, int B, DecodeArgs)
{
    typedef Tile<D, FP8> T;
    constexpr int KSTEPS = D / 16, DBLK = D / 32, NI = T::NI, NT = NW * 64, ROW = 2 * D;
    constexpr int DEPTH = FP8 ? 2 : 1;                     // steps a wavefront's tiles hold
    __shared__ __attribute__((aligned(1024))) char smem[NW * DEPTH * 2 * T::BYTES];
    __shared__ __attribute__((aligned(16))) float area[NW][kMergeCols][D];
    __shared__ float stat[NW][2][32];
    __shared__ int arrived;
    // (the structure lies behind the leading arguments)
    const const_decode_args *p = (const const_decode_args *)((__attribute__((address_space(4))) const char *)__builtin_amdgcn_kernarg_segment_ptr() + kDecodeLead);

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int half = lane >> 5, l32 = lane & 31;
    // a context length outside what the block table can describe is clamped: whatever the device
    // arrays hold, no address is formed from a block-table index out of range
    auto ctx_of = [&](int b) -> int { return min(max(((const const_i32 *)(uintptr_t)ctx_lens)[b], 0), max_blocks * kPage); };

    const int wg = magic_div(blockIdx.x, hkv_magic), kh = blockIdx.x - wg * Hkv;
    auto clear_next = [&]() {
        const int n = p->n_counters;
        for (int i = blockIdx.x * NT + tid; i < n; i += gridDim.x * NT) store_global(p->counters_next + i, 0);
    };
    // ---- the workgroup's first job; `left` steps of its range behind it
    Job job;
    int left = 0, div_q, div_r = 0, pos;
    if constexpr (!RANGES) {
        job.b = parts == 1 ? wg : wg / parts;
        pos = wg - job.b * parts;
        job.L = ctx_of(job.b);
        div_q = parts == 1 ? job.steps() : (job.steps() + parts - 1) / parts;
        job.begin = pos * div_q;
        job.end = min(job.steps(), job.begin + div_q);
        if (job.begin >= job.end) {                      // fewer steps than parts: nobody waits for this one
            clear_next();
            return;
        }
    } else {
        // lane l looks at requests l * R .. l * R + R - 1
        const int R = (B + 63) >> 6;
        const int32_t *ctx = ctx_lens;
        int mine = 0;
        for (int i = 0; i < R; ++i) {
            const int b = lane * R + i;
            if (b < B) mine += (min(max(ctx[b], 0), max_blocks * kPage) + 32) >> 5;
        }
        int incl = mine;
#pragma unroll
        for (int d = 1; d < 64; d <<= 1) {
            const int y = __shfl_up(incl, d, 64);
            if (lane >= d) incl += y;
        }
        const int total = __builtin_amdgcn_readlane(incl, 63);
        // equal ranges, but none shorter than min_steps
        const int ranges = min(p->ranges, (int)((uint32_t)(total + p->min_steps - 1) / (uint32_t)p->min_steps));
        if (wg >= ranges) {
            clear_next();
            return;
        }
        div_q = __builtin_amdgcn_readfirstlane((int)((uint32_t)total / (uint32_t)ranges));
        div_r = total - div_q * ranges;
        pos = wg * div_q + min(wg, div_r);
        left = div_q + (int)(wg < div_r);
        // the request of step `pos`: its lane, then inside the lane's block
        int base = incl - mine, found = -1, fl = 0, fbase = 0;
        if (pos >= base && pos < incl)
            for (int i = 0; i < R; ++i) {
                const int b = lane * R + i, L = min(max(ctx[min(b, B - 1)], 0), max_blocks * kPage);
                const int n = (L + 32) >> 5;
                if (found < 0 && pos < base + n) { found = b; fl = L; fbase = base; }
                base += n;
            }
        const int src = __builtin_ctzll(__builtin_amdgcn_ballot_w64(found >= 0) | (1ull << 63));
        job.b = __builtin_amdgcn_readlane(found, src);
        if (job.b < 0) return;                           // (ctx_lens written to while the launch runs: no address is formed from it)
        job.L = __builtin_amdgcn_readlane(fl, src);
        job.begin = pos - __builtin_amdgcn_readlane(fbase, src);
        job.end = min(job.steps(), job.begin + left);
        left -= job.end - job.begin;
    }
    // the job after `j`, with `rest` steps of the range behind j: rest goes down by the new job's steps
    auto next_job = [&](Job &j, int &rest) {
        ++j.b;
        j.L = ctx_of(min(j.b, B - 1));
        j.begin = 0;
        j.end = min(j.steps(), rest);
        rest -= j.end;
    };

    const uint32_t head_bytes = (uint32_t)kPage * T::RB, page_bytes = 2 * Hkv * head_bytes, v_delta = Hkv * head_bytes;
    const char *pool = reinterpret_cast<const char *>(pages) + (size_t)kh * head_bytes;
    char *my = smem + wave * (DEPTH * 2 * T::BYTES);
    const uint32_t my_lds = lds_address(my);
    const int r0 = lane / T::CH;
    const uint32_t k_off = r0 * T::RB + (((lane % T::CH) ^ T::swizzle(r0, false)) << 4);
    const uint32_t v_off = r0 * T::RB + (((lane % T::CH) ^ T::swizzle(r0, true)) << 4);

    // ---- the wavefront's cursor: the step whose loads are issued next (step fs of job fj, frest steps of the range behind
    // that job; fs < 0: there is none) and its pages (entries past the table's end belong to keys past L and are never
    // dereferenced)
    Job fj = job;
    int fs = job.begin + wave, frest = left, pg0 = 0, pg1 = 0;
    auto settle = [&]() {
        while (fs >= fj.end) {
            if (!RANGES || frest == 0) { fs = -1; return; }
            next_job(fj, frest);
            fs = wave;
        }
        const const_i32 *row = (const const_i32 *)(uintptr_t)(bt + (size_t)fj.b * max_blocks);
        pg0 = row[min(2 * fs, max_blocks - 1)];
        pg1 = row[min(2 * fs + 1, max_blocks - 1)];
    };
    auto issue = [&](bool is_v, uint32_t buf) {
        const char *base = pool + (is_v ? v_delta : 0);
        const char *lo = base + (size_t)pg0 * page_bytes, *hi = base + (size_t)pg1 * page_bytes;
        const uint32_t lds = my_lds + buf + (is_v ? T::BYTES : 0);
        if (fs + 1 < fj.steps()) {
            issue_page<D, FP8>(lo, is_v ? v_off : k_off, is_v, lds);
            issue_page<D, FP8>(hi, is_v ? v_off : k_off, is_v, lds + 16 * T::RB);
        } else {
            const char *row = nullptr;
            if constexpr (!FP8) row = reinterpret_cast<const char *>(is_v ? p->v_new : p->k_new) + ((size_t)fj.b * Hkv + kh) * ROW;
            issue_last<D, FP8>(lo, hi, row, fs * 32, fj.L, is_v, lane, lds);
        }
    };
    // Q fragments (B operand of S^T = K Q^T): column l32 is query head kh * g + l32, zero past g
    bf16x8 qf[KSTEPS];
    auto load_q = [&](int b) {
        int ln = lane;
        asm volatile("" : "+v"(ln));
        const int col = ln & 31, g = p->g;
        const global_u32x4 *qp = reinterpret_cast<const global_u32x4 *>((uintptr_t)(q + ((size_t)b * p->Hq + (size_t)kh * g + min(col, g - 1)) * D)) + (ln >> 5);
#pragma unroll
        for (int s = 0; s < KSTEPS; ++s) {
            u32x4 v = u32x4(qp[2 * s]);
            if (col >= g) v = u32x4{0u, 0u, 0u, 0u};
            qf[s] = __builtin_bit_cast(bf16x8, v);
        }
    };

    // ---- the first loads.  c*: the current step, n*: the one after it (FP8: in flight as well)
    settle();
    int cb = fj.b, cs = fs, cL = fj.L;
    [[maybe_unused]] int nb = 0, ns = -1, nL = 0;
    if (cs >= 0) {
        issue(false, 0);
        issue(true, 0);
        load_q(cb);
        fs += NW;
        settle();
        if constexpr (FP8) {
            nb = fj.b; ns = fs; nL = fj.L;
            if (ns >= 0) {
                issue(false, 2 * T::BYTES);
                issue(true, 2 * T::BYTES);
                fs += NW;
                settle();
            }
        }
    }

    // fragment addresses in the tiles: those of step s / block db are the first one's with a constant XOR-ed in.
    // 16-bit: accumulator element v is key 8 * (v / 4) + 4 * half + v % 4 of the step.  FP8: a V fragment holds 8 consecutive
    // keys, so K rows are read in the order that makes element v key 16 * (v / 8) + 8 * half + v % 8 (bits 2 and 3 of the
    // row index change places).
    uint32_t kbase0, vbase0;
    {
        const int blk = lane >> 4, i16 = lane & 15;
        if constexpr (FP8) {
            const int row = (l32 & 19) | (l32 & 4) << 1 | (l32 & 8) >> 1;
            kbase0 = row * T::RB + (T::swizzle(row, false) << 4) + 8 * half;
            const int rv = 8 * half + (i16 >> 1);
            vbase0 = T::BYTES + rv * T::RB + (((blk & 1) ^ T::swizzle(rv, true)) << 4) + 8 * (i16 & 1);
        } else {
            kbase0 = l32 * ROW + ((half ^ k_swizzle<D>(l32)) << 4);
            const int rr = 4 * half + (i16 >> 2), d0 = 16 * (blk & 1) + 4 * (i16 & 3);
            vbase0 = T::BYTES + rr * ROW + (((d0 >> 3) ^ v_swizzle<D>(rr)) << 4) + ((d0 & 7) << 1);
        }
    }
    auto key_of = [&](int v) -> int { return FP8 ? 16 * (v / 8) + 8 * half + v % 8 : 8 * (v / 4) + 4 * half + v % 4; };
    // FP8: the tiles hold code values; the K scale rides on the score factor (scales are positive: the sign of c is that of
    // the softmax scale)
    const float c_new = p->neg ? -p->c : p->c, c = FP8 ? c_new * p->k_scale : c_new;
    [[maybe_unused]] uint32_t buf = 0;                   // FP8: where the current step's tiles are

    for (;;) {                                           // the jobs of the range
    f32x16 o[DBLK];
    float m = -1e30f, lsum = 0.f;                        // m: a reference exponent, not the exact maximum
#pragma unroll
    for (int i = 0; i < DBLK; ++i)
#pragma unroll
        for (int v = 0; v < 16; ++v) o[i][v] = 0.f;
    bool first = true;                                   // the wavefront's first step of the job
    while (cs >= 0 && (!RANGES || cb == job.b)) {
        const bool far = fs >= 0, last = cs + 1 == (cL + 32) >> 5;      // loads to issue; the request's last step
        const int new_row = cL - cs * 32;                               // (the new token's place in the last step)
        // K has landed when only what was issued after it is outstanding
        if constexpr (FP8) {
            if (ns >= 0) wait_vm<3 * NI>();
            else wait_vm<NI>();
        } else {
            wait_vm<NI>();
        }
        asm volatile("" : "+v"(kbase0), "+v"(vbase0));
        const char *tiles = my + buf;
        bf16x8 kf[KSTEPS];
#pragma unroll
        for (int s = 0; s < KSTEPS; ++s) {
            if constexpr (FP8) {
                const uint2 x = *reinterpret_cast<const uint2 *>(tiles + (kbase0 ^ (s << 4)));
                kf[s] = codes_to_bf16(x.x, x.y);
            } else {
                kf[s] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const uint4 *>(tiles + (kbase0 ^ (s << 5))));
            }
        }
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");  // fragments are in registers: the tile may be overwritten
        if (far) issue(false, buf);
        f32x16 sc;
#pragma unroll
        for (int v = 0; v < 16; ++v) sc[v] = 0.f;
#pragma unroll
        for (int s = 0; s < KSTEPS; ++s) sc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[s], qf[s], sc, 0, 0, 0);
        if (last) {                                      // keys past the end do not exist (FP8: nor does key L, here)
            const float masked = p->neg ? INFINITY : -INFINITY;
#pragma unroll
            for (int v = 0; v < 16; ++v)
                if (key_of(v) > new_row - (FP8 ? 1 : 0)) sc[v] = masked;
        }
        bf16x8 pf[2];
        // (a lambda: as a function shared by the kernels it made the short kernel 4 % slower)
        auto weights = [&]() {                           // rounded to bf16 for the PV product
#pragma unroll
            for (int v = 0; v < 16; v += 2) {
                pf[v / 8][v % 8] = (__bf16)__builtin_amdgcn_exp2f(__builtin_fmaf(sc[v], c, -m));
                pf[v / 8][v % 8 + 1] = (__bf16)__builtin_amdgcn_exp2f(__builtin_fmaf(sc[v + 1], c, -m));
            }
        };
        if (first) {
            m = fmaxf(m, step_max(sc, c));                     // (a step without a key, FP8 only, leaves m and the weights 0)
            first = false;
            weights();
        } else {
            // m stays as it is unless a weight reaches 2
            weights();
            if (weights_reach_two(pf)) {
                const float m_new = fmaxf(m, step_max(sc, c));
                const float alpha = __builtin_amdgcn_exp2f(m - m_new);
                m = m_new;
                lsum *= alpha;
#pragma unroll
                for (int i = 0; i < DBLK; ++i)
#pragma unroll
                    for (int v = 0; v < 16; ++v) o[i][v] *= alpha;
                weights();
            }
        }
        add_weights(pf, lsum);
        // V has landed when only what was issued after it is outstanding
        if constexpr (FP8) {
            if (far) wait_vm<3 * NI>();
            else if (ns >= 0) wait_vm<2 * NI>();
            else wait_vm<0>();
        } else {
            if (far) wait_vm<NI>();
            else wait_vm<0>();
        }
        bf16x8 vf[2 * DBLK];
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int db = 0; db < DBLK; ++db) {
                if constexpr (FP8) {
                    const i32x2 x = __builtin_amdgcn_ds_read_tr8_b64_v2i32((lds_i32x2 *)(tiles + (vbase0 ^ (db << 5)) + j * (16 * T::RB)));
                    vf[j * DBLK + db] = codes_to_bf16((uint32_t)x[0], (uint32_t)x[1]);
                } else {
                    const char *a = tiles + (vbase0 ^ (db << 6)) + j * (16 * ROW);
                    const s16x4 va = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4 *)a);
                    const s16x4 vb = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4 *)(a + 8 * ROW));
                    vf[j * DBLK + db] = __builtin_bit_cast(bf16x8, __builtin_shufflevector(va, vb, 0, 1, 2, 3, 4, 5, 6, 7));
                }
            }
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        if (far) issue(true, buf);
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int db = 0; db < DBLK; ++db)
                o[db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vf[j * DBLK + db], pf[j], o[db], 0, 0, 0);
        if constexpr (FP8) {
            if (last) {
                // the new token: one key (row 0 of a product), not quantised
                const size_t at = ((size_t)cb * Hkv + kh) * D;
                const u32x4 none = {0u, 0u, 0u, 0u};
                const global_u32x4 *kp = reinterpret_cast<const global_u32x4 *>((uintptr_t)(p->k_new + at + 8 * half));
                u32x4 kn[KSTEPS];
                uint32_t vn[DBLK];
#pragma unroll
                for (int s = 0; s < KSTEPS; ++s) kn[s] = l32 == 0 ? u32x4(kp[2 * s]) : none;
#pragma unroll
                for (int db = 0; db < DBLK; ++db) vn[db] = half == 0 ? (uint32_t)p->v_new[at + 32 * db + l32] : 0u;
                f32x16 sn;
#pragma unroll
                for (int v = 0; v < 16; ++v) sn[v] = 0.f;
#pragma unroll
                for (int s = 0; s < KSTEPS; ++s) sn = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, kn[s]), qf[s], sn, 0, 0, 0);
                float score, unused;
                half_swap(sn[0] * c_new, score, unused);             // element 0 of the lower half-wave is key 0
                const float m_new = fmaxf(m, score);
                const float alpha = __builtin_amdgcn_exp2f(m - m_new);
                m = m_new;
                const __bf16 wgt = (__bf16)__builtin_amdgcn_exp2f(score - m);
                lsum = lsum * alpha + (half == 0 ? (float)wgt : 0.f);
                bf16x8 pn = __builtin_bit_cast(bf16x8, none);
                if (half == 0) pn[0] = (__bf16)((float)wgt * p->v_inv);
#pragma unroll
                for (int db = 0; db < DBLK; ++db) {
#pragma unroll
                    for (int v = 0; v < 16; ++v) o[db][v] *= alpha;
                    o[db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, u32x4{vn[db], 0u, 0u, 0u}), pn, o[db], 0, 0, 0);
                }
            }
        }
        // on to the next step (its Q rows, if it is another request's, are requested here)
        const int done_b = cb;
        if constexpr (FP8) {
            cb = nb; cs = ns; cL = nL;
            nb = fj.b; ns = fs; nL = fj.L;
            buf ^= 2 * T::BYTES;
        } else {
            cb = fj.b; cs = fs; cL = fj.L;
        }
        if (RANGES && cs >= 0 && cb != done_b) load_q(cb);
        if (far) {
            fs += NW;
            settle();
        }
    }

    // ---- the job is done: the wavefronts merge.  (The tiles may be receiving the next job's first steps: the merge has an
    // area of its own in LDS, for kMergeCols query heads at a time.)
    const const_decode_args *e = p;
    int te = tid;
    asm volatile("" : "+v"(te), "+s"(e));                // (values worked out and read here, not kept across the loop)
    const int half_e = (te >> 5) & 1, col_e = te & 31, g = e->g;
    const bool ends = job.end == job.steps(), whole = ends && job.begin == 0;
    const float ltot = half_swap_sum(lsum);
    if (half_e == 0) { stat[wave][0][col_e] = m; stat[wave][1][col_e] = ltot; }
    if (ends && e->pages_w != nullptr && job.L < max_blocks * kPage && wave == NW - 1 && (te & 63) < ROW / 8) {
        // fused append: the new token's K and V row of this kv head go to slot L % 16 of page block_table[b][L / 16], 16 bytes
        // per lane (nothing in this launch reads that slot: key L comes from k_new / v_new everywhere).  With an FP8
        // cache the row is quantised on the way: fl32(x * inv_scale) clamped to +-448, rounded to nearest even by
        // v_cvt_pk_fp8_f32, 8 codes per lane
        constexpr int LR = ROW / 16;                         // lanes of a row
        const int which = (te & 63) / LR, chunk = te % LR;
        const int page = ((const const_i32 *)(uintptr_t)(bt + (size_t)job.b * max_blocks))[job.L / kPage];
        const size_t at = (size_t)page * page_bytes + (which ? v_delta : 0) + (size_t)kh * head_bytes + (size_t)(job.L % kPage) * T::RB
                          + chunk * (T::RB / LR);
        const char *src = reinterpret_cast<const char *>(which ? e->v_new : e->k_new) + ((size_t)job.b * Hkv + kh) * ROW + chunk * 16;
        const u32x4 v = *reinterpret_cast<global_u32x4 *>((uintptr_t)src);
        char *dst = reinterpret_cast<char *>(e->pages_w) + at;
        if constexpr (FP8) {
            const uint2 x = bf16_to_codes(v, which ? e->v_inv : e->k_inv);
            *reinterpret_cast<global_u32x2_w *>((uintptr_t)dst) = u32x2{x.x, x.y};
        } else {
            *reinterpret_cast<global_u32x4_w *>((uintptr_t)dst) = v;
        }
    }
    // a request cut between workgroups: which part of how many this is, and where the parts are (a workgroup keeps the first
    // part of a request in its second place, any other part in its first one: it has at most one of each)
    int piece = 0, pieces = 1, w0 = 0, counter = 0;
    if (!whole) {
        if constexpr (!RANGES) {
            piece = pos;
            pieces = (job.steps() + div_q - 1) / div_q;
            w0 = wg - piece;
            counter = job.b;
        } else {
            auto owner = [&](int x) -> int {             // the range that has step x of the sequence
                const int cut = div_r * (div_q + 1);
                return __builtin_amdgcn_readfirstlane(x < cut ? (int)((uint32_t)x / (uint32_t)(div_q + 1)) : div_r + (int)((uint32_t)(x - cut) / (uint32_t)div_q));
            };
            w0 = owner(pos - job.begin);                 // pos: the sequence position of the job's first step
            pieces = owner(pos - job.begin + job.steps() - 1) - w0 + 1;
            piece = wg - w0;
            counter = w0;
        }
        counter = counter * Hkv + kh;
    }
    const int pfl = part_floats<D>(g);
    float *partial = e->partial;
    auto place = [&](int i) -> float * { return partial + ((size_t)(RANGES ? 2 * (w0 + i) + (int)(i == 0) : w0 + i) * Hkv + kh) * pfl; };
    const size_t head = (size_t)job.b * e->Hq + (size_t)kh * g;
    uint16_t *out = e->out;
    const float out_scale = e->out_scale;
    auto write_pair = [&](size_t at, float x, float y, float l) {
        const float inv = out_scale / l;
        bf16x2 r;
        r[0] = (__bf16)(x * inv);
        r[1] = (__bf16)(y * inv);
        *reinterpret_cast<__attribute__((address_space(1))) uint32_t *>((uintptr_t)(out + at)) = __builtin_bit_cast(uint32_t, r);
    };
    for (int c0 = 0; c0 < g; c0 += kMergeCols) {
        if (c0 != 0) lds_barrier();                      // everybody is done with the columns before
        if (col_e >= c0 && col_e < min(g, c0 + kMergeCols)) {
            float *mine = area[wave][col_e - c0];
#pragma unroll
            for (int db = 0; db < DBLK; ++db)
#pragma unroll
                for (int q4 = 0; q4 < 4; ++q4) {
                    f32x4 x;
#pragma unroll
                    for (int i = 0; i < 4; ++i) x[i] = o[db][q4 * 4 + i];
                    *reinterpret_cast<f32x4 *>(mine + 32 * db + 8 * q4 + 4 * half_e) = x;
                }
        }
        lds_barrier();
        // two neighbouring values of one head per thread
        for (int v = te; v < min(g - c0, kMergeCols) * (D / 2); v += NT) {
            const int cc = v / (D / 2), col = c0 + cc, d = 2 * (v - cc * (D / 2));
            float ms = stat[0][0][col];
#pragma unroll
            for (int i = 1; i < NW; ++i) ms = fmaxf(ms, stat[i][0][col]);
            float x = 0.f, y = 0.f, l = 0.f;
#pragma unroll
            for (int i = 0; i < NW; ++i) {
                const float wgt = __builtin_amdgcn_exp2f(stat[i][0][col] - ms);
                const float2 z = *reinterpret_cast<const float2 *>(&area[i][cc][d]);
                x = __builtin_fmaf(z.x, wgt, x);
                y = __builtin_fmaf(z.y, wgt, y);
                l = __builtin_fmaf(stat[i][1][col], wgt, l);
            }
            if (whole) {
                write_pair((head + col) * D + d, x, y, l);
            } else {
                float *mine = place(piece);
                store_coherent2(mine + col * D + d, x, y);
                if (d == 0) {
                    store_coherent(mine + g * D + col, ms);
                    store_coherent(mine + g * D + g + col, l);
                }
            }
        }
    }
    if (!whole) {
        coherent_stores_done();
        lds_barrier();
        if (te == 0) arrived = atomic_add_global(e->counters + counter, 1);
        lds_barrier();
        if (__builtin_amdgcn_readfirstlane(arrived) == pieces - 1) {
            // all the others have been here: the counter goes back to zero, the parts are merged in their order.  With few
            // columns the threads form groups that take every groups-th part, and the groups meet in LDS.
            if (te == 0) store_global(e->counters + counter, 0);
            const int pairs = g * (D / 2), groups = max(1, NT / pairs);
            for (int v0 = 0; v0 < pairs; v0 += NT) {
                const int grp = groups > 1 ? te / pairs : 0, v = groups > 1 ? te - grp * pairs : v0 + te;
                const bool on = grp < groups && v < pairs;
                const int col = v / (D / 2);
                float mm = -INFINITY, l = 0.f, x = 0.f, y = 0.f;
                if (on)
                    for (int i0 = grp; i0 < pieces; i0 += 8 * groups) {
                        float mi[8], li[8];
                        float2 xi[8];
#pragma unroll
                        for (int i = 0; i < 8; ++i) {
                            const float *src = place(min(i0 + i * groups, pieces - 1));
                            mi[i] = load_coherent(src + g * D + col);
                            li[i] = load_coherent(src + g * D + g + col);
                            xi[i] = load_coherent2(src + 2 * v);
                        }
#pragma unroll
                        for (int i = 0; i < 8; ++i)
                            if (i0 + i * groups < pieces) {
                                const float m_new = fmaxf(mm, mi[i]);
                                const float w_old = __builtin_amdgcn_exp2f(mm - m_new), w_new = __builtin_amdgcn_exp2f(mi[i] - m_new);
                                mm = m_new;
                                l = __builtin_fmaf(li[i], w_new, l * w_old);
                                x = __builtin_fmaf(xi[i].x, w_new, x * w_old);
                                y = __builtin_fmaf(xi[i].y, w_new, y * w_old);
                            }
                    }
                if (groups > 1) {
                    // (a group without a part has m = -inf and weighs nothing; group 0 always has one)
                    float *meet = &area[0][0][0];
                    static_assert(NW * kMergeCols * D >= 4 * NT, "four floats per thread");
                    if (on) *reinterpret_cast<f32x4 *>(meet + 4 * te) = f32x4{mm, l, x, y};
                    lds_barrier();
                    if (on && grp == 0)
                        for (int i = 1; i < groups; ++i) {
                            const f32x4 z = *reinterpret_cast<const f32x4 *>(meet + 4 * (i * pairs + v));
                            const float m_new = fmaxf(mm, z[0]);
                            const float w_old = __builtin_amdgcn_exp2f(mm - m_new), w_new = __builtin_amdgcn_exp2f(z[0] - m_new);
                            mm = m_new;
                            l = __builtin_fmaf(z[1], w_new, l * w_old);
                            x = __builtin_fmaf(z[2], w_new, x * w_old);
                            y = __builtin_fmaf(z[3], w_new, y * w_old);
                        }
                }
                if (on && grp == 0) write_pair(head * D + 2 * v, x, y, l);
            }
        }
    }
    if (!RANGES || left == 0) break;
    pos += job.end - job.begin;
    next_job(job, left);
    lds_barrier();                                       // everybody is done with stat, area and `arrived`
    }
    clear_next();
}

}  // namespace

// Scratch memory of tetri_decode_attn_static: the parts of split requests and their arrival counters, in arrays that
// are part of the loaded code object instead of an allocation (8 MiB on every device the library runs on,
// held until the process ends).  On the host an array's name is only a stand-in for the symbol: the
// device address is looked up once per device, with that device current, and only that address
// is ever handed to a kernel.
static __device__ __align__(256) unsigned char scratch[kDecodeStaticScratchBytes];
static __device__ __align__(256) int32_t scratch_counters[kCounterSets * kDecodeStaticCounters];

hipError_t tetri_decode_static_memory(DecodeStatic *out)
{
    constexpr int kMaxDevices = 64;
    static std::mutex lock;
    static DecodeStatic per_device[kMaxDevices];        // null until the device's addresses are known
    static std::atomic<uint32_t> turns[kMaxDevices];
    int dev = -1;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> guard(lock);
    if (!per_device[dev].scratch) {
        void *p = nullptr, *c = nullptr;
        e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e == hipSuccess) e = hipGetSymbolAddress(&c, HIP_SYMBOL(scratch_counters));
        if (e != hipSuccess) return e;
        if (!p || !c) return hipErrorInvalidSymbol;
        per_device[dev] = {static_cast<float *>(p), static_cast<int32_t *>(c), &turns[dev]};
    }
    *out = per_device[dev];
    return hipSuccess;
}

template <int D, bool FP8>
static hipError_t launch_decode(const DecodeParams &p, hipStream_t stream)
{
    const dim3 grid((p.parts > 0 ? p.B * p.parts : p.ranges) * p.Hkv);
    auto kernel = p.parts > 0 ? decode_attn_kernel<D, FP8, 4, false> : decode_attn_kernel<D, FP8, 4, true>;
    static_assert(KernelArgs<decltype(kernel)>::last_offset() == kDecodeLead, "where the kernel reads its structure");
    hipLaunchKernelGGL(kernel, grid, dim3(256), 0, stream, p.ctx, p.bt, p.pages, p.max_blocks, p.Hkv, p.hkv_magic, p.parts, p.q, p.B, static_cast<const DecodeArgs &>(p));
    return hipGetLastError();
}

hipError_t tetri_launch_decode(const tetri_ctx *h, const DecodeParams &p, hipStream_t stream)
{
    const int d = h->cfg.head_dim;
    if (d == 128) return p.fp8 ? launch_decode<128, true>(p, stream) : launch_decode<128, false>(p, stream);
    if (d == 64) return p.fp8 ? launch_decode<64, true>(p, stream) : launch_decode<64, false>(p, stream);
    return hipErrorInvalidValue;
}
