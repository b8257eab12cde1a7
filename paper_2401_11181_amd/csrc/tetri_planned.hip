// Chunked-prefill causal attention over a paged KV cache for gfx950: the shared-tile kernel (attn_tile.h, tetri_attn.hip) on a
// division of the work that the host has made, for chunks whose segments it knows.
//
// The launch that divides itself (tetri_attn.hip) looks its segments up on the device (2.2 us to a workgroup's first address) and
// gives every row tile a workgroup, or the tiles of a head equal stretches of keys.  Long launches then end with compute units
// idle (2048 rows of 32/8 heads at 12000 cached tokens: 12 to 21 % of the time, more where segments of different contexts meet).
// Here the jobs are laid out on the host (plan_tiles): one workgroup per compute unit, all with about the same number of stages,
// the pieces of a tile next to each other in time so that they share K and V through L2; a workgroup's first address is two reads
// of the kernel arguments away (1.0 us), and its new K and V rows go to their pages out of the stage buffers instead of through
// further workgroups.  With 8 slots a staged key serves 256 rows: half the bytes into LDS and half the barriers per product.
// What bounds it: the loop (attn_tile.h), 3.5 us for 8 blocks of 32 x 32 on each SIMD with the chip's clock at 1.8 to 2.05 GHz under
// that load; where tiles are shared, 6.6 us from the end of the last loop to the last row written.
// 2048 rows of 32/8 heads at 20000 cached tokens 688 -> 618 us, 300 rows at 20000 and 1700 at 0 371 -> 153, 512 rows of 40 heads at
// 8000 111 -> 103, 512 rows of 32/8 heads over FP8 codes at 3000 59.6 -> 49.6.
#include <hip/hip_ext.h>

#include "attn_tile.h"

namespace {

using namespace tetri_dev;

typedef __attribute__((address_space(4))) const TilePlan const_plan;
typedef __attribute__((address_space(4))) const u32x4 const_u32x4;

template <int D, int KS, bool F8>
__global__ __launch_bounds__(Shape<KS>::WAVES * 64, 2) void attn_planned_kernel(AttnParams p, TilePlan)
{
    constexpr int STAGE = Shape<KS>::STAGE, STAGE_U4 = STAGE * (D / 8), SLOTS = Shape<KS>::SLOTS, NT = Shape<KS>::WAVES * 64;
    __shared__ uint4 smem[4 * STAGE_U4];             // K and V of two stage buffers: K0 | K1 | V0 | V1
    __shared__ float Mstat[SLOTS][2][32];
    __shared__ uint32_t peek[SLOTS][64];             // where a look at a tile's arrival counter lands
    __shared__ int old_stash[SLOTS];                 // what a wavefront's announcement of an earlier job's piece found
    __shared__ AttnParams params;
    const const_plan *plan = (const const_plan *)((__attribute__((address_space(4))) const char *)__builtin_amdgcn_kernarg_segment_ptr()
                                                  + (sizeof(AttnParams) + alignof(TilePlan) - 1) / alignof(TilePlan) * alignof(TilePlan));
    TETRI_MARK(0);
    int tid = threadIdx.x;
    asm volatile("" : "+v"(tid));
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int slot = wave % SLOTS;
    // ---- workgroup id -> (pool, index in it): the workgroups of a head group run on the pool's XCDs and share their L2
    const int xcd = blockIdx.x % kXcd, pool = xcd >> p.span_shift;
    const int widx = ((blockIdx.x / kXcd) << p.span_shift) + (xcd & ((1 << p.span_shift) - 1));
    if (threadIdx.x == 0) params = p;                // from scalar registers: no memory read to wait for
    // the arrival counters of a later launch: all zero when this launch ends
    if (plan->places != 0)
        for (int i = blockIdx.x * NT + threadIdx.x; i < p.n_counters; i += p.attn_grid * NT) p.counters_next[i] = 0;
    if (plan->rows < p.C) {                          // the padding rows, written as +0 by all workgroups
        const size_t first = (size_t)plan->rows * p.Hq * (D / 8), n = (size_t)p.C * p.Hq * (D / 8);
        for (size_t i = first + (size_t)blockIdx.x * NT + threadIdx.x; i < n; i += (size_t)p.attn_grid * NT)
            reinterpret_cast<global_u32x4_w *>((uintptr_t)p.out)[i] = u32x4{0u, 0u, 0u, 0u};
    }
    if (widx >= plan->wgs) return;
    // job `index` of the plan; returns the workgroup's next one
    auto make_job = [&](const AttnParams &pp, int index, Job &X) __attribute__((always_inline)) -> int {
        const u32x4 w = *(const const_u32x4 *)&plan->job[index];
        const const_i32 *g = (const const_i32 *)plan->seg[w[0] & 63];
        const int seg_cu = g[0], n_s = g[1], L = g[2];
        X.grp = pool * pp.gpx + (int)((w[0] >> 6) & 1023);
        X.kh = magic_div(X.grp, pp.kv_magic);
        X.t0 = w[0] >> 16;
        X.seg_cu = seg_cu; X.n_s = n_s;
        X.it_begin = w[1] & 0xffff; X.it_end = w[1] >> 16;
        X.wf = pool * plan->places + (int)(w[2] & 0xffff);
        X.piece = (w[2] >> 16) & 255; X.npieces = w[2] >> 24;
        X.tile_index = 0;
        X.appends = (int)(X.grp * pp.hpw == X.kh * pp.g);   // (the first head group of its kv head)
        X.src.bt_off = (int)(w[0] & 63) * pp.max_blocks;
        X.src.new_off = (uint32_t)((seg_cu * pp.Hkv + X.kh) * (D * 2));
        X.src.L = L;
        X.src.n_new = min(n_s, X.t0 + (32 << pp.rb_shift));
        X.src.n_ctx_tiles = (L + STAGE - 1) / STAGE;
        return (int)(w[3] & 0xffff);
    };
    // (a pool with fewer head groups than the others skips the jobs of those it does not have)
    auto find_job = [&](const AttnParams &pp, int index, Job &X, int &after) __attribute__((always_inline)) -> bool {
        for (;;) {
            after = make_job(pp, index, X);
            if (X.grp < pp.groups && X.it_begin < X.it_end) return true;
            if (after <= index) return false;
            index = after;
        }
    };
    Job J;
    int after;
    if (!find_job(p, widx, J, after)) return;
    TETRI_MARK(9);

    // ---- the first job's Q rows, by way of the second stage buffer (8 KB a wavefront; its first loads go out behind the job's
    // first barrier), and its first stage
    Carry<D> cy;
    cy.par = J.it_begin & 1;                         // the first stage goes to buffer 0
    {
        char *q_tile = reinterpret_cast<char *>(smem + (wave < 4 ? 1 : 3) * STAGE_U4) + (wave & 3) * (32 * D * 2);
        request_q_rows<D>(p, J, J.grp * p.hpw + (slot & (p.hpw - 1)), slot >> p.hpw_shift, lane, lds_address(q_tile));
        const WaveSrc ws = make_wave_src<D, KS, F8>(p, J.kh);
        LaneOffsets<D> lo;
        init_lane_offsets<D>(lo, lane);
        const int page = load_stage_page<KS>(p.bt + J.src.bt_off, p.max_blocks, J.it_begin, wave);
        StageLoads sl;
        const bool full = describe_stage_loads<D, KS, F8>(J.src, ws, lo, page, J.it_begin, wave, p.Hkv * D * 2, lds_address(smem), sl);
        cy.have_codes = F8 && sl.codes;
        if (F8 && sl.codes) {
            fetch_stage_codes<D>(sl, full, cy.codes);
            wait_vm<0>();
        } else {
            issue_stage_loads<D, KS>(sl, full);
            wait_vm<2 * (D / 32)>();                 // (all but the stage's)
        }
        cy.page = load_stage_page<KS>(p.bt + J.src.bt_off, p.max_blocks, J.it_begin + 1, wave);
        read_q_rows<D>(q_tile, lane, cy.qf);
    }
    TETRI_MARK(1);

    Handover ho;
    for (bool first = true;; first = false) {
        bool more = false;
        Job N = J;
        if (after > 0) {
            AttnParams pj = p;                       // before the first job's first barrier the copy in LDS may be incomplete
            if (!first) {
                asm volatile("" ::: "memory");
                pj = read_params(&params);
            }
            more = find_job(pj, after, N, after);
        }
        tile_job<D, KS, F8, true>(p, first, &params, smem, Mstat, peek, old_stash, J, more, N, cy, ho);
        if (!more) break;
        J = N;
    }
    // ---- a piece whose hand-over was left open: if it was the last of its tile to arrive, this wavefront finishes the tile
    if (ho.unit >= 0) {
        asm volatile("" ::: "memory");
        const AttnParams pd = read_params(&params);
        int tid_end = threadIdx.x;
        asm volatile("" : "+v"(tid_end));
        const int ln = tid_end & 63, sl = __builtin_amdgcn_readfirstlane(tid_end >> 6) % SLOTS;
        if (__builtin_amdgcn_readfirstlane(old_stash[sl]) == ho.npieces - 1) {
            const int head = ho.grp * pd.hpw + (sl & (pd.hpw - 1));
            const int t = ho.t0 + 32 * (sl >> pd.hpw_shift) + (ln & 31);
            if (ln == 0) store_global(pd.counters + ho.unit, 0);        // (the last to arrive: see tile_job)
            finish_tile<D, SLOTS, true>(pd, ho.grp, ho.wf, ho.tile_index, ho.npieces, -1, sl, nullptr, 0.f, 0.f, ln, t < ho.n_s, ho.seg_cu + t, head);
        }
    }
    TETRI_MARK(7);
}

}  // namespace

hipError_t tetri_launch_planned(const AttnParams &p, bool fp8_pool, hipStream_t stream)
{
    static_assert(sizeof(AttnParams) + sizeof(TilePlan) + 16 <= 4096, "kernel arguments");
    auto kernel = p.hpw * p.rb == 4 ? (fp8_pool ? attn_planned_kernel<128, 2, true> : attn_planned_kernel<128, 2, false>)
                                    : (fp8_pool ? attn_planned_kernel<128, 3, true> : attn_planned_kernel<128, 3, false>);
    // (the event rides on the kernel's own completion signal)
    if (p.plan->done) hipExtLaunchKernelGGL(kernel, dim3(p.attn_grid), dim3(512), 0, stream, nullptr, p.plan->done, 0, p, *p.plan);
    else hipLaunchKernelGGL(kernel, dim3(p.attn_grid), dim3(512), 0, stream, p, *p.plan);
    return hipGetLastError();
}
