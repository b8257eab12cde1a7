// Chunked-prefill causal attention over a paged KV cache for gfx950 (CDNA4): shared-tile kernel.
// TetriInfer Sec. 3.3.3 (prefill one fixed-size chunk at a time; several requests may be merged
// into a chunk), Sec. 2.1 (causal prefill), Sec. 3.4 (paged KV).  The kernel is a flash-style
// single pass with online softmax; that structure is prior art (the paper names FlashAttention
// as orthogonal work), the paper itself gives no kernel.
//
// Mapping to the hardware
//   * A workgroup is 4*KS wavefronts.  A wavefront owns 32 query rows of one query head and one
//     of KS parts of every key stage; the 4 row/head slots are (heads sharing one kv head) x
//     (32-row blocks).  With KS = 2 a CU holds 8 wavefronts, two per SIMD, so one wavefront's
//     softmax (VALU) overlaps the other's MFMA, while every K/V byte brought into LDS still
//     serves 128 query rows.  The KS partial results are merged once through LDS at the end.
//     With KS = 1 a workgroup has 4 wavefronts and half the LDS, two workgroups share a CU and the
//     two wavefronts of a SIMD belong to different workgroups (no common barrier); the library
//     uses it for launches with at least two workgroups per CU (see softmax_pv for its schedule).
//   * A stage is 64*KS keys of K and V.  Stages go from HBM/L2 straight into LDS with
//     global_load_lds_dwordx4 (no register staging), double buffered: the loads of stage i+1 are
//     in flight while stage i is consumed; one workgroup barrier per stage.  The 16 key rows a
//     wavefront loads per stage are exactly one (page, kv head) block of the pool, 4 KB
//     contiguous: one scalar base address per block, per-lane offsets fixed for the whole kernel.
//   * Scores are computed transposed, S^T = K Q^T, with v_mfma_f32_32x32x16_bf16: K fragments
//     come from LDS (A operand), Q fragments stay in registers (B operand).  In the accumulator
//     layout every lane then holds 16 keys of ONE query, so row max / row sum are in-lane
//     reductions plus one exchange between the two half-waves, and the bf16-rounded weights are
//     already laid out as the B operand of the second product O^T += V^T P^T.
//   * V is staged row-major ([key][d]) and read with ds_read_b64_tr_b16, which hands each lane
//     four consecutive keys of one d: the A operand of the second product without a transpose
//     pass.
//   * LDS rows are XOR-swizzled in 16-byte units (the permutation is applied to the per-lane
//     global address of the direct load) so that the 128-bit K reads and the transposing V reads
//     are bank-conflict free.
//   * Workgroup ids are remapped so that all workgroups of a kv head run on one XCD (one L2).
//   * Two ways of handing out the work of a head group (all row tiles of the heads of one
//     workgroup column):
//       - tile mode: one workgroup per row tile, long (late) tiles first; for launches with at
//         least two workgroups per compute unit;
//       - stream mode: the stages of all tiles of the head group, laid end to end in tile order,
//         are cut into G equal ranges, one per workgroup (G = compute units / head groups), so
//         every compute unit gets the same number of stages however the causal triangle and the
//         segment lengths fall.  A range may start and end inside a tile: the pieces of such a
//         tile meet in scratch memory of the library's handle, without anybody waiting: every
//         piece but the last to arrive leaves its unnormalised (O, m, row sum) there, the last
//         one merges all of them in piece order (see finish_tile).  A workgroup whose range
//         spans several tiles runs them as consecutive jobs; the first K/V stage and the Q rows of
//         the next job are requested before the current job's epilogue.
//   * The fused form of the launch has further workgroups that copy the chunk's new K/V rows
//     into the page pool (append_rows).
#include "attn_tile.h"

namespace {

using namespace tetri_dev;

// Fused KV append: workgroup `blk` of `nblk` copies chunk rows blk, blk + nblk, ... (K and V of
// every kv head, 16 bytes per thread and pass) into slot (ctx + t) % 16 of page
// block_table[s][(ctx + t) / 16].  Same result as the stand-alone append kernel, bit for bit.
// First every thread looks up where one of the workgroup's rows goes (table in LDS); then rows
// are copied 8 at a time with all their loads issued before the first store, so that a
// workgroup has tens of KB in flight.
// F8: the pool holds FP8 codes; a row's 16-byte vectors (8 values) are quantised on the way (8 codes, 8 bytes) under
// the tensor's scale; the pool's layout is the same with half the element size.
template <int D, bool F8>
__device__ __forceinline__ void append_rows(const AttnParams &p, unsigned long long *row_dst, int blk, int nblk, int tid, int nthreads)
{
    constexpr int CH = D / 8, R = 8;
    const int n_real = p.cu[p.S];
    const int per_row = p.Hkv * CH;                    // 16-byte vectors per row and matrix
    for (int base = blk; base < n_real; base += nblk * nthreads) {     // one pass unless the chunk has more than nblk * nthreads rows
        const int mine = base + tid * nblk;
        if (mine < n_real) {
            int lo = 0, hi = p.S - 1;                  // largest s with cu[s] <= row
            while (lo < hi) {
                const int mid = (lo + hi + 1) >> 1;
                if (p.cu[mid] <= mine) lo = mid; else hi = mid - 1;
            }
            const int pos = p.ctx[lo] + (mine - p.cu[lo]);
            const int page = p.bt[(size_t)lo * p.max_blocks + pos / kPage];
            // of the row's K vector 0 of head 0, in units of a vector (16 bytes; 8 bytes of codes)
            row_dst[tid] = (unsigned long long)page * 2 * p.Hkv * (kPage * CH) + (unsigned long long)(pos % kPage) * CH;
        }
        __syncthreads();
        const int rows_here = min(nthreads, (n_real - base + nblk - 1) / nblk);
        for (int r0 = 0; r0 < rows_here; r0 += R) {
            for (int x = tid; x < 2 * per_row; x += nthreads) {
                const int which = x >= per_row, y = x - which * per_row;
                const int head = y / CH, c = y - head * CH;
                const size_t in_page = ((size_t)which * p.Hkv + head) * (kPage * CH) + c;
                const u32x4 *src = reinterpret_cast<const u32x4 *>(which ? p.v_new : p.k_new) + y;
                u32x4 v[R];                            // past the last row: that row once more
#pragma unroll
                for (int r = 0; r < R; ++r) v[r] = src[(size_t)(base + min(r0 + r, rows_here - 1) * nblk) * per_row];
#pragma unroll
                for (int r = 0; r < R; ++r) {
                    const size_t at = row_dst[min(r0 + r, rows_here - 1)] + in_page;
                    if constexpr (F8) reinterpret_cast<uint2 *>(p.pages_w)[at] = bf16_to_codes(v[r], which ? p.v_inv : p.k_inv);
                    else reinterpret_cast<u32x4 *>(p.pages_w)[at] = v[r];
                }
            }
        }
        __syncthreads();
    }
}

// Padding rows [cu[S], C) of this head group's heads, written as +0: row first, first + stride, ...
template <int D>
__device__ __forceinline__ void zero_padding_rows(const AttnParams &p, int grp, int first, int stride, int tid, int nthreads)
{
    constexpr int CH = D / 8;
    const int per_row = p.hpw * CH;                    // 16-byte vectors per row of this head group: a power of two <= 64
    const int rows_per_pass = nthreads / per_row;
    const int x = tid % per_row, rr = tid / per_row;
    for (int r = p.cu[p.S] + first + rr * stride; r < p.C; r += rows_per_pass * stride) {
        uint4 *o = reinterpret_cast<uint4 *>(p.out + ((size_t)r * p.Hq + (size_t)grp * p.hpw) * D);
        o[x] = make_uint4(0, 0, 0, 0);
    }
}

template <int D, int KS, bool F8>
__global__ __launch_bounds__(Shape<KS>::WAVES * 64, 2) void attn_tile_kernel(AttnParams p)
{
    constexpr int STAGE = Shape<KS>::STAGE;
    constexpr int STAGE_U4 = STAGE * (D / 8);
    constexpr int NT = Shape<KS>::WAVES * 64;
    __shared__ uint4 smem[4 * STAGE_U4];             // K and V of two stage buffers: K0 | K1 | V0 | V1
    __shared__ float Mstat[Shape<KS>::SLOTS][2][32];
    __shared__ uint32_t peek[Shape<KS>::SLOTS][64];            // where a look at a tile's arrival counter lands
    __shared__ int old_stash[Shape<KS>::SLOTS];                // what a wavefront's announcement of an earlier job's piece found
    __shared__ int4 seg_tab[64];                     // stream mode: (first row, rows, cached tokens) of every segment
    __shared__ AttnParams params;
    TETRI_MARK(0);

    // ---- fused KV append: append_blocks workgroups copy the chunk's new K/V rows into their page
    // slots.  They come after the attention workgroups, on the compute units those leave idle.
    int abid = blockIdx.x;                           // index in the attention grid
    if (abid >= p.attn_first) {
        if (abid < p.attn_first + p.append_blocks) {
            append_rows<D, F8>(p, reinterpret_cast<unsigned long long *>(smem), abid - p.attn_first, p.append_blocks, threadIdx.x, NT);
            return;
        }
        abid -= p.append_blocks;
    }
    // ---- workgroup id -> (head group, index inside the group).  The workgroups of a head group run
    // on one XCD (they read the same K and V through its L2); an XCD has gpx groups and starts their
    // workgroups index by index.  With four or fewer groups each runs on 1 << span_shift = 2, 4 or 8 XCDs: the
    // others would have nothing to do (8 heads sharing 2 kv heads, 2048 rows: 80 us on two XCDs, 35 on all).
    const int xcd = abid % kXcd, local = abid / kXcd;
    const int lidx = magic_div(local, p.gpx_magic);
    const int grp = (xcd >> p.span_shift) * p.gpx + (local - lidx * p.gpx);
    const int widx = (lidx << p.span_shift) + (xcd & ((1 << p.span_shift) - 1));
    const int G = p.stream_wgs;
    // the arrival counters of a later launch: all zero when this launch ends
    if (G != 0 || p.helpers != 0)
        for (int i = abid * NT + threadIdx.x; i < p.n_counters; i += p.attn_grid * NT) p.counters_next[i] = 0;
    if (grp >= p.groups || widx >= (G != 0 ? G : (p.helpers != 0 ? p.tiles + p.helpers - 2 : p.tiles))) return;
    if (threadIdx.x == 0) params = p;                // from scalar registers: no memory read to wait for

    int tid = threadIdx.x;
    asm volatile("" : "+v"(tid));
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int slot = wave % Shape<KS>::SLOTS, kq = wave / Shape<KS>::SLOTS;
    const int bm_shift = 5 + p.rb_shift, BM = 1 << bm_shift;
    const int S = p.S;
    const int kh = magic_div(grp, p.kv_magic);
    const int first_page = min(wave, p.max_blocks - 1), first_page_hi = min(wave + Shape<KS>::SLOTS, p.max_blocks - 1);

    const WaveSrc ws = make_wave_src<D, KS, F8>(p, kh);    // for the first job's first loads; every job derives its own

    // ---- the workgroup's first job.  Lane l looks at segment s0 + l (64 at a time); it also fetches
    // what the owner of the job will need next (context length, the pages of the segment's first
    // stage), so that the kernel's first loads of K and V are one memory round trip away from its
    // start wherever possible.
    Job J;
    SegInfo seg = {-1, 0, 0, 0};
    int page = 0, page_hi = 0;
    // stream mode: the range of stages of this workgroup, [pos, b1) in the group's tile order, of W
    // stages shared by Gp workgroups; the tile the next job is in: tile j of nt in its segment,
    // starting at position tile_lin
    int pos = 0, b1 = 0, W = 1, Gp = 1, j = 0, nt = 1, tile_lin = 0, tile_index = 0;
    // stream mode, one segment whose block-table row fits two registers per lane: the whole row is fetched together
    // with the segment lengths, so that the pages of the workgroup's first stage, wherever its range starts, do not
    // cost a second round trip to memory
    const bool row_in_lanes = G != 0 && S == 1 && p.max_blocks <= 128;
    int bt_lo = 0, bt_hi = 0;
    // tile and tail modes: the workgroup's second tile (a helper's, or the bound's last tile), as found by the lookup;
    // its job is made when its turn comes
    SegInfo lg0 = {-1, 0, 0, 0};
    int lw0 = -1, lt0 = -1, n_later = 0, tail_piece = 0;
    bool later_whole = false;                        // the second tile is done whole, whatever its length
    int first_want = -1, first_t0 = -1;              // the first one (its segment is in `seg`)
    bool pages_fetched = true;                       // page / page_hi are those of the first job's stage 0
    if (G == 0) {
        // Tile mode: row tile T - 1 - widx, late (long) tiles first.  Tail mode (helpers != 0): first the owners
        // of the tiles but the last one of the host's bound (which is real only in chunks with ragged segments),
        // each doing its tile's key range but for the tail, then the helpers, each doing the tails of two of
        // those tiles.  The bound's last tile gets no workgroup of its own (it would start when the first compute
        // unit becomes free and, though empty, end after everybody else): it is one more job, done whole, of
        // the owner of tile 0, whose key range is the shortest.  Tiles never span two segments.
        const int T = p.tiles, H = p.helpers;
        int want0, want1 = -1;
        int &piece = tail_piece;
        if (H == 0) {
            want0 = T - 1 - widx;
        } else if (widx < T - 1) {
            want0 = T - 2 - widx;
            if (want0 == 0) { want1 = T - 1; later_whole = true; }
        } else {
            piece = 1;
            want0 = T - 2 - 2 * (widx - (T - 1));
            if (want0 >= 1) want1 = want0 - 1;
        }
        // one pass over the segments finds both
        SegInfo g0 = {-1, 0, 0, 0}, g1 = g0;
        int t00 = -1, t01 = -1, base = 0;
        for (int s0 = 0; s0 < S; s0 += 64) {
            const int idx = s0 + lane;
            const int a = idx < S ? p.cu[idx] : 0, b = idx < S ? p.cu[idx + 1] : 0;
            const int ctx_len = idx < S ? p.ctx[idx] : 0;
            const int pg = idx < S ? p.bt[(size_t)idx * p.max_blocks + first_page] : 0;
            const int pg_hi = idx < S ? p.bt[(size_t)idx * p.max_blocks + first_page_hi] : 0;
            const int ntl = (b - a + BM - 1) >> bm_shift;          // 0 for lanes past the last segment
            int incl = ntl;
#pragma unroll
            for (int d = 1; d < 64; d <<= 1) {
                const int y = __shfl_up(incl, d, 64);
                if (lane >= d) incl += y;
            }
            auto find = [&](int want, SegInfo &g, int &t0, bool pages) __attribute__((always_inline)) {
                const int rel = want - base;
                const unsigned long long owner = __builtin_amdgcn_ballot_w64(t0 < 0 && want >= 0 && rel >= incl - ntl && rel < incl);
                if (owner != 0) {
                    const int o = __builtin_ctzll(owner);
                    g.s = s0 + o;
                    t0 = (rel - __builtin_amdgcn_readlane(incl - ntl, o)) * BM;
                    g.seg_cu = __builtin_amdgcn_readlane(a, o);
                    g.n_s = __builtin_amdgcn_readlane(b - a, o);
                    g.L = __builtin_amdgcn_readlane(ctx_len, o);
                    if (pages) {
                        page = __builtin_amdgcn_readlane(pg, o);
                        page_hi = __builtin_amdgcn_readlane(pg_hi, o);
                    }
                }
            };
            find(want0, g0, t00, true);
            if (want1 >= 0) find(want1, g1, t01, false);
            base += __builtin_amdgcn_readlane(incl, 63);
        }
        TETRI_MARK(8);
        // a wanted tile past the last segment's tiles: the padding rows [cu[S], C), one 32-row block per wavefront slot
        auto pad_tile = [&](int want, int t0) __attribute__((always_inline)) {
            if (want >= 0 && t0 < 0 && piece == 0 && kq == 0) {
                const int hh = slot & (p.hpw - 1), rbk = slot >> p.hpw_shift;
                const int r = p.cu[S] + (want - base) * BM + 32 * rbk + (lane & 31);
                if (r < p.C) {
                    uint4 *o = reinterpret_cast<uint4 *>(p.out + ((size_t)r * p.Hq + grp * p.hpw + hh) * D);
                    for (int c = lane >> 5; c < D / 8; c += 2) o[c] = make_uint4(0, 0, 0, 0);
                }
            }
        };
        pad_tile(want0, t00);
        if (want1 >= 0) pad_tile(want1, t01);
        auto tail_ok = [&](int want, const SegInfo &g, int t0) __attribute__((always_inline)) -> bool {
            // whether this workgroup has a job on that tile: it exists, and a helper's tile hands a tail over
            if (want < 0 || t0 < 0) return false;
            if (piece == 0) return true;
            const int n_new = min(g.n_s, t0 + BM);
            const int n_all = (g.L + STAGE - 1) / STAGE + (n_new + STAGE - 1) / STAGE;
            return n_all >= p.split_min && ((max(n_all - p.split_bias, 0) * p.tail_q8 + 128) >> 8) != 0;
        };
        const bool v0 = tail_ok(want0, g0, t00), v1 = want1 >= 0 && tail_ok(want1, g1, t01);
        if (!v0 && !v1) return;
        // the first valid one becomes J, a second one waits as (tile, segment, first row)
        pages_fetched = v0;
        seg.s = v0 ? g0.s : g1.s;
        seg.seg_cu = v0 ? g0.seg_cu : g1.seg_cu;
        seg.n_s = v0 ? g0.n_s : g1.n_s;
        seg.L = v0 ? g0.L : g1.L;
        first_want = v0 ? want0 : want1;
        first_t0 = v0 ? t00 : t01;
        n_later = (int)(v0 && v1);
        lg0 = g1; lw0 = want1; lt0 = t01;
    }
    // The piece of a tile this workgroup does in tile and tail mode: all of it, or with a tail handed over (key ranges
    // of at least split_min stages) everything but the tail / the tail.  A helper has about split_bias stages' worth of
    // extra work (a second tile's prologue, handing its first result over): owners and helpers finish together when
    // each tile hands over the share tail_q8 / 256 of what exceeds that.
    // (pp: the launch parameters, from the kernel arguments for a workgroup's first jobs, from their copy in LDS later:
    // kept in scalar registers across the jobs they would push other values out to memory)
    auto make_piece = [&](const AttnParams &pp, int want, const SegInfo &g, int t0, bool whole, Job &X) __attribute__((always_inline)) {
        const int H = whole ? 0 : pp.helpers, piece = tail_piece;
        {
            X.grp = grp; X.kh = kh; X.seg_cu = g.seg_cu; X.n_s = g.n_s; X.t0 = t0; X.tile_index = want;
            X.src = make_src<D, KS>(pp, kh, g, t0);
            const int n_all = X.src.n_ctx_tiles + (X.src.n_new + STAGE - 1) / STAGE;
            const int n_tail = (H != 0 && n_all >= pp.split_min) ? (max(n_all - pp.split_bias, 0) * pp.tail_q8 + 128) >> 8 : 0;
            X.it_begin = piece == 0 ? 0 : n_all - n_tail;
            X.it_end = piece == 0 ? n_all - n_tail : n_all;
            X.piece = piece; X.npieces = n_tail != 0 ? 2 : 1; X.wf = 0;
        }
    };
    if (G == 0) {
        make_piece(p, first_want, seg, first_t0, false, J);
    } else {
        // stream mode (S <= 64): every workgroup of the group works out the same division
        const int a = lane < S ? p.cu[lane] : 0, b = lane < S ? p.cu[lane + 1] : 0;
        const int ctx_len = lane < S ? p.ctx[lane] : 0;
        const int pg = lane < S ? p.bt[(size_t)lane * p.max_blocks + first_page] : 0;
        const int pg_hi = lane < S ? p.bt[(size_t)lane * p.max_blocks + first_page_hi] : 0;
        if (row_in_lanes) {
            bt_lo = p.bt[min(lane, p.max_blocks - 1)];
            bt_hi = p.bt[min(lane + 64, p.max_blocks - 1)];
        }
        const int n = b - a;
        const int ntl = (n + BM - 1) >> bm_shift;                  // 0 for lanes past the last segment
        const int csl = (ctx_len + STAGE - 1) / STAGE;
        const int wk = ntl > 0 ? ntl * csl + new_stages_before<STAGE>(ntl - 1, bm_shift) + (n + STAGE - 1) / STAGE : 0;
        if (lane < S) seg_tab[lane] = make_int4(a, n, ctx_len, 0);  // every wavefront writes the same values
        int t_incl = ntl, w_incl = wk;
#pragma unroll
        for (int d = 1; d < 64; d <<= 1) {
            const int y = __shfl_up(t_incl, d, 64), z = __shfl_up(w_incl, d, 64);
            if (lane >= d) { t_incl += y; w_incl += z; }
        }
        W = __builtin_amdgcn_readlane(w_incl, 63);
        TETRI_MARK(8);
        // the padding rows, shared by the G workgroups of the group
        zero_padding_rows<D>(p, grp, widx, G, tid, NT);
        Gp = min(G, W);
        if (widx >= Gp) return;
        // (the divisions run on the vector unit: their results are marked as the wave-uniform values they are)
        // and the host has checked that no product below reaches 2^31)
        pos = __builtin_amdgcn_readfirstlane((int)((uint32_t)(widx * W) / (uint32_t)Gp));
        b1 = __builtin_amdgcn_readfirstlane((int)((uint32_t)((widx + 1) * W) / (uint32_t)Gp));
        const unsigned long long owner = __builtin_amdgcn_ballot_w64(pos >= w_incl - wk && pos < w_incl);
        if (owner == 0) return;                      // cannot happen for well-formed metadata
        const int o = __builtin_ctzll(owner);
        seg.s = o;
        seg.seg_cu = __builtin_amdgcn_readlane(a, o);
        seg.n_s = __builtin_amdgcn_readlane(n, o);
        seg.L = __builtin_amdgcn_readlane(ctx_len, o);
        nt = __builtin_amdgcn_readlane(ntl, o);
        const int cs = __builtin_amdgcn_readlane(csl, o);
        page = __builtin_amdgcn_readlane(pg, o);
        page_hi = __builtin_amdgcn_readlane(pg_hi, o);
        const int seg_lin = __builtin_amdgcn_readlane(w_incl - wk, o);
        const int x = pos - seg_lin;
        // the tile of the segment position x falls into: the last one that starts at or before x
        j = 0;
        for (int j0 = 0; j0 < nt; j0 += 64) {
            const int cand = j0 + lane;
            const bool ok = cand < nt && cand * cs + new_stages_before<STAGE>(cand, bm_shift) <= x;
            const int cnt = __builtin_popcountll(__builtin_amdgcn_ballot_w64(ok));
            if (cnt == 0) break;
            j = j0 + cnt - 1;
            if (cnt < 64) break;
        }
        tile_lin = seg_lin + j * cs + new_stages_before<STAGE>(j, bm_shift);
        tile_index = __builtin_amdgcn_readlane(t_incl - ntl, o) + j;
    }

    // a job of stream mode from the cursor (seg, j, tile_lin, tile_index, pos); moves the cursor behind it
    auto stream_job = [&](const AttnParams &pp, Job &X) __attribute__((always_inline)) {
        X.grp = grp; X.kh = kh; X.seg_cu = seg.seg_cu; X.n_s = seg.n_s; X.t0 = j << bm_shift; X.tile_index = tile_index;
        X.src = make_src<D, KS>(pp, kh, seg, X.t0);
        const int n_all = X.src.n_ctx_tiles + (X.src.n_new + STAGE - 1) / STAGE;
        const int tile_end = tile_lin + n_all;
        X.it_begin = pos - tile_lin;
        X.it_end = min(b1, tile_end) - tile_lin;
        X.wf = __builtin_amdgcn_readfirstlane((int)((uint32_t)((tile_lin + 1) * Gp - 1) / (uint32_t)W));
        const int wl = __builtin_amdgcn_readfirstlane((int)((uint32_t)(tile_end * Gp - 1) / (uint32_t)W));
        X.npieces = wl - X.wf + 1;
        X.piece = widx - X.wf;
        pos = tile_lin + X.it_end;
        if (pos == tile_end) {
            tile_lin = tile_end;
            ++tile_index;
            if (++j >= nt) {
                j = 0;
                if (seg.s + 1 < S) {
                    const int4 e = seg_tab[seg.s + 1];
                    ++seg.s;
                    seg.seg_cu = __builtin_amdgcn_readfirstlane(e.x);
                    seg.n_s = __builtin_amdgcn_readfirstlane(e.y);
                    seg.L = __builtin_amdgcn_readfirstlane(e.z);
                    nt = (seg.n_s + BM - 1) >> bm_shift;
                }
            }
        }
    };
    if (G != 0) stream_job(p, J);
    TETRI_MARK(9);

    // ---- the first job's first stage and its Q rows.  The wavefronts of key part 0 reach this point
    // first (the older wavefront of a SIMD is served first), so they issue the loads of their partner
    // in part 1 as well.
    static_assert(Shape<KS>::STAGE / kPage == Shape<KS>::WAVES, "stage 0: wavefront w loads page w of the segment");
    Carry<D> cy;
    cy.par = J.it_begin & 1;                         // the first stage goes to buffer 0
    {
        // the job's Q rows, by way of the second stage buffer (its first loads go out behind the job's first barrier)
        char *q_tile = reinterpret_cast<char *>(smem + (wave < Shape<KS>::WAVES / 2 ? 1 : 3) * STAGE_U4) + (wave % (Shape<KS>::WAVES / 2)) * (32 * D * 2);
        request_q_rows<D>(p, J, grp * p.hpw + (slot & (p.hpw - 1)), slot >> p.hpw_shift, lane, lds_address(q_tile));
        const int new_row_bytes = p.Hkv * D * 2;
        LaneOffsets<D> lo;
        init_lane_offsets<D>(lo, lane);
        // entry e of the job's block-table row (clamped entries are never used)
        auto row_entry = [&](int e) -> int {
            e = min(e, p.max_blocks - 1);
            if (row_in_lanes) return e < 64 ? __builtin_amdgcn_readlane(bt_lo, e) : __builtin_amdgcn_readlane(bt_hi, e - 64);
            return ((const const_i32 *)(uintptr_t)(p.bt + J.src.bt_off))[e];
        };
        constexpr int PPS = Shape<KS>::STAGE / kPage;           // pages per stage
        cy.have_codes = false;
        if (F8 && J.it_begin < J.src.n_ctx_tiles) {
            // a pool of FP8 codes and a first stage of cached keys: every wavefront requests the codes of its own rows
            if (J.it_begin != 0 || !pages_fetched) page = row_entry(J.it_begin * PPS + wave);
            StageLoads sl;
            const bool full = describe_stage_loads<D, KS, F8>(J.src, ws, lo, page, J.it_begin, wave, new_row_bytes, lds_address(smem), sl);
            fetch_stage_codes<D>(sl, full, cy.codes);
            cy.have_codes = true;
            wait_vm<0>();
        } else if (kq == 0) {
            if (J.it_begin != 0 || !pages_fetched) {     // the lookup fetched the pages of stage 0 of its first tile
                page = row_entry(J.it_begin * PPS + wave);
                page_hi = row_entry(J.it_begin * PPS + wave + Shape<KS>::SLOTS);
            }
            StageLoads sl;
#pragma unroll
            for (int part = 0; part < Shape<KS>::PARTS; ++part) {
                const bool full = describe_stage_loads<D, KS>(J.src, ws, lo, part == 0 ? page : page_hi, J.it_begin, wave + part * Shape<KS>::SLOTS,
                                                              new_row_bytes, lds_address(smem), sl);
                issue_stage_loads<D, KS>(sl, full);
            }
            wait_vm<Shape<KS>::PARTS * 2 * (D / 32)>();      // (all but the stage's)
        } else {
            wait_vm<0>();
        }
        cy.page = row_entry((J.it_begin + 1) * PPS + wave);
        read_q_rows<D>(q_tile, lane, cy.qf);
    }
    TETRI_MARK(1);

    Handover ho;
    int guard = p.tiles + 2;                         // a workgroup never has more jobs than the chunk has tiles: malformed metadata cannot keep it here
    for (bool first = true;; first = false) {
        const bool more = G != 0 ? (pos < b1 && --guard > 0) : n_later > 0;
        Job N = J;
        if (more) {
            AttnParams pj = p;                       // before the first job's first barrier the copy in LDS may be incomplete
            if (!first) {
                asm volatile("" ::: "memory");
                pj = read_params(&params);
            }
            if (G != 0) {
                stream_job(pj, N);
            } else {
                make_piece(pj, lw0, lg0, lt0, later_whole, N);
                --n_later;
            }
        }
        tile_job<D, KS, F8, false>(p, first, &params, smem, Mstat, peek, old_stash, J, more, N, cy, ho);
        if (!more) break;
        J = N;
    }
    // ---- a piece whose hand-over was left open: if it was the last of its tile to arrive, this
    // wavefront finishes the tile from the partial results in the scratch memory (its own included).
    if (ho.unit >= 0) {
        constexpr int DBLK = D / 32;
        asm volatile("" ::: "memory");
        const AttnParams pd = read_params(&params);
        // (derived anew from the thread id: kept from the start of the kernel they would occupy registers across all jobs)
        int tid_end = threadIdx.x;
        asm volatile("" : "+v"(tid_end));
        const int lane = tid_end & 63, slot = __builtin_amdgcn_readfirstlane(tid_end >> 6) % Shape<KS>::SLOTS;
        if (__builtin_amdgcn_readfirstlane(old_stash[slot]) == ho.npieces - 1) {
            const int head = grp * pd.hpw + (slot & (pd.hpw - 1));
            const int t = ho.t0 + 32 * (slot >> pd.hpw_shift) + (lane & 31);
            if (lane == 0) store_global(pd.counters + ho.unit, 0);      // (the last to arrive: see tile_job)
            finish_tile<D, Shape<KS>::SLOTS, false>(pd, grp, ho.wf, ho.tile_index, ho.npieces, -1, slot, nullptr, 0.f, 0.f, lane, t < ho.n_s, ho.seg_cu + t, head);
        }
    }
    TETRI_MARK(7);
}

template <int D, int KS, bool F8>
hipError_t launch(const AttnParams &p, hipStream_t stream)
{
    hipLaunchKernelGGL((attn_tile_kernel<D, KS, F8>), dim3(p.attn_grid + p.append_blocks), dim3(Shape<KS>::WAVES * 64), 0, stream, p);
    return hipGetLastError();
}

}  // namespace

hipError_t tetri_launch_attn(const tetri_ctx *h, const AttnParams &p, int key_parts, bool fp8_pool, hipStream_t stream)
{
    if (p.plan != nullptr) return tetri_launch_planned(p, fp8_pool, stream);
    if (fp8_pool) {
        if (h->cfg.head_dim == 128)
            return key_parts == 2 ? launch<128, 2, true>(p, stream) : launch<128, 1, true>(p, stream);
        return key_parts == 2 ? launch<64, 2, true>(p, stream) : launch<64, 1, true>(p, stream);
    }
    if (h->cfg.head_dim == 128)
        return key_parts == 2 ? launch<128, 2, false>(p, stream) : launch<128, 1, false>(p, stream);
    return key_parts == 2 ? launch<64, 2, false>(p, stream) : launch<64, 1, false>(p, stream);
}
