// Chunked-prefill causal attention for chunks with little work in them, gfx950.
//
// The shared-tile kernel (tetri_attn.hip) is made for key ranges of thousands of keys: its workgroups of 128 rows walk
// stages of 128 keys that all wavefronts enter together, and a launch costs it about 12 us before and after that loop.
// A chunk of short prompts has a few hundred keys per row and is over before that pays.  What bounds such a launch is
// the chain of memory round trips and the number of wavefronts at work, not a throughput.  Here
//   * a workgroup owns 32 rows of one query head and its NW wavefronts share the keys: step s (32 keys) goes to
//     wavefront s % NW, each with K and V tiles of its own in LDS and no barrier in the loop (as in the decode kernel);
//   * the host, which knows the segments of the chunk, sends them and the list of row blocks, longest first,
//     along in the kernel arguments: a workgroup's first memory access is its page ids, the second K and V;
//   * few row blocks with long key ranges: the keys of a row block are split over several workgroups, so that every compute
//     unit has work; the last one to finish merges;
//   * the wavefront that does the step on the diagonal has the block's new K and V rows in LDS and writes them to their
//     page slots from there (fused append), so there are no workgroups for that.
// What bounds it in turn: the chain of steps of the wavefront with the most of them, about 0.9 us a step (FP8 codes 1.7),
// because a wavefront has one step of loads in flight and the tiles of a step serve 32 rows instead of 128.  Long chains go
// to the shared-tile kernel: the host chooses (tetri_host.cpp, plan_short).
// Arithmetic is that of the shared-tile kernel: bf16 operands, fp32 accumulation, weights rounded to bf16 before the PV
// product and summed as rounded, parts of the keys merged in a fixed order.
#include "attn_common.h"

namespace {

using namespace tetri_dev;

typedef __attribute__((address_space(4))) const ShortParams const_params;

// 32 rows of K or V, as two halves of 16 rows with a scalar base each, into a wavefront's tile (swizzled like
// everywhere); rows of a half are row_bytes apart.
template <int D>
__device__ __forceinline__ void issue_half(const char *base, uint32_t off, bool is_v, uint32_t step, uint32_t lds)
{
    constexpr int CH = D / 8, RPI = 64 / CH, NI = 16 / RPI;
    auto x = [&](int i) -> uint32_t { return (off ^ (uint32_t)((is_v ? v_swizzle<D>(RPI * i) : k_swizzle<D>(RPI * i)) * 16)) + i * step; };
    if constexpr (NI == 4) dma16_group4(base, x(0), x(1), x(2), x(3), lds);
    else dma16_group2(base, x(0), x(1), lds);
}

// Two neighbouring vectors of O (1 KB apart) and m and the row sum (128 bytes apart) of four parts, in one round trip.
__device__ __forceinline__ void load_four_partials(const char *const (&po)[4], const char *const (&ps)[4], f32x4 (&xa)[4], f32x4 (&xb)[4],
                                                   float (&m)[4], float (&l)[4])
{
    asm volatile("global_load_dword %8, %20, off sc1\n\t"
                 "global_load_dword %9, %21, off sc1\n\t"
                 "global_load_dword %10, %22, off sc1\n\t"
                 "global_load_dword %11, %23, off sc1\n\t"
                 "global_load_dword %12, %20, off offset:128 sc1\n\t"
                 "global_load_dword %13, %21, off offset:128 sc1\n\t"
                 "global_load_dword %14, %22, off offset:128 sc1\n\t"
                 "global_load_dword %15, %23, off offset:128 sc1\n\t"
                 "global_load_dwordx4 %0, %16, off sc1\n\t"
                 "global_load_dwordx4 %1, %17, off sc1\n\t"
                 "global_load_dwordx4 %2, %18, off sc1\n\t"
                 "global_load_dwordx4 %3, %19, off sc1\n\t"
                 "global_load_dwordx4 %4, %16, off offset:1024 sc1\n\t"
                 "global_load_dwordx4 %5, %17, off offset:1024 sc1\n\t"
                 "global_load_dwordx4 %6, %18, off offset:1024 sc1\n\t"
                 "global_load_dwordx4 %7, %19, off offset:1024 sc1\n\t"
                 "s_waitcnt vmcnt(0)"
                 : "=&v"(xa[0]), "=&v"(xa[1]), "=&v"(xa[2]), "=&v"(xa[3]), "=&v"(xb[0]), "=&v"(xb[1]), "=&v"(xb[2]), "=&v"(xb[3]),
                   "=&v"(m[0]), "=&v"(m[1]), "=&v"(m[2]), "=&v"(m[3]), "=&v"(l[0]), "=&v"(l[1]), "=&v"(l[2]), "=&v"(l[3])
                 : "v"(po[0]), "v"(po[1]), "v"(po[2]), "v"(po[3]), "v"(ps[0]), "v"(ps[1]), "v"(ps[2]), "v"(ps[3]) : "memory");
}

template <int D, bool F8, int NW>
__global__ __launch_bounds__(NW * 64, 2) void attn_short_kernel(ShortParams)
{
    constexpr int KSTEPS = D / 16, DBLK = D / 32, NI = D / 16, CH = D / 8, RPI = 64 / CH;
    constexpr int ROW = D * 2, TILE_BYTES = 32 * ROW;
    constexpr int ESZ = F8 ? 1 : 2;
    constexpr int LPR = D / 16, RPC = 64 / LPR, NL = 32 / RPC;      // codes: lanes per row, rows per load, loads per tile
    __shared__ __attribute__((aligned(1024))) char smem[NW * 2 * TILE_BYTES];
    __shared__ float stat[NW][2][32];
    __shared__ int last;
    const const_params *p = (const const_params *)__builtin_amdgcn_kernarg_segment_ptr();

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int half = lane >> 5, l32 = lane & 31;
    const int Hq = p->Hq, Hkv = p->Hkv;
    const int splits = p->splits;
    const int x0 = magic_div(blockIdx.x, p->splits_magic), part = blockIdx.x - x0 * splits;
    const int u = magic_div(x0, p->hq_magic), hidx = x0 - u * Hq;
    const int attn_wgs = p->units * Hq * splits;
    if ((int)blockIdx.x >= attn_wgs) {
        // ---- padding rows [rows, C) are written as +0, 16 bytes per lane and pass
        const size_t first = (size_t)p->rows * Hq * CH, n = (size_t)p->C * Hq * CH;
        const size_t stride = (size_t)(gridDim.x - attn_wgs) * (NW * 64);
        for (size_t i = first + (size_t)(blockIdx.x - attn_wgs) * (NW * 64) + tid; i < n; i += stride)
            reinterpret_cast<global_u32x4_w *>((uintptr_t)p->out)[i] = u32x4{0u, 0u, 0u, 0u};
        return;
    }
    // consecutive workgroups take different kv heads: the heads that share one run on one XCD (when Hkv is a multiple of 8)
    const int hgrp = magic_div(hidx, p->hkv_magic), kh = hidx - hgrp * Hkv, head = kh * p->g + hgrp;
    const uint32_t code = p->unit[u >> 1] >> ((u & 1) * 16);
    const int seg = code & 63, t0 = ((code >> 6) & 1023) * 32;
    const int row0 = p->cu[seg], n_s = p->cu[seg + 1] - row0, L = p->ctx[seg];
    const int ctx_steps = (L + 31) >> 5, steps = ctx_steps + (t0 >> 5) + 1;   // the last one holds the diagonal

    // the steps of this workgroup: all of them, or a part
    const int spp = splits == 1 ? steps : (steps + splits - 1) / splits;
    const int s_begin = part * spp, s_end = min(steps, s_begin + spp);
    auto clear_next = [&]() {
        const int n = p->n_counters;
        for (int i = blockIdx.x * (NW * 64) + tid; i < n; i += attn_wgs * (NW * 64)) store_global(p->counters_next + i, 0);
    };
    if (s_begin >= s_end) {
        if (splits > 1) clear_next();
        return;
    }

    const const_i32 *bt = (const const_i32 *)(uintptr_t)(p->bt + (size_t)seg * p->max_blocks);
    const int last_entry = p->max_blocks - 1;
    const size_t head_bytes = (size_t)kPage * D * ESZ, page_bytes = 2 * (size_t)Hkv * head_bytes;
    const char *pool_k = reinterpret_cast<const char *>(p->pages) + (size_t)kh * head_bytes;
    const size_t v_delta = (size_t)Hkv * head_bytes;
    const uint32_t new_row_bytes = Hkv * ROW;
    const char *new_k = reinterpret_cast<const char *>(p->k_new) + ((size_t)row0 * Hkv + kh) * ROW;
    const char *new_v = reinterpret_cast<const char *>(p->v_new) + ((size_t)row0 * Hkv + kh) * ROW;
    char *my = smem + wave * (2 * TILE_BYTES);
    const uint32_t k_lds = lds_address(my);

    int st = s_begin + wave;
    // pages of the step whose loads come next (entries past the table's end are clamped and never used)
    int pg0 = bt[min(2 * st, last_entry)], pg1 = bt[min(2 * st + 1, last_entry)];

    const int r0 = lane / CH;
    const uint32_t k_off = r0 * ROW + (((lane % CH) ^ k_swizzle<D>(r0)) << 4);
    const uint32_t v_off = r0 * ROW + (((lane % CH) ^ v_swizzle<D>(r0)) << 4);

    // K or V of step s: cached keys from the two pages, new keys from k_new / v_new
    auto issue = [&](int s, bool is_v) {
        const bool ctx = s < ctx_steps;
        const int j0 = ctx ? s * 32 : (s - ctx_steps) * 32;
        const int limit = ctx ? L : n_s;
        const char *b0, *b1;
        uint32_t stride;                             // bytes from one row to the next
        if (ctx) {
            b0 = pool_k + (size_t)pg0 * page_bytes + (is_v ? v_delta : 0);
            b1 = pool_k + (size_t)pg1 * page_bytes + (is_v ? v_delta : 0);
            stride = ROW;
        } else {
            b0 = (is_v ? new_v : new_k) + (size_t)j0 * new_row_bytes;
            b1 = b0 + (size_t)16 * new_row_bytes;
            stride = new_row_bytes;
        }
        const uint32_t lds = k_lds + (is_v ? TILE_BYTES : 0);
        const uint32_t off = (is_v ? v_off : k_off) + (uint32_t)r0 * (stride - ROW);
        const uint32_t step = RPI * (stride - ROW);
        if (j0 + 32 <= limit) {
            issue_half<D>(b0, off, is_v, step, lds);
            issue_half<D>(b1, off, is_v, step, lds + 16 * ROW);
        } else {
            // ragged end of the key range: rows past it come from a row of zeros
            const char *zero = reinterpret_cast<const char *>(g_zero_row);
#pragma unroll
            for (int i = 0; i < NI; ++i) {
                const int ri = RPI * i;
                const uint32_t swz = (uint32_t)((is_v ? v_swizzle<D>(ri & 15) : k_swizzle<D>(ri & 15)) * 16);
                const char *base = ri < 16 ? b0 : b1;
                const char *src = base + ((off ^ swz) + (uint32_t)(ri & 15) * stride);
                dma16(j0 + ri + r0 < limit ? src : zero, lds + 1024 * i);
            }
        }
    };
    // a pool of FP8 codes: the codes of a step of cached keys travel through registers
    [[maybe_unused]] u32x4 rk[NL], rv[NL];
    [[maybe_unused]] auto load_codes = [&](int s, bool is_v, u32x4 (&raw)[NL]) {
        int ln = lane;
        asm volatile("" : "+v"(ln));                 // (addresses worked out here, not kept across the loop)
#pragma unroll
        for (int i = 0; i < NL; ++i) {
            const int r = i * RPC + ln / LPR;
            const char *src = pool_k + (size_t)((i * RPC) / kPage == 0 ? pg0 : pg1) * page_bytes + (is_v ? v_delta : 0)
                              + (size_t)(r % kPage) * D + (ln % LPR) * 16;
            u32x4 v = {0u, 0u, 0u, 0u};
            if (s * 32 + r < L) v = *reinterpret_cast<global_u32x4 *>((uintptr_t)src);
            raw[i] = v;
        }
    };
    [[maybe_unused]] auto write_codes = [&](const u32x4 (&raw)[NL], bool is_v) {
        int ln = lane;
        asm volatile("" : "+v"(ln));
#pragma unroll
        for (int i = 0; i < NL; ++i) {
            const int r = i * RPC + ln / LPR, c16 = ln % LPR;
            u32x4 lo, hi;
            codes_to_bf16(raw[i], lo, hi);
            const int swz = is_v ? v_swizzle<D>(r) : k_swizzle<D>(r);
            char *row = my + (is_v ? TILE_BYTES : 0) + r * ROW;
            *reinterpret_cast<u32x4 *>(row + (((2 * c16) ^ swz) << 4)) = lo;
            *reinterpret_cast<u32x4 *>(row + (((2 * c16 + 1) ^ swz) << 4)) = hi;
            __builtin_amdgcn_sched_barrier(0);       // (one load's codes converted at a time: all at once do not fit the registers)
        }
    };
    auto request = [&](int s, bool is_v) {
        if (F8 && s < ctx_steps) load_codes(s, is_v, is_v ? rv : rk);
        else issue(s, is_v);
    };

    // Q fragments (B operand of S^T = K Q^T): column l32 is row t0 + l32; rows past the segment's end read its row t0
    bf16x8 qf[KSTEPS];
    if (st < s_end) {
        const global_u32x4 *qp = reinterpret_cast<const global_u32x4 *>((uintptr_t)(p->q + ((size_t)(row0 + t0 + (t0 + l32 < n_s ? l32 : 0)) * Hq + head) * D));
#pragma unroll
        for (int s = 0; s < KSTEPS; ++s) qf[s] = __builtin_bit_cast(bf16x8, u32x4(qp[2 * s + half]));
        request(st, false);
        request(st, true);
        pg0 = bt[min(2 * (st + NW), last_entry)];
        pg1 = bt[min(2 * (st + NW) + 1, last_entry)];
    }
    // pages of the block's own rows, for the append: positions L + t0 .. L + t0 + 31 touch up to three
    const bool appends = p->pages_w != nullptr && hgrp == 0;
    const int ap = (L + t0) / kPage;
    const int ap0 = bt[min(ap, last_entry)], ap1 = bt[min(ap + 1, last_entry)], ap2 = bt[min(ap + 2, last_entry)];

    // fragment addresses in the wavefront's tiles: those of step s / block db are the first one's with a constant XOR-ed in
    // (worked out where they are used: kept, they would take ten registers more)
    uint32_t kbase0 = l32 * ROW + ((half ^ k_swizzle<D>(l32)) << 4), vbase0;
    {
        const int blk = lane >> 4, i16 = lane & 15;
        const int rv_ = 4 * half + (i16 >> 2), d0 = 16 * (blk & 1) + 4 * (i16 & 3);
        vbase0 = TILE_BYTES + rv_ * ROW + (((d0 >> 3) ^ v_swizzle<D>(rv_)) << 4) + ((d0 & 7) << 1);
    }
    f32x16 o[DBLK];
#pragma unroll
    for (int i = 0; i < DBLK; ++i)
#pragma unroll
        for (int v = 0; v < 16; ++v) o[i][v] = 0.f;
    const float c_new = p->neg ? -p->c : p->c;
    float m = -1e30f, lsum = 0.f;                        // reference exponent of the row (not its exact maximum), this lane's row sum
    bool first = true;
    [[maybe_unused]] bool o_scaled = st >= ctx_steps;    // FP8: O is in units of code values until the first new keys

    for (; st < s_end; st += NW) {
        const bool more = st + NW < s_end, ctx = st < ctx_steps;
        const bool next_codes = F8 && st + NW < ctx_steps;       // the next step's rows come as codes
        float c = c_new;
        if constexpr (F8) {
            // the K scale rides on the score factor of cached keys, the V scale is applied to O once, before the first
            // new keys add to it (or behind the loop)
            if (ctx) {
                c = c_new * p->k_scale;
                write_codes(rk, false);
                write_codes(rv, true);
                if (next_codes) {
                    load_codes(st + NW, false, rk);
                    load_codes(st + NW, true, rv);
                }
                asm volatile("" ::: "memory");           // the fragment reads below stay behind the tile writes
            } else {
                if (!o_scaled) {
                    const float vs = p->v_scale;
#pragma unroll
                    for (int i = 0; i < DBLK; ++i)
#pragma unroll
                        for (int v = 0; v < 16; ++v) o[i][v] *= vs;
                    o_scaled = true;
                }
                wait_vm<NI>();
            }
        } else {
            wait_vm<NI>();                               // K has landed; behind it only V
        }
        asm volatile("" : "+v"(kbase0), "+v"(vbase0));
        bf16x8 kf[KSTEPS];
#pragma unroll
        for (int s = 0; s < KSTEPS; ++s) kf[s] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const uint4 *>(my + (kbase0 ^ (s << 5))));
        // fragments are in registers: the tile may be overwritten (unless the new rows in it are still to be cached: then
        // this is the last step and nothing follows)
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        if (more && !next_codes) issue(st + NW, false);
        f32x16 sc;
#pragma unroll
        for (int v = 0; v < 16; ++v) sc[v] = 0.f;
#pragma unroll
        for (int s = 0; s < KSTEPS; ++s) sc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[s], qf[s], sc, 0, 0, 0);
        // accumulator element v is key 8 * (v / 4) + 4 * half + v % 4 of the step; keys past `bound` (the end of the cached
        // context, or the lane's own row on the diagonal) get weight exp2(-inf) = 0
        if (st == steps - 1 || (ctx && st * 32 + 32 > L)) {
            const int bound = ctx ? L - 1 - st * 32 : l32;
            const float masked = c < 0.f ? INFINITY : -INFINITY;
#pragma unroll
            for (int v = 0; v < 16; ++v)
                if ((v / 4) * 8 + 4 * half + (v % 4) > bound) sc[v] = masked;
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
            m = fmaxf(m, step_max(sc, c));
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
        if (!(F8 && ctx)) {
            if (more) wait_vm<NI>();                     // V of this step: behind it only the next step's K
            else wait_vm<0>();
        }
        s16x8 vf[2 * DBLK];
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int db = 0; db < DBLK; ++db) {
                const char *a = my + (vbase0 ^ (db << 6)) + j * (16 * ROW);
                const s16x4 va = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4 *)a);
                const s16x4 vb = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4 *)(a + 8 * ROW));
                vf[j * DBLK + db] = __builtin_shufflevector(va, vb, 0, 1, 2, 3, 4, 5, 6, 7);
            }
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        if (more) {
            if (!next_codes) issue(st + NW, true);
            pg0 = bt[min(2 * (st + 2 * NW), last_entry)];
            pg1 = bt[min(2 * (st + 2 * NW) + 1, last_entry)];
        }
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int db = 0; db < DBLK; ++db)
                o[db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, vf[j * DBLK + db]), pf[j], o[db], 0, 0, 0);
    }
    if constexpr (F8) {
        if (!o_scaled) {
            const float vs = p->v_scale;
#pragma unroll
            for (int i = 0; i < DBLK; ++i)
#pragma unroll
                for (int v = 0; v < 16; ++v) o[i][v] *= vs;
        }
    }

    // ---- fused append: the wavefront of the last step has rows t0 .. t0 + 31 of K and V in its tiles
    if (appends && s_end == steps && wave == ((steps - 1 - s_begin) & (NW - 1))) {
        const int pos0 = L + t0, n_here = min(32, n_s - t0);
#pragma unroll
        for (int mat = 0; mat < 2; ++mat)
#pragma unroll
            for (int i = 0; i < NI; ++i) {
                const int r = RPI * i + r0, ch = lane % CH;
                if (r < n_here) {
                    const int pos = pos0 + r, e = pos / kPage - ap;
                    const int page = e == 0 ? ap0 : (e == 1 ? ap1 : ap2);
                    const u32x4 v = *reinterpret_cast<const u32x4 *>(my + mat * TILE_BYTES + r * ROW + ((ch ^ (mat ? v_swizzle<D>(r) : k_swizzle<D>(r))) << 4));
                    const size_t at = (size_t)page * page_bytes + (size_t)(mat * Hkv + kh) * head_bytes + (size_t)((pos % kPage) * CH + ch) * (8 * ESZ);
                    char *dst = reinterpret_cast<char *>(p->pages_w) + at;
                    if constexpr (F8) {
                        const uint2 x = bf16_to_codes(v, mat ? p->v_inv : p->k_inv);
                        *reinterpret_cast<global_u32x2_w *>((uintptr_t)dst) = u32x2{x.x, x.y};
                    } else {
                        *reinterpret_cast<global_u32x4_w *>((uintptr_t)dst) = v;
                    }
                }
            }
    }

    // ---- the wavefronts meet in LDS: each leaves its unnormalised O in its own tiles (vector (db * 4 + q4) of lane l at
    // index (db * 4 + q4) * 64 + l: no bank conflicts), m and the row sum beside; then every wavefront finishes
    // some of the columns.  Wavefronts that had no step are not looked at.
    const int parts = min(s_end - s_begin, NW);
    if (wave < parts) {
        const float ltot = half_swap_sum(lsum);
        f32x4 *mine = reinterpret_cast<f32x4 *>(my);
        static_assert(DBLK * 4 * 64 * 16 == 2 * TILE_BYTES, "an O fits a wavefront's tiles");
        asm volatile("" ::: "memory");
#pragma unroll
        for (int db = 0; db < DBLK; ++db)
#pragma unroll
            for (int q4 = 0; q4 < 4; ++q4) {
                f32x4 x;
#pragma unroll
                for (int e = 0; e < 4; ++e) x[e] = o[db][q4 * 4 + e];
                mine[(db * 4 + q4) * 64 + lane] = x;
            }
        if (half == 0) { stat[wave][0][l32] = m; stat[wave][1][l32] = ltot; }
    }
    lds_barrier();
    const int t = t0 + l32;
    float ms = stat[0][0][l32];
    for (int w = 1; w < parts; ++w) ms = fmaxf(ms, stat[w][0][l32]);
    // normalises vectors vec and vec + 1 of O and writes them: the half-waves exchange what they hold of the two, 16 bytes
    // per lane and store
    auto finish = [&](int vec, const f32x4 &a, const f32x4 &b, float l) {
        const float inv = __builtin_amdgcn_rcpf(l);
        bf16x4 wa, wb;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            wa[e] = (__bf16)(a[e] * inv);
            wb[e] = (__bf16)(b[e] * inv);
        }
        uint2 x = __builtin_bit_cast(uint2, wa), y = __builtin_bit_cast(uint2, wb);
        asm volatile("s_nop 1\n\tv_permlane32_swap_b32 %0, %2\n\tv_permlane32_swap_b32 %1, %3\n\ts_nop 1" : "+v"(x.x), "+v"(x.y), "+v"(y.x), "+v"(y.y));
        if (t < n_s) {
            uint16_t *orow = p->out + ((size_t)(row0 + t) * Hq + head) * D;
            *reinterpret_cast<global_u32x4_w *>((uintptr_t)(orow + (vec + half) * 8)) = u32x4{x.x, x.y, y.x, y.y};
        }
    };
    auto partial = [&](int i) -> float * { return p->scratch + ((size_t)(u * Hq + head) * splits + i) * (32 * D + 64); };
    // an item is 16 of the columns, two neighbouring vectors: 2 * DBLK of them
    for (int item = wave; item < 2 * DBLK; item += NW) {
        const int vec = item * 2;                        // = db * 4 + q4 with q4 in {0, 2}
        f32x4 a = {0.f, 0.f, 0.f, 0.f}, b = a;
        float l = 0.f;
        for (int w = 0; w < parts; ++w) {
            const float wgt = __builtin_amdgcn_exp2f(stat[w][0][l32] - ms);
            l = __builtin_fmaf(stat[w][1][l32], wgt, l);
            const f32x4 *src = reinterpret_cast<const f32x4 *>(smem + w * (2 * TILE_BYTES)) + lane;
            const f32x4 xa = src[vec * 64], xb = src[(vec + 1) * 64];
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                a[e] = __builtin_fmaf(xa[e], wgt, a[e]);
                b[e] = __builtin_fmaf(xb[e], wgt, b[e]);
            }
        }
        if (splits == 1) {
            finish(vec, a, b, l);
        } else {
            store_coherent(reinterpret_cast<f32x4 *>(partial(part)) + vec * 64 + lane, a);
            store_coherent(reinterpret_cast<f32x4 *>(partial(part)) + (vec + 1) * 64 + lane, b);
            if (item == 0 && half == 0) {
                store_coherent(partial(part) + 32 * D + l32, ms);
                store_coherent(partial(part) + 32 * D + 32 + l32, l);
            }
        }
    }
    if (splits == 1) return;
    clear_next();
    // ---- the parts of a row block meet in scratch memory: whoever arrives last finds all of them there, merges them in
    // part order (the result does not depend on who that is) and sets the counter back to zero.  Nobody waits.
    const int used = (steps + spp - 1) / spp;
    coherent_stores_done();
    __syncthreads();
    if (tid == 0) last = atomic_add_global(p->counters + (u * Hq + head), 1) == used - 1;
    __syncthreads();
    if (!last) return;
    if (tid == 0) store_global(p->counters + (u * Hq + head), 0);
    // (read with coherent loads, four parts per round trip; an acquire fence would empty the XCD's L2 under everybody)
    for (int item = wave; item < 2 * DBLK; item += NW) {
        const int vec = item * 2;
        f32x4 a = {0.f, 0.f, 0.f, 0.f}, b = a;
        float l = 0.f, mm = -INFINITY;
        for (int i = 0; i < used; i += 4) {
            f32x4 xa[4], xb[4];
            float mi[4], li[4];
            const char *po[4], *ps[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const float *x = partial(min(i + e, used - 1));
                po[e] = reinterpret_cast<const char *>(x) + (vec * 64 + lane) * 16;
                ps[e] = reinterpret_cast<const char *>(x + 32 * D + l32);
            }
            load_four_partials(po, ps, xa, xb, mi, li);
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                if (i + e >= used) break;
                const float m_new = fmaxf(mm, mi[e]);
                const float w_old = __builtin_amdgcn_exp2f(mm - m_new), w = __builtin_amdgcn_exp2f(mi[e] - m_new);
                mm = m_new;
                l = __builtin_fmaf(li[e], w, l * w_old);
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    a[v] = __builtin_fmaf(xa[e][v], w, a[v] * w_old);
                    b[v] = __builtin_fmaf(xb[e][v], w, b[v] * w_old);
                }
            }
        }
        finish(vec, a, b, l);
    }
}

template <int D, bool F8>
hipError_t launch(const ShortParams &p, int wavefronts, hipStream_t stream)
{
    const dim3 grid(p.units * p.Hq * p.splits + p.zero_wgs);
    if (wavefronts == 8) hipLaunchKernelGGL((attn_short_kernel<D, F8, 8>), grid, dim3(512), 0, stream, p);
    else if (wavefronts == 2) hipLaunchKernelGGL((attn_short_kernel<D, F8, 2>), grid, dim3(128), 0, stream, p);
    else if (wavefronts == 1) hipLaunchKernelGGL((attn_short_kernel<D, F8, 1>), grid, dim3(64), 0, stream, p);
    else hipLaunchKernelGGL((attn_short_kernel<D, F8, 4>), grid, dim3(256), 0, stream, p);
    return hipGetLastError();
}

}  // namespace

hipError_t tetri_launch_short(int head_dim, bool fp8_pool, const ShortParams &p, int wavefronts, hipStream_t stream)
{
    if (head_dim == 128) return fp8_pool ? launch<128, true>(p, wavefronts, stream) : launch<128, false>(p, wavefronts, stream);
    return fp8_pool ? launch<64, true>(p, wavefronts, stream) : launch<64, false>(p, wavefronts, stream);
}
