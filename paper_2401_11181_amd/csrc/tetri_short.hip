// Chunked-prefill causal attention for chunks with little work in them, gfx950.
//
// The shared-tile kernel (tetri_attn.hip, tetri_planned.hip) is made for key ranges of thousands of keys: its workgroups of 128 or 256
// rows walk stages of 128 keys that all wavefronts enter together, and a launch costs it 9 to 12 us before and after that loop.
// A chunk of short prompts has a few hundred keys per row and is over before that pays.  What bounds such a launch is
// the chain of memory round trips and the number of wavefronts at work, not a throughput.  Here
//   * a row block of 32 rows of one query head is the work of a team of 1, 2, 4 or 8 wavefronts that share its keys: step s (32
//     keys) goes to wavefront s modulo the team, each with two regions of its own in LDS and no barrier in the loop (as in the
//     decode kernel).  The host, which knows the segments of the chunk, gives each row block the team that leaves its
//     wavefronts about as many steps as those of the others and fills the chip's places for wavefronts (plan_short): with one
//     size of team for all row blocks a launch lasted as long as its longest one (512 rows of 40 heads: 18.3 us, now 14.0; 286 short
//     prompts of 40 heads, 71 chunks: 1154 us, with teams 1006);
//   * the row blocks, longest first, travel in the kernel arguments: a workgroup's first memory access after those is its page
//     ids, the second Q, K and V;
//   * few row blocks with long key ranges: the keys of a row block are split over several workgroups, so that every compute
//     unit has work; the last one to finish merges;
//   * codes of an FP8 cache stay codes in LDS, a step in the place of one matrix of a 16-bit step, and become bf16 (exactly) where
//     their fragments are read: two steps in flight and no second trip through registers and LDS (512 rows of 32/8 heads at 1000 cached
//     tokens: 38 us, now 29.5);
//   * the wavefront that does the step on the diagonal has the block's new K and V rows in LDS and writes them to their
//     page slots from there (fused append), so there are no workgroups for that.
// What bounds it in turn: the chain of steps of the wavefront with the most of them, 1.0 to 1.3 us a step, because a wavefront
// has one step of loads in flight (codes two) and the keys of a step serve 32 rows instead of 256.  Long chains go to the shared-tile
// kernel: the host chooses.  The 71 packed chunks of 286 short prompts take 12.6 us each.  At 13.7, by clock values stored at points of the kernel
// (which cost 2 %), they were 2.4 us from the last wavefront's end to the next launch's first instruction, then for the wavefront that
// ends last 0.8 to its row block, 0.4 to its page ids, 4.2 to Q and the first K (up to 16 MB that no launch before has touched, all
// asked for at once; 2.3 in the median wavefront), 2.9 the steps, 1.9 the append and the team's barrier, 1.3 merge and output.
// Arithmetic is that of the shared-tile kernel: bf16 operands, fp32 accumulation, weights rounded to bf16 before the PV
// product and summed as rounded, parts of the keys merged in a fixed order.
#include <string.h>

#include <type_traits>

#include "attn_common.h"

namespace {

using namespace tetri_dev;

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

// 16 codes per lane and instruction: how the 32 rows of a step of cached keys lie in a region, K codes then V codes (rows of D
// bytes, 16-byte chunks XOR-ed by the row).
template <int D> struct CodeTile {
    static constexpr int CH = D / 16, BYTES = 32 * D, RPI = 1024 / D, NI = BYTES / 1024, PI = 16 / RPI;
    static __device__ __forceinline__ constexpr int swizzle(int row) { return D == 128 ? row & 7 : (row >> 2) & 3; }
};

// Bytes of the kernel's arguments in front of its structure (which starts on a cache line).  What a wavefront's row block is found with
// comes first and by itself: those words are in scalar registers when a wavefront starts, and the row block, with the pointers that
// go with it, is one read of the arguments away instead of two.
// (Ragged prompts over codes 649.9 us with the words read from memory, 642.8 so; the packed chunks above 998.7, so 977.0.)
constexpr int kShortLead = 64;

// Args: ShortArgs, or ShortCarry for the first launch of a batch's step, which brings the metadata of all its launches (block_tables is then
// the offset of the chunk's in it, in int32): one launch less in front of the first result.  (Four chunks of 64 rows of 4 heads of 64: 23.5 us with
// the upload in front, 20.1 so; four of 512 of 40 heads 116.3, 115.3.)
template <int D, bool F8, int NW, typename Args>
__global__ __launch_bounds__(NW * 64, D == 64 ? (F8 ? 3 : 4) : 2) void attn_short_kernel(
    const int32_t *block_tables, int max_blocks, int first_wg0, int first_wg1, int first_wg2, uint32_t first_units, int attn_wgs, uint32_t shape,
    uint32_t splits_magic, uint32_t hpx_magic, uint32_t hkx_magic, uint32_t per_x, Args)
{
    constexpr bool CARRY = std::is_same<Args, ShortCarry>::value;
    typedef __attribute__((address_space(4))) const Args const_params;
    typedef CodeTile<D> CT;
    constexpr int KSTEPS = D / 16, DBLK = D / 32, NI = D / 16, CH = D / 8, RPI = 64 / CH;
    constexpr int ROW = D * 2, TILE_BYTES = 32 * ROW;
    constexpr int ESZ = F8 ? 1 : 2, NWL = NW == 8 ? 3 : 2;
    static_assert(2 * CT::NI == NI && 2 * CT::BYTES == TILE_BYTES, "a step of codes takes a region");
    __shared__ __attribute__((aligned(1024))) char smem[NW * 2 * TILE_BYTES];
    __shared__ __attribute__((aligned(1024))) char q_rows[F8 ? 16 : NW / 4 * TILE_BYTES];      // of teams of 4 and 8, 16-bit cache
    __shared__ float stat[NW][2][32];
    __shared__ int last;
    // (the structure lies behind the leading arguments)
    const const_params *p = (const const_params *)((__attribute__((address_space(4))) const char *)__builtin_amdgcn_kernarg_segment_ptr() + kShortLead);

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int half = lane >> 5, l32 = lane & 31;
    const int bid = blockIdx.x;
    if (bid >= attn_wgs) {
        const int extra = bid - attn_wgs - (int)CARRY;
        if constexpr (CARRY) {
            if (extra < 0) {                             // ---- the metadata, first: the launches behind this one wait for it
                const int n = p->meta_vectors;
                const auto *v = (__attribute__((address_space(4))) const u32x4 *)p->meta;
                for (int i = tid; i < n; i += NW * 64) reinterpret_cast<global_u32x4_w *>((uintptr_t)p->meta_dev)[i] = v[i];
                return;
            }
        }
        const int fetch_wgs = F8 ? 0 : p->fetch_wgs;
        if (extra < fetch_wgs) {
            // ---- rows of the next chunk, 1 KB to an instruction, into a place that nobody reads: they are in the cache in front of the memory
            // when its launch asks for them.  What bounds a launch is that all of its first reads are made at once and none after that: 512 rows of
            // 40 heads are 16 MB, 4.2 us, of 13.  (286 short prompts of 40 heads, 71 chunks, 928 us without this; 4 us of sleep before: 893, none 897, 8 us 919.  With
            // 16 KB to a wavefront 920, 40 905, 64 974: a compute unit takes 25 GB/s of such reads.  Asked for by the wavefronts with row blocks, behind their
            // loop, 945, behind their first step 990.  With Q, K and V in the cache from the start, 748.)
            const uint32_t k_kb = p->next_kb[0], v_kb = p->next_kb[1], n = k_kb + v_kb + p->next_kb[2], kv_bytes = p->next_bytes[0], q_bytes = p->next_bytes[1];
            const char *const nx[3] = {reinterpret_cast<const char *>(p->next[0]), reinterpret_cast<const char *>(p->next[1]),
                                       reinterpret_cast<const char *>(p->next[2])};
            const uint32_t to = lds_address(smem + wave * 1024);
            __builtin_amdgcn_s_sleep(64);                // (2 us: behind the launch's own first reads)
            for (uint32_t i = extra * NW + wave; i < n; i += fetch_wgs * NW) {
                const FetchAt f = fetch_at(i, lane, k_kb, v_kb, kv_bytes, q_bytes);
                dma16((f.matrix == 0 ? nx[0] : (f.matrix == 1 ? nx[1] : nx[2])) + f.byte, to);
            }
            wait_vm<0>();                                // (nothing may be on its way to LDS when a wavefront ends)
            return;
        }
        // ---- padding rows [rows, C) are written as +0, 16 bytes per lane and pass
        const size_t first = (size_t)p->rows * p->Hq * CH, n = (size_t)p->C * p->Hq * CH;
        const size_t stride = (size_t)(gridDim.x - attn_wgs - fetch_wgs - (int)CARRY) * (NW * 64);
        for (size_t i = first + (size_t)(extra - fetch_wgs) * (NW * 64) + tid; i < n; i += stride)
            reinterpret_cast<global_u32x4_w *>((uintptr_t)p->out)[i] = u32x4{0u, 0u, 0u, 0u};
        return;
    }
    // ---- the wavefront's row block, head and place in its team.  Row blocks come in classes of 8, 4, 2 or 1 wavefronts (1 <<
    // tl), the longest first.  The heads whose kv head is x modulo R (R = 1 << rshift) sit in workgroups x modulo R: those
    // that share a kv head run on one XCD (R = 8).
    const ShortShapeWords sw = short_unpack({first_units, shape, per_x});
    const int fu0 = sw.first_unit[0], fu1 = sw.first_unit[1], fu2 = sw.first_unit[2], units = sw.units;
    const int splits = sw.splits, rshift = sw.rshift, hpx = sw.hpx, hkx = sw.hkx;
    const int tl = bid >= first_wg0 ? 0 : (bid >= first_wg1 ? 1 : (bid >= first_wg2 ? 2 : 3));
    const int T = 1 << tl;
    int j = bid - (tl == 0 ? first_wg0 : (tl == 1 ? first_wg1 : (tl == 2 ? first_wg2 : 0)));
    const int u_first = tl == 0 ? fu0 : (tl == 1 ? fu1 : (tl == 2 ? fu2 : 0));
    const int u_end = tl == 0 ? units : (tl == 1 ? fu0 : (tl == 2 ? fu1 : fu2));
    int part = 0;
    if (splits > 1) {
        const int q = magic_div(j, splits_magic);
        part = j - q * splits;
        j = q;
    }
    const int x = j & ((1 << rshift) - 1);
    const int pack = sw.spread != 0 ? 0 : NWL - tl;      // log2 of a workgroup's teams (few row blocks: one, on a compute unit of its own)
    const int team_ = wave >> tl, item_ = ((j >> rshift) << pack) + team_, rank = wave & (T - 1), team0 = wave - rank;
    const int ul = magic_div(item_, hpx_magic), hh = item_ - ul * hpx;
    const int hgrp = magic_div(hh, hkx_magic), kh = x + ((hh - hgrp * hkx) << rshift);
    const bool valid = u_first + ul < u_end && (team_ >> pack) == 0;
    const int u = valid ? u_first + ul : u_first;

    // the row block, and the launch's shape and pointers, in one round trip: read where they are used, they are four or five
    typedef __attribute__((ext_vector_type(16))) int i32x16;
    typedef __attribute__((ext_vector_type(2))) int i32x2s;
    typedef __attribute__((address_space(4))) const i32x16 const_i32x16;
    typedef __attribute__((address_space(4))) const i32x2s const_i32x2s;
    static_assert(offsetof(ShortArgs, q) == 0 && offsetof(ShortArgs, Hq) == 56 && offsetof(ShortArgs, g) == 64, "read as vectors");
    i32x16 hp = *(const const_i32x16 *)p;
    i32x2s hg = *(const const_i32x2s *)&p->g, unit = *(const const_i32x2s *)&p->unit[u];
    asm volatile("" : "+s"(hp), "+s"(hg), "+s"(unit));
    auto pointer = [&](auto i) __attribute__((always_inline)) -> char * {
        constexpr int I = decltype(i)::value;
        return reinterpret_cast<char *>((uintptr_t)((uint64_t)(uint32_t)hp[2 * I] | (uint64_t)(uint32_t)hp[2 * I + 1] << 32));
    };
    typedef std::integral_constant<int, 0> R0;
    typedef std::integral_constant<int, 1> R1;
    char *const p_q = pointer(R0()), *const p_k_new = pointer(R1()), *const p_v_new = pointer(std::integral_constant<int, 2>()),
         *const p_pages = pointer(std::integral_constant<int, 3>()), *const p_out = pointer(std::integral_constant<int, 4>()),
         *const p_pages_w = pointer(std::integral_constant<int, 5>()), *const p_zero = pointer(std::integral_constant<int, 6>());
    const int Hq = hp[14], Hkv = hp[15], heads_per_kv = hg[0], out_past_l2 = hg[1];
    const uint32_t unit_lo = unit[0], unit_hi = unit[1];
    const int seg = unit_lo & 63, t0 = ((unit_lo >> 6) & 127) * 32, n_s = (unit_lo >> 13) & 8191, L = unit_hi & 0x3ffffff;
    const int row0 = (int)(unit_lo >> 26) | (int)(unit_hi >> 26) << 6;
    const int head = kh * heads_per_kv + hgrp;
    const int ctx_steps = (L + 31) >> 5, steps = ctx_steps + (t0 >> 5) + 1;   // the last one holds the diagonal

    // the steps of this team: all of the row block's, or a part
    const int spp = splits == 1 ? steps : (steps + splits - 1) / splits;
    const int s_begin = part * spp, s_end = min(steps, s_begin + spp);
    auto clear_next = [&]() {
        const int n = p->n_counters;
        for (int i = bid * (NW * 64) + tid; i < n; i += attn_wgs * (NW * 64)) store_global(p->counters_next + i, 0);
    };
    if (splits > 1 && s_begin >= s_end) {
        clear_next();
        return;
    }

    const const_i32 *bt;
    if constexpr (CARRY) bt = (const const_i32 *)p->meta + ((uintptr_t)block_tables + (size_t)seg * max_blocks);
    else bt = (const const_i32 *)(uintptr_t)(block_tables + (size_t)seg * max_blocks);
    const int last_entry = max_blocks - 1;
    const size_t head_bytes = (size_t)kPage * D * ESZ, page_bytes = 2 * (size_t)Hkv * head_bytes;
    const char *pool_k = p_pages + (size_t)kh * head_bytes;
    const size_t v_delta = (size_t)Hkv * head_bytes;
    const uint32_t new_row_bytes = Hkv * ROW;
    const char *new_k = p_k_new + ((size_t)row0 * Hkv + kh) * ROW;
    const char *new_v = p_v_new + ((size_t)row0 * Hkv + kh) * ROW;
    char *my = smem + wave * (2 * TILE_BYTES);
    const uint32_t my_lds = lds_address(my);

    // The wavefront's steps: every T-th of the team's, upwards: codes first (O is scaled once, where the new keys begin).  (From the
    // diagonal down, with the block's own rows cached in the first step: 226 registers instead of 179, 2 % less for 286 short
    // prompts of 40 heads, 1 to 7 % more for chunks of 32/8 and 24/8.)
    int st = s_begin + rank;
    int left = valid ? (s_end - s_begin - rank + T - 1) >> tl : 0;             // steps the wavefront still has
    const int parts = min(s_end - s_begin, T);                                  // wavefronts of the team that have any
    const bool owns_diagonal = s_end == steps && rank == ((steps - 1 - s_begin) & (T - 1));
    const bool appends = p_pages_w != nullptr && hgrp == 0 && left > 0 && owns_diagonal;

    // ---- The loads are a stream of regions of TILE_BYTES, NI instructions each, that alternate between the wavefront's two: K
    // and V rows of a 16-bit step, or K and V codes of one step; a region's next load goes out when its rows have been read.
    // (codes: the first region is chosen so that the last step of codes lies in region 1)
    const int code_steps = F8 ? min(left, max(0, (ctx_steps - st + T - 1) >> tl)) : 0;
    int fs = st, fleft = left;                           // the step whose loads go out next, and how many with it are left
    int pg0 = 0, pg1 = 0;                                // its pages (entries past the table's end are clamped and never used)
    auto pages_of = [&](int s) __attribute__((always_inline)) {
        pg0 = bt[min(max(2 * s, 0), last_entry)];
        pg1 = bt[min(max(2 * s + 1, 0), last_entry)];
    };
    pages_of(fs);
    const int r0 = lane / CH;
    const uint32_t k_off = r0 * ROW + (((lane % CH) ^ k_swizzle<D>(r0)) << 4);
    const uint32_t v_off = r0 * ROW + (((lane % CH) ^ v_swizzle<D>(r0)) << 4);
    // K or V rows of step fs: cached keys from the two pages, new keys from k_new / v_new
    auto issue_rows = [&](bool is_v, uint32_t lds) __attribute__((always_inline)) {
        const int s = fs;
        const bool ctx = s < ctx_steps;
        const int j0 = ctx ? s * 32 : (s - ctx_steps) * 32;
        const int limit = ctx ? L : n_s;
        const char *b0, *b1;
        uint32_t stride;                             // bytes from one row to the next
        if (!F8 && ctx) {
            b0 = pool_k + (size_t)pg0 * page_bytes + (is_v ? v_delta : 0);
            b1 = pool_k + (size_t)pg1 * page_bytes + (is_v ? v_delta : 0);
            stride = ROW;
        } else {
            b0 = (is_v ? new_v + 0 : new_k + 0) + (size_t)j0 * new_row_bytes;
            b1 = b0 + (size_t)16 * new_row_bytes;
            stride = new_row_bytes;
        }
        const uint32_t off = (is_v ? +v_off : +k_off) + (uint32_t)r0 * (stride - ROW);
        const uint32_t step = RPI * (stride - ROW);
        if (j0 + 32 <= limit) {
            issue_half<D>(b0, off, is_v, step, lds);
            issue_half<D>(b1, off, is_v, step, lds + 16 * ROW);
        } else {
            // ragged end of the key range: rows past it come from a row of zeros
            int ln = lane;
            if constexpr (D == 64) asm volatile("" : "+v"(ln));       // (worked out here, not kept across the loop)
            const int rl = ln / CH;
#pragma unroll
            for (int i = 0; i < NI; ++i) {
                const int ri = RPI * i;
                const uint32_t swz = (uint32_t)((is_v ? v_swizzle<D>(ri & 15) : k_swizzle<D>(ri & 15)) * 16);
                const char *base = ri < 16 ? b0 : b1;
                const char *src = base + ((off ^ swz) + (uint32_t)(ri & 15) * stride);
                dma16(j0 + ri + rl < limit ? src : p_zero, lds + 1024 * i);
            }
        }
    };
    // the codes of step fs, K then V
    [[maybe_unused]] auto issue_codes = [&](uint32_t lds) __attribute__((always_inline)) {
        int ln = lane;
        asm volatile("" : "+v"(ln));                 // (offsets worked out here, not kept across the loop)
        const int rc = ln / CT::CH;
        const uint32_t off = rc * D + (((ln % CT::CH) ^ CT::swizzle(rc)) << 4);
        const bool full = fs * 32 + 32 <= L;
#pragma unroll
        for (int mat = 0; mat < 2; ++mat) {
            const char *b0 = pool_k + (size_t)pg0 * page_bytes + (mat ? v_delta : 0), *b1 = pool_k + (size_t)pg1 * page_bytes + (mat ? v_delta : 0);
            const uint32_t at = lds + mat * CT::BYTES;
            if (full) {
                if constexpr (CT::PI == 2) {
                    dma16_group2(b0, off, off, at);
                    dma16_group2(b1, off, off, at + 2048);
                } else {
                    dma16(b0 + off, at);
                    dma16(b1 + off, at + 1024);
                }
            } else {
    #pragma unroll
                for (int i = 0; i < CT::NI; ++i) {
                    const int r = CT::RPI * i;
                    const char *src = (r < 16 ? b0 : b1) + (r & 15) * D + off;
                    dma16(fs * 32 + r + rc < L ? src : p_zero, at + 1024 * i);
                }
            }
        }
    };
    // the stream's next load, into `region` (of 16-bit rows: K into 0, V into 1)
    auto feed = [&](auto reg) __attribute__((always_inline)) {
        constexpr int region = decltype(reg)::value;
        if (fleft <= 0) return;
        const uint32_t lds = my_lds + region * TILE_BYTES;
        bool step_done;
        if (F8 && fs < ctx_steps) {
            issue_codes(lds);
            step_done = true;
        } else {
            issue_rows(region == 1, lds);
            step_done = region == 1;
        }
        if (step_done) {
            fs += T;
            --fleft;
            pages_of(fs);
        }
    };

    // fragment addresses in the regions: those of step s / block db are the first one's with a constant XOR-ed in (worked out
    // where they are used: kept, they would take ten registers more).  16-bit rows: accumulator element v is key 8 * (v / 4)
    // + 4 * half + v % 4 of the step.  Codes: a V fragment holds 8 consecutive keys, so K rows are read in the order that makes
    // element v key 16 * (v / 8) + 8 * half + v % 8 (bits 2 and 3 of the row index change places).
    uint32_t kbase0 = l32 * ROW + ((half ^ k_swizzle<D>(l32)) << 4), vbase0, kcode0 = 0, vcode0 = 0;
    {
        const int blk = lane >> 4, i16 = lane & 15;
        const int rv_ = 4 * half + (i16 >> 2), d0 = 16 * (blk & 1) + 4 * (i16 & 3);
        vbase0 = TILE_BYTES + rv_ * ROW + (((d0 >> 3) ^ v_swizzle<D>(rv_)) << 4) + ((d0 & 7) << 1);
        if constexpr (F8) {
            const int row = (l32 & 19) | (l32 & 4) << 1 | (l32 & 8) >> 1;
            kcode0 = row * D + (CT::swizzle(row) << 4) + 8 * half;
            const int rc = 8 * half + (i16 >> 1);
            vcode0 = CT::BYTES + rc * D + (((blk & 1) ^ CT::swizzle(rc)) << 4) + 8 * (i16 & 1);
        }
    }
    // Q fragments (B operand of S^T = K Q^T): column l32 is row t0 + l32; rows past the segment's end are its row t0.  The rows
    // come by way of LDS, whole rows per instruction: as fragments, 32 bytes of 32 rows each, they took 1.6 us more of a launch with
    // 1920 wavefronts.  (Fragments loaded from inline assembly with the wait further down are not safe: where the compiler spills, it
    // spills registers that the load has yet to write.)
    const int n_here = min(32, n_s - t0);
    bf16x8 qf[KSTEPS];
    int region = F8 ? (code_steps & 1) : 0;                   // of the step about to run (a 16-bit step: 0, and 1 for V)
    const uint32_t q_row = Hq * ROW;
    const char *qb = p_q + ((size_t)(row0 + t0) * Hq + head) * ROW;
    auto q_source = [&](int i) __attribute__((always_inline)) -> const char * {     // of instruction i of the block's rows
        const int r = RPI * i + r0;
        return qb + (size_t)(r < n_here ? r : 0) * q_row + (((lane % CH) ^ k_swizzle<D>(r)) << 4);
    };
    auto read_q = [&](const char *qt) __attribute__((always_inline)) {
#pragma unroll
        for (int s = 0; s < KSTEPS; ++s) qf[s] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const uint4 *>(qt + (kbase0 ^ (s << 5))));
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    };
    // A team of 4 or 8 loads them once, a share each wavefront, into a place of their own: nothing of the stream waits for them (286
    // short prompts of 40 heads: 981.0 us, this way 977.7).  The others take the region that the stream needs second (places of their
    // own would not fit); so do all teams over codes, whose regions hold whole steps (ragged prompts of 32/8 heads: 642.5 us
    // with a place of their own, 640.6 without).
    const bool shared_q = !F8 && tl >= 2;
    char *qt = shared_q ? q_rows + (valid ? team_ : 0) * TILE_BYTES : my + (region ^ 1) * TILE_BYTES;
    if (shared_q) {
        if (valid)
            for (int i = rank; i < NI; i += T) dma16(q_source(i), lds_address(qt) + 1024 * i);
    } else if (left > 0) {
        if (n_here == 32) {
            const uint32_t off = r0 * q_row + (((lane % CH) ^ k_swizzle<D>(r0)) << 4), step = RPI * q_row - 1024;
            issue_half<D>(qb, off, false, step, lds_address(qt));
            issue_half<D>(qb + (size_t)16 * q_row, off, false, step, lds_address(qt) + 16 * ROW);
        } else {
#pragma unroll
            for (int i = 0; i < NI; ++i) dma16(q_source(i), lds_address(qt) + 1024 * i);
        }
    }
    if (left > 0) {
        if (F8 && region != 0) feed(R1());
        else feed(R0());
        if (!shared_q) {
            wait_vm<NI>();                                   // behind Q only the first load of the stream
            read_q(qt);
        }
        if (F8 && region != 0) feed(R0());
        else feed(R1());
    }
    if (shared_q) {
        // (the wavefront's share; behind it the stream's first two loads)
        if (left <= 0) wait_vm<0>();
        else wait_vm<2 * NI>();
        lds_barrier();
        read_q(qt);
    }
    // pages of the block's own rows, for the append: positions L + t0 .. L + t0 + 31 touch up to three
    const int ap = (L + t0) / kPage;
    const int ap0 = bt[min(ap, last_entry)], ap1 = bt[min(ap + 1, last_entry)], ap2 = bt[min(ap + 2, last_entry)];

    f32x16 o[DBLK];
#pragma unroll
    for (int i = 0; i < DBLK; ++i)
#pragma unroll
        for (int v = 0; v < 16; ++v) o[i][v] = 0.f;
    const float c_new = p->neg ? -p->c : p->c;
    float m = -1e30f, lsum = 0.f;                        // reference exponent of the row (not its exact maximum), this lane's row sum
    bool first = true;

    // (Steps of codes and of rows are two loops.  In one loop the ways through it that multiply O and those that do not met in registers of their own: O
    // was copied twice a step of codes, 64 instructions, and 254 registers were in use, now 199.  Ragged prompts of 32/8 heads over codes 636 us, now 599.)
    auto step = [&](auto codes_) __attribute__((always_inline)) {
        constexpr bool codes = decltype(codes_)::value;
        const bool more = left > 1, ctx = codes || st < ctx_steps;
        const float c = codes ? c_new * p->k_scale : c_new;
        // K has landed when only what was issued after it is outstanding: the other region's load (behind a step of codes, if there
        // is one; the V rows of a 16-bit step) and the second half of a step of codes
        if (codes) {
            if (more) wait_vm<NI + NI / 2>();
            else wait_vm<NI / 2>();
        } else {
            wait_vm<NI>();
        }
        asm volatile("" : "+v"(kbase0), "+v"(vbase0));
        if constexpr (F8) asm volatile("" : "+v"(kcode0), "+v"(vcode0));
        const char *tile = my + region * TILE_BYTES;     // (a step of codes)
        bf16x8 kf[KSTEPS];
        if (codes) {
#pragma unroll
            for (int s = 0; s < KSTEPS; ++s) {
                const uint2 y = *reinterpret_cast<const uint2 *>(tile + (kcode0 ^ (s << 4)));
                kf[s] = codes_to_bf16(y.x, y.y);
            }
        } else {
#pragma unroll
            for (int s = 0; s < KSTEPS; ++s) kf[s] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const uint4 *>(my + (kbase0 ^ (s << 5))));
        }
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");  // the rows are in registers: the region may be overwritten
        if (!codes && more) feed(R0());
        f32x16 sc;
#pragma unroll
        for (int v = 0; v < 16; ++v) sc[v] = 0.f;
#pragma unroll
        for (int s = 0; s < KSTEPS; ++s) sc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[s], qf[s], sc, 0, 0, 0);
        // keys past `bound` (the end of the cached context, or the lane's own row on the diagonal) get weight exp2(-inf) = 0
        if (st == steps - 1 || (ctx && st * 32 + 32 > L)) {
            const int bound = ctx ? L - 1 - st * 32 : l32;
            const float masked = c < 0.f ? INFINITY : -INFINITY;
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                const int key = codes ? 16 * (v / 8) + 8 * half + v % 8 : 8 * (v / 4) + 4 * half + v % 4;
                if (key > bound) sc[v] = masked;
            }
        }
        bf16x8 pf[2];
        // (a lambda: as a function shared by the kernels it made the short kernel 4 % slower)
        auto weights = [&]() __attribute__((always_inline)) {                           // rounded to bf16 for the PV product
#pragma unroll
            for (int v = 0; v < 16; v += 2) {
                pf[v / 8][v % 8] = (__bf16)__builtin_amdgcn_exp2f(__builtin_fmaf(sc[v], c, -m));
                pf[v / 8][v % 8 + 1] = (__bf16)__builtin_amdgcn_exp2f(__builtin_fmaf(sc[v + 1], c, -m));
            }
        };
        if constexpr (F8) {
            // (one branch that writes to O, in place: the first step's multiplies nothing by nothing)
            bool raise = first;
            if (!first) {
                weights();
                raise = weights_reach_two(pf);
            }
            first = false;
            if (raise) {
                const float m_new = fmaxf(m, step_max(sc, c));
                const float alpha = __builtin_amdgcn_exp2f(m - m_new);
                m = m_new;
                lsum *= alpha;
                scale_in_place(o, alpha);
                weights();
            }
        } else if (first) {
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
        // V has landed: behind it only the next load of the stream
        if (codes) {
            if (more) wait_vm<NI>();
            else wait_vm<0>();
        } else if (more) {
            wait_vm<NI>();
        } else {
            wait_vm<0>();
        }
        bf16x8 vf[2 * DBLK];
        if (codes) {
#pragma unroll
            for (int jj = 0; jj < 2; ++jj)
#pragma unroll
                for (int db = 0; db < DBLK; ++db) {
                    const i32x2 y = __builtin_amdgcn_ds_read_tr8_b64_v2i32((lds_i32x2 *)(tile + (vcode0 ^ (db << 5)) + jj * (16 * D)));
                    vf[jj * DBLK + db] = codes_to_bf16((uint32_t)y[0], (uint32_t)y[1]);
                }
        } else {
#pragma unroll
            for (int jj = 0; jj < 2; ++jj)
#pragma unroll
                for (int db = 0; db < DBLK; ++db) {
                    const char *a = my + (vbase0 ^ (db << 6)) + jj * (16 * ROW);
                    const s16x4 va = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4 *)a);
                    const s16x4 vb = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4 *)(a + 8 * ROW));
                    vf[jj * DBLK + db] = __builtin_bit_cast(bf16x8, __builtin_shufflevector(va, vb, 0, 1, 2, 3, 4, 5, 6, 7));
                }
        }
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        if (codes) {
            if (region != 0) feed(R1());
            else feed(R0());
            region ^= 1;
        } else if (more) {
            feed(R1());
        }
#pragma unroll
        for (int jj = 0; jj < 2; ++jj)
#pragma unroll
            for (int db = 0; db < DBLK; ++db)
                o[db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vf[jj * DBLK + db], pf[jj], o[db], 0, 0, 0);
    };
    if constexpr (F8) {
        // the K scale rides on the score factor of cached keys, the V scale is applied to O once, before the first new keys add to it
        if (code_steps > 0) {
            for (int i = 0; i < code_steps; ++i, --left, st += T) step(std::true_type());
            scale_in_place(o, p->v_scale);
        }
    }
    for (; left > 0; --left, st += T) step(std::false_type());
    // ---- fused append: the wavefront of the last step has rows t0 .. t0 + 31 of K and V in its regions.  (The rows of a matrix are read
    // together: row by row, each behind the condition of its store, its LDS round trips held the whole team up before the merge: 286
    // short prompts of 40 heads 987.1 us, this way 977.9; ragged prompts over codes 648.9, this way 642.3.)
    // How they are stored the host says (new_row_stores), in ways of their own: decided store by store, a chunk of 128 rows of 8/2 heads took 0.6 us more.
    if (appends) {
        const int slot0 = (L + t0) % kPage, ch = lane % CH;
        auto append_rows = [&](auto how_) __attribute__((always_inline)) {
            constexpr int HOW = decltype(how_)::value;
#pragma unroll
            for (int mat = 0; mat < 2; ++mat) {
                char *const slab = p_pages_w + (size_t)(mat * Hkv + kh) * head_bytes;
                char *const to0 = slab + (size_t)ap0 * page_bytes, *const to1 = slab + (size_t)ap1 * page_bytes, *const to2 = slab + (size_t)ap2 * page_bytes;
                u32x4 rows[NI];
#pragma unroll
                for (int i = 0; i < NI; ++i) {
                    const int r = RPI * i + r0;
                    rows[i] = *reinterpret_cast<const u32x4 *>(my + mat * TILE_BYTES + r * ROW + ((ch ^ (mat ? v_swizzle<D>(r) : k_swizzle<D>(r))) << 4));
                }
#pragma unroll
                for (int i = 0; i < NI; ++i) asm volatile("" : "+v"(rows[i]));
#pragma unroll
                for (int i = 0; i < NI; ++i) {
                    const int r = RPI * i + r0, e = (slot0 + r) / kPage;
                    char *dst = (e == 0 ? to0 : (e == 1 ? to1 : to2)) + (uint32_t)(((slot0 + r) % kPage) * CH + ch) * (8 * ESZ);
                    if (r < n_here) {
                        if constexpr (F8) {
                            const uint2 y = bf16_to_codes(rows[i], mat ? p->v_inv : p->k_inv);
                            global_u32x2_w *at = reinterpret_cast<global_u32x2_w *>((uintptr_t)dst);
                            if constexpr (HOW == kRowsThrough) store_coherent(at, u32x2{y.x, y.y});
                            else *at = u32x2{y.x, y.y};
                        } else {
                            global_u32x4_w *at = reinterpret_cast<global_u32x4_w *>((uintptr_t)dst);
                            if constexpr (HOW == kRowsPast) store_past_caches(at, rows[i]);
                            else if constexpr (HOW == kRowsThrough) store_coherent(at, rows[i]);
                            else *at = rows[i];
                        }
                    }
                }
            }
        };
        const int how = D == 64 ? kRowsCached : p->new_rows;
        if (how == kRowsCached) append_rows(std::integral_constant<int, kRowsCached>());
        else if (F8 || how == kRowsThrough || row0 + n_s == p->rows) append_rows(std::integral_constant<int, kRowsThrough>());
        else append_rows(std::integral_constant<int, kRowsPast>());
    }

    const int t = t0 + l32;
    // normalises vectors vec and vec + 1 of O and writes them: the half-waves exchange what they hold of the two, 16 bytes
    // per lane and store
    auto finish = [&](int vec, const f32x4 &a, const f32x4 &b, float l) __attribute__((always_inline)) {
        const float inv = __builtin_amdgcn_rcpf(l);
        bf16x4 wa, wb;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            wa[e] = (__bf16)(a[e] * inv);
            wb[e] = (__bf16)(b[e] * inv);
        }
        uint2 y = __builtin_bit_cast(uint2, wa), z = __builtin_bit_cast(uint2, wb);
        asm volatile("s_nop 1\n\tv_permlane32_swap_b32 %0, %2\n\tv_permlane32_swap_b32 %1, %3\n\ts_nop 1" : "+v"(y.x), "+v"(y.y), "+v"(z.x), "+v"(z.y));
        if (valid && t < n_s) {
            uint16_t *orow = reinterpret_cast<uint16_t *>(p_out) + ((size_t)(row0 + t) * Hq + head) * D;
            global_u32x4_w *at = reinterpret_cast<global_u32x4_w *>((uintptr_t)(orow + (vec + half) * 8));
            const u32x4 row = {y.x, y.y, z.x, z.y};
            if (out_past_l2 != 0) store_past_caches(at, row);
            else *at = row;
        }
    };
    const float ltot = half_swap_sum(lsum);
    if (tl == 0) {                                       // a wavefront by itself
#pragma unroll
        for (int db = 0; db < DBLK; ++db)
#pragma unroll
            for (int q4 = 0; q4 < 4; q4 += 2) {
                f32x4 a, b;
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    a[e] = o[db][q4 * 4 + e];
                    b[e] = o[db][q4 * 4 + 4 + e];
                }
                finish(db * 4 + q4, a, b, ltot);
            }
        return;
    }
    // ---- the wavefronts of a team meet in LDS: each leaves its unnormalised O in its own regions (vector (db * 4 + q4) of lane l
    // at index (db * 4 + q4) * 64 + l: no bank conflicts), m and the row sum beside; then every wavefront finishes
    // some of the columns.  Wavefronts that had no step are not looked at.
    if (rank < parts) {
        f32x4 *mine = reinterpret_cast<f32x4 *>(my);
        static_assert(DBLK * 4 * 64 * 16 == 2 * TILE_BYTES, "an O fits a wavefront's regions");
        asm volatile("" ::: "memory");
#pragma unroll
        for (int db = 0; db < DBLK; ++db)
#pragma unroll
            for (int q4 = 0; q4 < 4; ++q4) {
                f32x4 y;
#pragma unroll
                for (int e = 0; e < 4; ++e) y[e] = o[db][q4 * 4 + e];
                mine[(db * 4 + q4) * 64 + lane] = y;
            }
        if (half == 0) { stat[wave][0][l32] = m; stat[wave][1][l32] = ltot; }
    }
    lds_barrier();
    // (whatever lies in LDS is read together, places past the last wavefront as the last one's: read one by one as it is used, it cost
    // teams of eight a round trip each, three times over: 286 short prompts of 40 heads 981.1 us, this way 977.3; ragged prompts over
    // codes 644.7, this way 642.6)
    float wgt[NW], sum[NW];
#pragma unroll
    for (int w = 0; w < NW; ++w) {
        const int from = team0 + min(w, parts - 1);
        wgt[w] = stat[from][0][l32];
        sum[w] = stat[from][1][l32];
    }
    float ms = wgt[0], l = 0.f;
#pragma unroll
    for (int w = 1; w < NW; ++w) ms = fmaxf(ms, wgt[w]);
#pragma unroll
    for (int w = 0; w < NW; ++w) {
        wgt[w] = __builtin_amdgcn_exp2f(wgt[w] - ms);
        if (w < parts) l = __builtin_fmaf(sum[w], wgt[w], l);
    }
    auto partial = [&](int i) -> float * { return p->scratch + ((size_t)(u * Hq + head) * splits + i) * (32 * D + 64); };
    // an item is 16 of the columns, two neighbouring vectors: 2 * DBLK of them
    for (int item = rank; item < 2 * DBLK; item += T) {
        const int vec = item * 2;                        // = db * 4 + q4 with q4 in {0, 2}
        f32x4 a = {0.f, 0.f, 0.f, 0.f}, b = a;
        auto add = [&](auto first_, auto count_) __attribute__((always_inline)) {
            constexpr int W0 = decltype(first_)::value, N = decltype(count_)::value;
            f32x4 xa[N], xb[N];
#pragma unroll
            for (int w = 0; w < N; ++w) {
                const f32x4 *src = reinterpret_cast<const f32x4 *>(smem + (team0 + min(W0 + w, parts - 1)) * (2 * TILE_BYTES)) + lane;
                xa[w] = src[vec * 64];
                xb[w] = src[(vec + 1) * 64];
            }
#pragma unroll
            for (int w = 0; w < N; ++w) asm volatile("" : "+v"(xa[w]), "+v"(xb[w]));
#pragma unroll
            for (int w = 0; w < N; ++w)
                if (W0 + w < parts) {
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        a[e] = __builtin_fmaf(xa[w][e], wgt[W0 + w], a[e]);
                        b[e] = __builtin_fmaf(xb[w][e], wgt[W0 + w], b[e]);
                    }
                }
        };
        typedef std::integral_constant<int, 2> N2;
        typedef std::integral_constant<int, 4> N4;
        if (T == 2) {
            add(R0(), N2());
        } else {
            add(R0(), N4());
            if constexpr (NW == 8)
                if (parts > 4) add(N4(), N4());
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
    for (int item = rank; item < 2 * DBLK; item += T) {
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
    const dim3 grid(p.attn_wgs + p.fetch_wgs + p.zero_wgs);
    const ShortWords w = short_pack(p);
    if constexpr (!F8) {
        if (p.carry != nullptr) {
            auto kernel = wavefronts == 8 ? attn_short_kernel<D, F8, 8, ShortCarry> : attn_short_kernel<D, F8, 4, ShortCarry>;
            static_assert(KernelArgs<decltype(kernel)>::last_offset() == kShortLead && kShortLead + sizeof(ShortCarry) <= 4096, "the kernel's arguments");
            ShortCarry a;
            static_cast<ShortArgs &>(a) = p;
            a.meta_dev = p.carry->dev;
            a.meta_vectors = (int32_t)((p.carry->len + 3) / 4);
            memcpy(a.meta, p.carry->host, (size_t)a.meta_vectors * 16);
            hipLaunchKernelGGL(kernel, dim3(grid.x + 1), dim3(64 * wavefronts), 0, stream, reinterpret_cast<const int32_t *>((uintptr_t)(p.bt - p.carry->dev)),
                               p.max_blocks, p.first_wg[0], p.first_wg[1], p.first_wg[2], w.first_units, p.attn_wgs, w.shape, p.splits_magic, p.hpx_magic,
                               p.hkx_magic, w.per_x, a);
            return hipGetLastError();
        }
    }
    auto kernel = wavefronts == 8 ? attn_short_kernel<D, F8, 8, ShortArgs> : attn_short_kernel<D, F8, 4, ShortArgs>;
    static_assert(KernelArgs<decltype(kernel)>::last_offset() == kShortLead, "where the kernel reads its structure");
    hipLaunchKernelGGL(kernel, grid, dim3(64 * wavefronts), 0, stream, p.bt, p.max_blocks, p.first_wg[0], p.first_wg[1], p.first_wg[2],
                       w.first_units, p.attn_wgs, w.shape, p.splits_magic, p.hpx_magic, p.hkx_magic, w.per_x, static_cast<const ShortArgs &>(p));
    return hipGetLastError();
}

}  // namespace

hipError_t tetri_launch_short(int head_dim, bool fp8_pool, const ShortParams &p, int wavefronts, hipStream_t stream)
{
    if (head_dim == 128) return fp8_pool ? launch<128, true>(p, wavefronts, stream) : launch<128, false>(p, wavefronts, stream);
    return fp8_pool ? launch<64, true>(p, wavefronts, stream) : launch<64, false>(p, wavefronts, stream);
}
