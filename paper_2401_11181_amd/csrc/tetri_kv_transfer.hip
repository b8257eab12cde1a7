// KV export / import for gfx950: the data plane of the dispatcher (TetriInfer Sec. 3.3.4).  Export
// gathers token ranges of requests out of the paged pool (Sec. 3.4) into a dense transfer buffer,
// request after request as [2 (K, V)][Hkv][n_r][D]; import scatters such a buffer into the pages of
// the receiving pool.  Pure 16-byte vector copies, HBM-bound, bit-exact by construction.
//
// Work split: a workgroup moves one tile of consecutive tokens of one request (4 KB per slab: 16 tokens
// for head dimension 128, 32 for 64) for a run of (K / V, head) slabs; each lane owns 16 bytes of one
// token and walks the slabs, four loads in flight.  On the pool side 16 consecutive tokens of a slab are
// one contiguous 16 * D * 2 bytes of a page, on the buffer side the tile is contiguous, so both sides
// are touched in whole cache lines.  The page of a token is looked up once and reused for all slabs.
// The data is used once: loads and stores are non-temporal.
#include "attn_common.h"

namespace {

using namespace tetri_dev;

constexpr int kThreads = 256;
constexpr int kTileBytes = kThreads * 16;     // one slab of a tile

// A workgroup's tile: its request, where that begins in the buffer, how many tokens it has, its first token's position and the
// tile's first token inside the request.
struct Tile {
    int r, c0, n, first, j0;
};

// Finds tile `tile` when the tiles (TILE tokens each) of all requests are numbered request after request (request r has
// ceil(n_r / TILE) of them).  Wavefront-wide: 64 requests per step, prefix sum by shuffles, over as many lanes as there are
// requests.  Every wavefront computes the same result.  False when the grid's upper bound overshoots the real number of tiles.
// A short transfer is bound by this chain: what is known of the request travels in its lane, so that nothing about it is
// read a second time (512 tokens of 40 heads, export and import: 12.25 us when begin, end and first token were read again and
// the arguments first, now 11.4).
template <int TILE>
__device__ inline bool find_tile(const int32_t *cu, const int32_t *first, int R, int tile, int lane, Tile &x)
{
    int base = 0;
    for (int r0 = 0; r0 < R; r0 += 64) {
        const int r = r0 + lane, m = min(R - r0, 64);
        int begin = 0, n = 0, f = 0;
        if (lane < m) {
            begin = cu[r];
            n = cu[r + 1] - begin;
            if (first) f = first[r];
        }
        const int t = (n + TILE - 1) / TILE;
        int incl = t;
#pragma unroll 1
        for (int d = 1; d < m; d <<= 1) {
            const int up = __shfl_up(incl, d);
            if (lane >= d) incl += up;
        }
        incl += base;
        const unsigned long long hit = __ballot(tile < incl && tile >= incl - t);
        if (hit) {
            const int src = __builtin_ctzll(hit);
            x.r = r0 + src;
            x.c0 = __builtin_amdgcn_readlane(begin, src);
            x.n = __builtin_amdgcn_readlane(n, src);
            x.first = max(__builtin_amdgcn_readlane(f, src), 0);
            x.j0 = (tile - __builtin_amdgcn_readlane(incl - t, src)) * TILE;
            return true;
        }
        base = __builtin_amdgcn_readlane(incl, 63);      // (only a full step has a next one)
    }
    return false;
}

// Workgroup -> tile and run of slabs.  Four tiles take their first run, then their second one, and so on, then come the
// next four: what is under way at a time (2048 workgroups) are then about a dozen pages of the pool, each a contiguous
// 2 * Hkv * 4 KB, and on the buffer's side a few hundred KB of every slab.  Moving one slab of all tiles first touches
// two thousand pages at a time (16 requests of 51 to 516 tokens: 61 us, this way 56); all slabs of a single tile
// first spreads the buffer's side as thin (a request of 12485 tokens: 364 us, this way 354).
constexpr int kTilesAbreast = 4;
__device__ inline void tile_of(int slab_groups, uint32_t groups_magic, int bid, int &tile, int &group)
{
    const int run = bid / kTilesAbreast, block = magic_div(run, groups_magic);
    group = run - block * slab_groups;
    tile = block * kTilesAbreast + bid % kTilesAbreast;
}

// grid: (upper bound of the number of tiles, rounded up to kTilesAbreast) x runs of slabs.  (The first 56 bytes of the
// arguments are in registers when a wavefront starts: all that the look-ups need.)
template <int D, bool TO_POOL>
__global__ __launch_bounds__(kThreads) void kv_transfer_kernel(const int32_t *cu, const int32_t *first, const int32_t *bt, uint16_t *pool, int R,
                                                               int max_blocks, int Hkv, int slab_groups, uint32_t groups_magic, int slabs_per_wg,
                                                               uint16_t *buf)
{
    constexpr int LPR = D / 8;                 // lanes that move one token's D bf16 of one slab
    constexpr int TILE = kThreads / LPR;       // tokens per workgroup
    const int tid = threadIdx.x;
    int tile, group;
    tile_of(slab_groups, groups_magic, blockIdx.x, tile, group);
    Tile x;
    if (!find_tile<TILE>(cu, first, R, tile, tid & 63, x)) return;
    const int j = x.j0 + tid / LPR;
    if (j >= x.n) return;                        // no barrier below: lanes past the request's end just leave
    const int col = (tid % LPR) * 8;
    const int slabs = 2 * Hkv;
    const int pos = x.first + j;
    // the block-table index is clamped: a range the table cannot describe never forms an address outside it
    const int page = bt[(size_t)x.r * max_blocks + min(pos / kPage, max_blocks - 1)];
    // slab = kv * Hkv + head in both layouts: from one slab to the next both sides advance by a fixed step
    const int slab0 = group * slabs_per_wg;
    int left = min(slabs, slab0 + slabs_per_wg) - slab0;
    const size_t pool_step = (size_t)kPage * D, buf_step = (size_t)x.n * D;
    uint16_t *in_pool = pool + ((size_t)page * slabs + slab0) * pool_step + (size_t)(pos % kPage) * D + col;
    uint16_t *in_buf = buf + (size_t)slabs * D * x.c0 + slab0 * buf_step + (size_t)j * D + col;
    const uint16_t *src = TO_POOL ? in_buf : in_pool;
    uint16_t *dst = TO_POOL ? in_pool : in_buf;
    const size_t src_step = TO_POOL ? buf_step : pool_step, dst_step = TO_POOL ? pool_step : buf_step;
    auto ld = [&]() {
        const u32x4 v = __builtin_nontemporal_load(reinterpret_cast<const u32x4 *>(src));
        src += src_step;
        return v;
    };
    auto st = [&](u32x4 v) {
        __builtin_nontemporal_store(v, reinterpret_cast<u32x4 *>(dst));
        dst += dst_step;
    };
#pragma unroll 1
    for (; left >= 4; left -= 4) {
        const u32x4 v0 = ld(), v1 = ld(), v2 = ld(), v3 = ld();
        st(v0), st(v1), st(v2), st(v3);
    }
    if (left >= 2) {
        const u32x4 v0 = ld(), v1 = ld();
        st(v0), st(v1);
        left -= 2;
    }
    if (left) st(ld());
}

// Export with quantisation: the 16-bit pool is gathered into a dense buffer of FP8 E4M3 codes, the K
// half of every request's block under the K scale, the V half under the V scale (this build's extension:
// half the bytes on the link between the instances).  A code is fl32(x * inv_scale) clamped to +-448 and
// rounded to nearest even by v_cvt_pk_fp8_f32.  Same work split as the copy kernel: a lane reads 16 bytes (8 values) and
// writes 8 codes.  (16 values per lane, two loads 32 bytes apart between lanes and one 16-byte store: 10 % slower.)
template <int D>
__global__ __launch_bounds__(kThreads) void kv_export_fp8_kernel(const int32_t *cu, const int32_t *first, const int32_t *bt, const uint16_t *pool, int R,
                                                                 int max_blocks, int Hkv, int slab_groups, uint32_t groups_magic, int slabs_per_wg,
                                                                 uint8_t *buf, float k_inv, float v_inv)
{
    constexpr int LPR = D / 8, TILE = kThreads / LPR;
    const int tid = threadIdx.x;
    int tile, group;
    tile_of(slab_groups, groups_magic, blockIdx.x, tile, group);
    Tile x;
    if (!find_tile<TILE>(cu, first, R, tile, tid & 63, x)) return;
    const int j = x.j0 + tid / LPR;
    if (j >= x.n) return;
    const int col = (tid % LPR) * 8;
    const int slabs = 2 * Hkv;
    const int pos = x.first + j;
    const int page = bt[(size_t)x.r * max_blocks + min(pos / kPage, max_blocks - 1)];
    int slab = group * slabs_per_wg;
    const int slab_end = min(slabs, slab + slabs_per_wg);
    const size_t pool_step = (size_t)kPage * D, buf_step = (size_t)x.n * D;
    const uint16_t *src = pool + ((size_t)page * slabs + slab) * pool_step + (size_t)(pos % kPage) * D + col;
    uint8_t *dst = buf + (size_t)slabs * D * x.c0 + slab * buf_step + (size_t)j * D + col;
    auto ld = [&]() {
        const u32x4 v = __builtin_nontemporal_load(reinterpret_cast<const u32x4 *>(src));
        src += pool_step;
        return v;
    };
    auto st = [&](const u32x4 &v) {
        const uint2 x = bf16_to_codes(v, slab < Hkv ? k_inv : v_inv);
        __builtin_nontemporal_store(u32x2{x.x, x.y}, reinterpret_cast<u32x2 *>(dst));
        dst += buf_step;
        ++slab;
    };
#pragma unroll 1
    while (slab + 4 <= slab_end) {
        const u32x4 v0 = ld(), v1 = ld(), v2 = ld(), v3 = ld();
        st(v0), st(v1), st(v2), st(v3);
    }
#pragma unroll 1
    while (slab < slab_end) st(ld());
}

}  // namespace

hipError_t tetri_launch_kv_export_fp8(const tetri_ctx *h, const TransferParams &p, int32_t tiles, hipStream_t stream)
{
    const dim3 grid((unsigned)((tiles + kTilesAbreast - 1) / kTilesAbreast * kTilesAbreast * p.slab_groups)), block(kThreads);
    const int d = h->cfg.head_dim;
    if (d != 128 && d != 64) return hipErrorInvalidValue;
    auto kernel = d == 128 ? kv_export_fp8_kernel<128> : kv_export_fp8_kernel<64>;
    hipLaunchKernelGGL(kernel, grid, block, 0, stream, p.cu, p.first, p.bt, p.pool, p.R, p.max_blocks, p.Hkv, p.slab_groups, p.groups_magic,
                       p.slabs_per_wg, reinterpret_cast<uint8_t *>(p.buf), p.k_inv, p.v_inv);
    return hipGetLastError();
}

// `row_units`: 16-bit units of one row of the pool (head_dim for a 16-bit pool, head_dim / 2 for FP8 codes,
// which the copy moves as opaque bytes)
hipError_t tetri_launch_kv_transfer(const tetri_ctx *, const TransferParams &p, int32_t row_units, int32_t tiles,
                                    bool to_pool, hipStream_t stream)
{
    const dim3 grid((unsigned)((tiles + kTilesAbreast - 1) / kTilesAbreast * kTilesAbreast * p.slab_groups)), block(kThreads);
    const int d = row_units;
    if (d != 128 && d != 64 && d != 32) return hipErrorInvalidValue;
    auto kernel = d == 128 ? (to_pool ? kv_transfer_kernel<128, true> : kv_transfer_kernel<128, false>)
                : d == 64  ? (to_pool ? kv_transfer_kernel<64, true> : kv_transfer_kernel<64, false>)
                           : (to_pool ? kv_transfer_kernel<32, true> : kv_transfer_kernel<32, false>);
    hipLaunchKernelGGL(kernel, grid, block, 0, stream, p.cu, p.first, p.bt, p.pool, p.R, p.max_blocks, p.Hkv, p.slab_groups, p.groups_magic,
                       p.slabs_per_wg, p.buf);
    return hipGetLastError();
}
