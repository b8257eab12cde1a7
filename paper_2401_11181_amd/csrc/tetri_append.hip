// Paged KV append for gfx950: copies the chunk's new K/V rows into their page slots.
// TetriInfer Sec. 2.1 (prefill generates the KV cache) and Sec. 3.4 (the cache is paged).
// Pure 16-byte vector copy, HBM-bound: no arithmetic, bit-exact by construction.
#include <hip/hip_ext.h>
#include <string.h>

#include "tetri_internal.h"

namespace {

constexpr int kPage = 16;

// grid: (chunk row, 0 = K / 1 = V).  One workgroup moves the Hkv*D elements of one token.
__global__ __launch_bounds__(256) void kv_append_kernel(AppendParams p)
{
    const int row = blockIdx.x;
    const int which = blockIdx.y;
    const int S = p.S;
    if (row >= p.cu[S]) return;                       // padding rows are never cached
    // segment of this row: largest s with cu[s] <= row (uniform across the workgroup)
    int lo = 0, hi = S - 1;
    while (lo < hi) {
        int mid = (lo + hi + 1) >> 1;
        if (p.cu[mid] <= row) lo = mid; else hi = mid - 1;
    }
    const int s = lo;
    const int pos = p.ctx[s] + (row - p.cu[s]);
    const int page = p.bt[(size_t)s * p.max_blocks + pos / kPage];
    const int slot = pos % kPage;
    const int ch = p.D / 8;                           // 16-byte vectors per head row
    const int per_row = p.Hkv * ch;
    const uint4 *src = reinterpret_cast<const uint4 *>(which ? p.v_new : p.k_new) + (size_t)row * per_row;
    uint4 *dst = reinterpret_cast<uint4 *>(p.pages)
                 + ((size_t)page * 2 + which) * p.Hkv * kPage * ch + (size_t)slot * ch;
    for (int x = threadIdx.x; x < per_row; x += 256) {
        const int head = x / ch, c = x - head * ch;
        dst[(size_t)head * kPage * ch + c] = src[x];
    }
}

// A batch's metadata from pinned host memory to the device.  The vectors cross the host link as ordinary loads: in
// stream order like any kernel, without the engine change of a copy (64 KB ahead of a chunk's launch: 13.8 us as a
// copy, 2 us this way; 4 KB costs the same both ways).  Bound by the link's round trip: four loads in flight per lane.
__global__ __launch_bounds__(256) void upload_kernel(const uint4 *__restrict__ src, uint4 *__restrict__ dst, int n)
{
    const int stride = gridDim.x * 256;
    for (int i = blockIdx.x * 256 + threadIdx.x; i < n; i += 4 * stride) {
        uint4 v[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) v[u] = src[min(i + u * stride, n - 1)];
#pragma unroll
        for (int u = 0; u < 4; ++u)
            if (i + u * stride < n) dst[i + u * stride] = v[u];
    }
}

// A small batch's metadata, at most N vectors, in the kernel's own arguments: the launch copies them, so the staging buffer is
// free again at once and no event has to say so.  Bound by one round trip to the arguments instead of two (the staging
// buffer behind them): a step of four small chunks 26.7 us through the staging buffer and its event, 24.8 this way.
template <int N> struct InlineUpload {
    uint4 *dst;
    int n;
    uint4 v[N];
};
template <int N> __global__ __launch_bounds__(N < 256 ? N : 256) void upload_inline_kernel(InlineUpload<N>)
{
    typedef __attribute__((address_space(4))) const InlineUpload<N> const_args;
    const const_args *p = (const const_args *)__builtin_amdgcn_kernarg_segment_ptr();
    const int i = threadIdx.x;
    if (i < p->n) {
        const auto *v = (__attribute__((address_space(4))) const uint32_t *)&p->v[i];
        p->dst[i] = make_uint4(v[0], v[1], v[2], v[3]);
    }
}

template <int N> hipError_t launch_inline(const int32_t *host, int32_t *dev, int64_t len, hipStream_t stream)
{
    InlineUpload<N> a;
    a.dst = reinterpret_cast<uint4 *>(dev);
    a.n = (int)((len + 3) / 4);
    memcpy(a.v, host, (size_t)a.n * 16);
    hipLaunchKernelGGL(upload_inline_kernel<N>, dim3(1), dim3(N), 0, stream, a);
    return hipGetLastError();
}

}  // namespace

hipError_t tetri_launch_upload_inline(const int32_t *host, int32_t *dev, int64_t len, hipStream_t stream)
{
    static_assert(kUploadInline == 4 * 224, "the larger size");
    return len <= 4 * 64 ? launch_inline<64>(host, dev, len, stream) : launch_inline<224>(host, dev, len, stream);
}

hipError_t tetri_launch_upload(const int32_t *pinned, int32_t *dev, int64_t len, hipStream_t stream, hipEvent_t done)
{
    const int n = (int)((len + 3) / 4);
    const int blocks = (n + 255) / 256;
    const dim3 grid(blocks < 256 ? blocks : 256);
    const uint4 *src = reinterpret_cast<const uint4 *>(pinned);
    uint4 *dst = reinterpret_cast<uint4 *>(dev);
    // (the event rides on the kernel's own completion signal: 0.9 us of a step of 26; recorded behind the kernel, with a packet of
    // its own in the queue, 2.8)
    if (done) hipExtLaunchKernelGGL(upload_kernel, grid, dim3(256), 0, stream, nullptr, done, 0, src, dst, n);
    else hipLaunchKernelGGL(upload_kernel, grid, dim3(256), 0, stream, src, dst, n);
    return hipGetLastError();
}

hipError_t tetri_launch_append(const tetri_ctx *, const AppendParams &p, int32_t chunk_rows, hipStream_t stream)
{
    dim3 grid(chunk_rows, 2), block(256);
    hipLaunchKernelGGL(kv_append_kernel, grid, block, 0, stream, p);
    return hipGetLastError();
}
