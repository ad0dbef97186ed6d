// Row gather: dst[j, :] = src[kept_idx[j], :]   (Algorithm 1, Gather(KV, index); the same
// kernel compacts the hidden rows that enter the next layer).
//
// Pure data movement, bound by HBM bandwidth: 2 * n_kept * row_bytes bytes move per source.
// One wavefront owns one output row; its 64 lanes move 16 bytes each per access, so a row is
// read and written in fully coalesced 1 KiB pieces, and up to kUnroll loads per lane are issued
// before the first store to keep enough bytes in flight per compute unit.  The grid has a
// wavefront per row (the stride loop only matters beyond 2^31 workgroups): workgroups start in
// index order, so the rows in flight at any moment are neighbours in memory, which HBM serves
// about a tenth faster than the far-apart rows a short grid with a stride loop has in flight
// (measured on an 8 KB-row copy of 1 GiB: 6.1-6.3 TB/s read + write against 5.5; two wavefronts
// per workgroup were the best of 1, 2, 4, 8, 16).
#include "pyr_internal.h"

namespace pyr {
namespace {

constexpr int kThreads = 128;
constexpr int kWavesPerBlock = kThreads / 64;
constexpr int64_t kMaxBlocks = 0x7fffffff;      // gridDim.x limit; beyond it the kernels' stride loops take over

// One row by the calling wavefront: 16 bytes a lane, up to kUnroll loads per lane issued before the first store.
__device__ __forceinline__ void copy_row(const u32x4* __restrict__ src, u32x4* __restrict__ dst, int32_t chunks_per_row, int lane) {
    constexpr int kUnroll = 8;
    for (int c0 = 0; c0 < chunks_per_row; c0 += 64 * kUnroll) {
        u32x4 buf[kUnroll];
#pragma unroll
        for (int u = 0; u < kUnroll; ++u) {
            const int c = c0 + u * 64 + lane;
            if (c < chunks_per_row) buf[u] = __builtin_nontemporal_load(src + c);
        }
#pragma unroll
        for (int u = 0; u < kUnroll; ++u) {
            const int c = c0 + u * 64 + lane;
            if (c < chunks_per_row) __builtin_nontemporal_store(buf[u], dst + c);
        }
    }
}

__global__ __launch_bounds__(kThreads) void gather_rows_kernel(
    const u32x4* __restrict__ src0, u32x4* __restrict__ dst0,
    const u32x4* __restrict__ src1, u32x4* __restrict__ dst1,
    const int32_t* __restrict__ kept_idx, int64_t n_rows, int32_t chunks_per_row, int32_t blocks) {
    const int lane = threadIdx.x & 63;
    const int wave = threadIdx.x >> 6;
    const u32x4* __restrict__ src = blockIdx.y == 0 ? src0 : src1;
    u32x4* __restrict__ dst = blockIdx.y == 0 ? dst0 : dst1;
    const int64_t wave_stride = (int64_t)blocks * kWavesPerBlock;
    for (int64_t j = (int64_t)blockIdx.x * kWavesPerBlock + wave; j < n_rows; j += wave_stride) {
        copy_row(src + (int64_t)kept_idx[j] * chunks_per_row, dst + j * chunks_per_row, chunks_per_row, lane);
    }
}

// Several sources gathered with one index list in ONE launch (K, V, the hidden rows, the position ids): at small
// batch every launch costs about as much as the rows it moves (Appendix A.1 is about exactly this regime).
// (Arguments of 112 bytes and less, the grid's size among them, which would bring the implicit ones along: 0.7 us less host time a launch.)
static_assert(sizeof(GatherSources) + sizeof(int32_t*) + sizeof(int64_t) + sizeof(int32_t) <= 112, "short arguments");
// blockIdx.y picks the source; the last y, if pos is given, gathers the 4-byte position ids.
__global__ __launch_bounds__(kThreads) void gather_multi_kernel(GatherSources g, const int32_t* __restrict__ kept_idx,
                                                                int64_t n_rows, int32_t blocks) {
    const int lane = threadIdx.x & 63;
    const int wave = threadIdx.x >> 6;
    const int y = blockIdx.y;
    if (y >= g.n) {                    // position ids
        for (int64_t j = (int64_t)blockIdx.x * kThreads + threadIdx.x; j < n_rows; j += (int64_t)blocks * kThreads)
            g.pos_out[j] = g.pos[kept_idx[j]];
        return;
    }
    const u32x4* __restrict__ src = y == 0 ? g.src[0] : y == 1 ? g.src[1] : g.src[2];
    u32x4* __restrict__ dst = y == 0 ? g.dst[0] : y == 1 ? g.dst[1] : g.dst[2];
    const int32_t chunks_per_row = y == 0 ? g.chunks[0] : y == 1 ? g.chunks[1] : g.chunks[2];
    const int64_t wave_stride = (int64_t)blocks * kWavesPerBlock;
    for (int64_t j = (int64_t)blockIdx.x * kWavesPerBlock + wave; j < n_rows; j += wave_stride) {
        copy_row(src + (int64_t)kept_idx[j] * chunks_per_row, dst + j * chunks_per_row, chunks_per_row, lane);
    }
}

// Position ids of the kept tokens (Appendix A.2: the survivors keep the position encodings
// they had; the ids are gathered with the same index as K and V): pos_out[j] = pos[kept_idx[j]].
__global__ __launch_bounds__(256) void gather_positions_kernel(const int32_t* __restrict__ pos,
                                                               const int32_t* __restrict__ kept_idx, int64_t n_kept,
                                                               int32_t* __restrict__ pos_out) {
    for (int64_t j = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; j < n_kept; j += (int64_t)gridDim.x * blockDim.x)
        pos_out[j] = pos[kept_idx[j]];
}

}  // namespace

int launch_gather_positions(const int32_t* pos, const int32_t* kept_idx, int64_t n_kept, int32_t* pos_out,
                            hipStream_t stream) {
    if (n_kept == 0) return PYR_OK;
    int64_t blocks = (n_kept + 255) / 256;
    if (blocks > 256 * 8) blocks = 256 * 8;
    hipLaunchKernelGGL(gather_positions_kernel, dim3((unsigned)blocks), dim3(256), 0, stream, pos, kept_idx, n_kept, pos_out);
    return check_launch();
}

int launch_gather_multi(const GatherSources& g, const int32_t* kept_idx, int64_t n_kept, hipStream_t stream) {
    if (n_kept == 0 || (g.n == 0 && g.pos == nullptr)) return PYR_OK;
    int64_t blocks = (n_kept + kWavesPerBlock - 1) / kWavesPerBlock;
    if (blocks > kMaxBlocks) blocks = kMaxBlocks;
    dim3 grid((unsigned)blocks, (unsigned)(g.n + (g.pos != nullptr ? 1 : 0)), 1);
    hipLaunchKernelGGL(gather_multi_kernel, grid, dim3(kThreads), 0, stream, g, kept_idx, n_kept, (int32_t)blocks);
    return check_launch();
}

int launch_gather(const void* src0, void* dst0, const void* src1, void* dst1, size_t row_bytes,
                  const int32_t* kept_idx, int64_t n_kept, hipStream_t stream) {
    if (n_kept == 0) return PYR_OK;
    const int32_t chunks = (int32_t)(row_bytes / 16);
    int64_t blocks = (n_kept + kWavesPerBlock - 1) / kWavesPerBlock;
    if (blocks > kMaxBlocks) blocks = kMaxBlocks;
    dim3 grid((unsigned)blocks, src1 != nullptr ? 2 : 1, 1);
    hipLaunchKernelGGL(gather_rows_kernel, grid, dim3(kThreads), 0, stream,
                       (const u32x4*)src0, (u32x4*)dst0, (const u32x4*)src1, (u32x4*)dst1,
                       kept_idx, n_kept, chunks, (int32_t)blocks);
    return check_launch();
}

}  // namespace pyr
