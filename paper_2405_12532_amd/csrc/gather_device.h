// Device code shared by the row gathers (gather.hip) and the selection that gathers its own rows (select.hip).
#pragma once

#include "pyr_internal.h"

namespace pyr {

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

}  // namespace pyr
