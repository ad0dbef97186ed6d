// Device pieces the walks over K share: LDS-direct loads that the wavefront orders itself.
#pragma once

#include "pyr_internal.h"

namespace pyr {

typedef __attribute__((address_space(3))) char* lptr_t;
typedef __attribute__((address_space(3))) float* lfloat_t;

// 64 lanes x 16 bytes (or x 4 bytes) from base + voff[lane] to LDS at lds_addr + 16 (4) * lane.
// Assembly because the wavefront orders these loads itself with s_waitcnt vmcnt(N); they
// retire in the order issued.
__device__ __forceinline__ void lds_dma(const char* base_, uint32_t voff, uint32_t lds_addr, bool dword) {
    const uint32_t m0 = (uint32_t)__builtin_amdgcn_readfirstlane((int)lds_addr);
    const uint64_t b64 = (uint64_t)(uintptr_t)base_;         // wave-uniform by construction: keep it in scalar registers
    const uint32_t b_lo = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)b64);          // (the builtin returns a signed int:
    const uint32_t b_hi = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(b64 >> 32));  //  widen it unsigned)
    const char* base = (const char*)(uintptr_t)(((uint64_t)b_hi << 32) | (uint64_t)b_lo);
    if (dword)
        asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dword %1, %2" ::"s"(m0), "v"(voff), "s"(base) : "memory", "m0");
    else
        asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" ::"s"(m0), "v"(voff), "s"(base) : "memory", "m0");
}

template <int N>
__device__ __forceinline__ void wait_loads() {      // until at most N of this wavefront's loads are outstanding
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
}
__device__ __forceinline__ void wait_lds() { asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory"); }

}  // namespace pyr
