// Device pieces the attention kernels share: LDS-direct loads, transposing LDS reads, exchanges between the
// halves of a wavefront.
#pragma once

#include <math.h>

#include "pyr_internal.h"

namespace pyr {

// The lowest exponent reference of a row.  A row's reference is the largest logit of its first 32 keys; where those are all -inf it is this, a finite
// number, also times c, so that the row's sum is zero so far and not the NaN of -inf - -inf: the first key that can be seen outgrows it.  (Logits below
// it, finite ones, have no finite product with c.)
inline float lowest_reference(float c) { return -0x1.fffffcp127f / fmaxf(c, 1.0f); }

typedef __attribute__((ext_vector_type(4))) short s16x4;
typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2;
typedef __attribute__((address_space(3))) char* lptr_t;

// v_permlane32_swap(x, x): result 0 holds lanes 0..31 of x in both halves, result 1 holds
// lanes 32..63 of x in both halves; combining the two gives "own op other half" in every lane.
__device__ __forceinline__ float max_with_other_half(float x) {
    auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}
__device__ __forceinline__ float sum_with_other_half(float x) {
    auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}

// Transposing LDS read (ds_read_b64_tr_b16).  Inside every group of 16 lanes, lane j receives
// element (j & 3) of the 8-byte words addressed by lanes (j >> 2), 4 + (j >> 2), 8 + (j >> 2)
// and 12 + (j >> 2), in this order.
__device__ __forceinline__ s16x4 lds_read_tr(int lds_addr) {
    return __builtin_amdgcn_ds_read_tr16_b64_v4i16((s16x4 __attribute__((address_space(3)))*)(uintptr_t)lds_addr);
}

// 16 bytes per lane from global memory straight into LDS: lane l's data lands at
// lds + 16*l (lds wave-uniform), its source is base (wave-uniform) + voff (per lane).
// Written in assembly on purpose: the compiler would make every later LDS read wait for ALL
// outstanding loads of this kind (it cannot tell the ring slots apart).  The kernels order
// these loads themselves: s_waitcnt vmcnt and a barrier before a slot is read.
__device__ __forceinline__ void lds_dma16(const char* base_, uint32_t voff, uint32_t lds_addr) {
    const uint32_t m0 = (uint32_t)__builtin_amdgcn_readfirstlane((int)lds_addr);
    const uint64_t b64 = (uint64_t)(uintptr_t)base_;         // wave-uniform by construction: keep it in scalar registers
    const uint32_t b_lo = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)b64);          // (the builtin returns a signed int:
    const uint32_t b_hi = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(b64 >> 32));  //  widen it unsigned)
    const char* base = (const char*)(uintptr_t)(((uint64_t)b_hi << 32) | (uint64_t)b_lo);
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2"
                 :: "s"(m0), "v"(voff), "s"(base) : "memory", "m0");
}

__device__ __forceinline__ uint32_t pack_bf16(float a, float b) {      // v_cvt_pk_bf16_f32
    bf16x2 v;
    v[0] = (__bf16)a;
    v[1] = (__bf16)b;
    return __builtin_bit_cast(uint32_t, v);
}

}  // namespace pyr
