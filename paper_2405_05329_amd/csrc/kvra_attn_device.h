// Device helpers the two attention kernels share (not installed).
#ifndef KVRA_ATTN_DEVICE_H
#define KVRA_ATTN_DEVICE_H

#include "kvra_internal.h"

namespace kvra {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef short s16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) s16x4 lds_s16x4;
typedef __attribute__((address_space(3))) bf16x8 lds_bf16x8;
typedef __attribute__((address_space(3))) void lds_void;

// Exponent reference of a row before its first visible key: the lowest finite number, so that no finite score lies below
// it and a merge that takes the larger of two references always takes that of a row that has met a key.
constexpr float kNoKeyYet = -3.402823466e38f;

// A store that is visible to the whole device once it has been acknowledged, and a load that sees such
// stores (they go past whatever a non-coherent cache level holds).
__device__ __forceinline__ void store_coherent(float* p, float v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ float load_coherent(const float* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// The value held by lane ^ 32, and by lane ^ 16.
__device__ __forceinline__ float other_half(float x) {
  auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return __uint_as_float((threadIdx.x & 32) ? r[0] : r[1]);
}
__device__ __forceinline__ float other_row(float x) {
  auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return __uint_as_float((threadIdx.x & 16) ? r[0] : r[1]);
}

// 64 lanes x 16 bytes from global memory straight into 1 KiB of consecutive LDS starting at
// lds_byte_addr (lane l lands at +16 l).  Global address = base of the buffer resource + per-lane byte offset; a lane whose
// offset lies beyond the resource's size gets zeros, so a tile that straddles the end of what may be read, or lies
// beyond it, needs no other care.
// Written as inline assembly on purpose: the compiler guards every LDS-direct load it knows about
// with a full vmcnt(0) wait (it cannot tell the ring slots apart), which would serialise the
// prefetch; here completion is awaited by hand, once per block, with s_waitcnt vmcnt(n).
// Wait states: a memory instruction may read a scalar register that a vector instruction wrote (the resource comes from
// v_readfirstlane, or from the lanes it was spilled to) five states later at the earliest, and the compiler, which does not
// know that a memory instruction stands in here, keeps no such distance.  s_mov (one) and s_nop 3 (four) make it up whatever
// is scheduled in front of the block.
__device__ __forceinline__ void lds_dma16(u32x4 resource, unsigned lane_byte_off, unsigned lds_byte_addr) {
  asm volatile("s_mov_b32 m0, %2\n\ts_nop 3\n\tbuffer_load_dwordx4 %0, %1, 0 offen lds"
               :
               : "v"(lane_byte_off), "s"(resource), "s"(lds_byte_addr)
               : "memory", "m0");
}

}  // namespace kvra

#endif
