// Helpers of the kernels that run one search per wavefront.
#pragma once

#include "dlm_common.h"

namespace dlm {

// Orders the wave's LDS accesses around it in the compiler's view; the LDS
// itself serves one wave's instructions in issue order.
__device__ __forceinline__ void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// a uniform 32-bit value in a scalar register of its own
__device__ __forceinline__ uint32_t own_u32(uint32_t x) {
  asm volatile("" : "+s"(x));
  return x;
}

__device__ __forceinline__ uint64_t own_u64(uint64_t x) {
  asm volatile("" : "+s"(x));
  return x;
}

// The twenty Philox4x32-10 round keys (the seed's two words bumped by the
// Weyl constants), computed once and held in vector registers: in scalar
// registers, the scarce file here, they would spill, and recomputing them
// per call costs twenty scalar adds.
struct RoundKeys {
  uint32_t k[20];
};

__device__ __forceinline__ uint32_t to_vgpr(uint32_t x) {
  uint32_t y;
  asm volatile("v_mov_b32 %0, %1" : "=v"(y) : "s"(x));
  return y;
}

__device__ __forceinline__ RoundKeys round_keys(Key key) {
  RoundKeys rk;
  uint32_t k0 = key.k0, k1 = key.k1;
#pragma unroll
  for (int r = 0; r < 10; ++r) {
    rk.k[2 * r] = to_vgpr(k0);
    rk.k[2 * r + 1] = to_vgpr(k1);
    k0 += 0x9E3779B9u;
    k1 += 0xBB67AE85u;
  }
  return rk;
}

// one v_bitop3_b32
__device__ __forceinline__ uint32_t xor3(uint32_t a, uint32_t b, uint32_t c) {
  return (uint32_t)__builtin_amdgcn_bitop3_b32((int)a, (int)b, (int)c, 0x96);
}

// Philox4x32-10 word 0 (the same function as philox_w0) from precomputed round keys
__device__ __forceinline__ uint32_t philox_w0_rk(uint32_t x0, uint32_t x1, uint32_t x2, uint32_t x3,
                                                 const RoundKeys& rk) {
#pragma unroll
  for (int r = 0; r < 10; ++r) {
    const uint64_t p0 = (uint64_t)0xD2511F53u * x0, p1 = (uint64_t)0xCD9E8D57u * x2;
    const uint32_t y0 = xor3((uint32_t)(p1 >> 32), x1, rk.k[2 * r]), y2 = xor3((uint32_t)(p0 >> 32), x3, rk.k[2 * r + 1]);
    x1 = (uint32_t)p1;
    x3 = (uint32_t)p0;
    x0 = y0;
    x2 = y2;
  }
  return x0;
}

__device__ __forceinline__ uint32_t rfl(uint32_t x) {
  return (uint32_t)__builtin_amdgcn_readfirstlane((int)x);
}

// The kernel's arguments (its first parameter, an Args block), read again where
// they are needed late and rarely: output pointers would otherwise hold (and
// spill) scalar registers all along.
template <class Args>
__device__ __forceinline__ const Args* late_args() {
  uint64_t p = (uint64_t)__builtin_amdgcn_kernarg_segment_ptr();
  asm volatile("" : "+s"(p));
  return (const Args*)p;
}

}  // namespace dlm
