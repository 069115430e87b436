// Direct global -> LDS loads, shared by the attention kernels.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace sv {

// 16 bytes per lane from global memory straight into LDS: lane L's bytes land at lds_dst + 16 L (lds_dst is
// uniform over the wavefront and travels in M0).  Written as assembly on purpose: the compiler then does not
// see a pending write to LDS and inserts no wait for ALL outstanding direct loads in front of later LDS
// reads; the kernel waits itself (vmcnt, and a workgroup barrier where other wavefronts read it) before a tile is first read.
// (M0 is named as clobbered on purpose: nothing else in these kernels uses it, and the compiler must not assume it
// survives; clang notes that M0 is a reserved register, which is the point.)
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"
__device__ __forceinline__ void dma16(const void* base, uint32_t lane_off, char* lds_dst) {
  // base (uniform) travels in a scalar register pair, the lane's byte offset in one VGPR
  const uint32_t l = __builtin_amdgcn_readfirstlane((uint32_t)(uintptr_t)(__attribute__((address_space(3))) char*)lds_dst);
  const uint64_t b = (uint64_t)base;
  // (the builtin returns a signed int: convert each half through uint32_t, or the low half sign-extends)
  const uint64_t bu = ((uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((uint32_t)(b >> 32)) << 32) |
                      (uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((uint32_t)b);
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" ::"s"(l), "v"(lane_off), "s"(bu)
               : "memory", "m0");
}
__device__ __forceinline__ uint32_t lds_addr(char* p) { return (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char*)p; }
// A pointer that is the same in all lanes, in scalar registers.
__device__ __forceinline__ const char* uniform_ptr(const char* p) {
  const uint64_t b = (uint64_t)p;
  const uint32_t lo = (uint32_t)__builtin_amdgcn_readfirstlane((uint32_t)b), hi = (uint32_t)__builtin_amdgcn_readfirstlane((uint32_t)(b >> 32));
  return (const char*)((uint64_t)hi << 32 | lo);
}
// ... with the base known to be uniform and the place in LDS as its address (lds_addr), which costs no scalar instructions per
// call.  NT: non-temporal.
template <bool NT = false>
__device__ __forceinline__ void dma16(const void* base, uint32_t lane_off, uint32_t lds) {
  if constexpr (NT)
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2 nt" ::"s"(lds), "v"(lane_off), "s"(base) : "memory", "m0");
  else
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" ::"s"(lds), "v"(lane_off), "s"(base) : "memory", "m0");
}
// Two of them, 1 KB further on in memory and in LDS (the instruction's offset counts for both).
template <bool NT>
__device__ __forceinline__ void dma16x2(const void* base, uint32_t lane_off, uint32_t lds) {
  if constexpr (NT)
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2 nt\n\tglobal_load_lds_dwordx4 %1, %2 offset:1024 nt" ::"s"(
                     lds), "v"(lane_off), "s"(base) : "memory", "m0");
  else
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2\n\tglobal_load_lds_dwordx4 %1, %2 offset:1024" ::"s"(
                     lds), "v"(lane_off), "s"(base) : "memory", "m0");
}
#pragma clang diagnostic pop

}  // namespace sv
