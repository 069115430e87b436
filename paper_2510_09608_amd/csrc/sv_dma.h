// Direct global -> LDS loads and stores past the L2, shared by the attention kernels.
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

// A store that goes through the L2 to memory (device scope) instead of waiting there as a dirty line.  A launch ends with the
// write-back of the eight L2s: of what its last workgroups stored, at least, nothing has left by itself, and the next launch
// starts that much later; and a launch with no dirty line at all ends sooner than one with a few.  So it counts for launches of
// microseconds that write to their end, and there only if ALL their stores are of this kind.
// Chunk attention with its merge, 256 queries of 28 / 4 heads, on 1376 keys 21.1 -> 19.9 us, on 5376 30.7 -> 29.7 (its last
// partial result was stored after 25.4 us, the merge began after 28.4); decode, 28 / 4 heads, 5392 tokens, 6.10 -> 6.00.
// Not used where it gains nothing: the moves of whole caches (76 us at head_dim 128 either way; 12 layers of 64 11.6 and 17), the
// storing of new tokens, fp32 chunk attention by fp32 instructions (256 on 5392, 4 layers and their decode, 788 us, with it 793), merges of
// fp32 chunks.
// (16 bytes as assembly, which has no builtin; the s_nop keeps the compiler, which does not know of the store, from overwriting its
// registers while they are read: a vector instruction that does so has to stay two wait states behind a store of more than 8 bytes.)
template <typename V>
__device__ __forceinline__ void store_through(void* p, const V& v) {
  static_assert(sizeof(V) == 2 || sizeof(V) == 4 || sizeof(V) == 8 || sizeof(V) == 16, "one store");
  if constexpr (sizeof(V) == 16) {
    typedef __attribute__((__vector_size__(4 * sizeof(unsigned)))) unsigned u32x4;
    const u32x4 x = __builtin_bit_cast(u32x4, v);
    asm volatile("global_store_dwordx4 %0, %1, off sc1\n\ts_nop 1" ::"v"(p), "v"(x) : "memory");
  } else if constexpr (sizeof(V) == 8) {
    __hip_atomic_store((unsigned long long*)p, __builtin_bit_cast(unsigned long long, v), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  } else if constexpr (sizeof(V) == 4) {
    __hip_atomic_store((uint32_t*)p, __builtin_bit_cast(uint32_t, v), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  } else {
    __hip_atomic_store((unsigned short*)p, __builtin_bit_cast(unsigned short, v), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
}

}  // namespace sv
