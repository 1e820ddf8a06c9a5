// What the product kernels share: DMA into LDS, hand-written waits.
#pragma once
#include <type_traits>

#include "common.h"

namespace bt {

#define BT_AS1 __attribute__((address_space(1)))
#define BT_AS3 __attribute__((address_space(3)))

// One 16-byte-per-lane DMA from global memory straight into LDS: lane i's 16 bytes land at
// lds_base + 16*i (lds_base is wave-uniform and travels in M0).  Issued through inline assembly so
// that the compiler does not serialise later LDS reads behind every outstanding DMA; completion is
// tracked by hand with s_waitcnt vmcnt + s_barrier.  The s_nop covers the M0-write -> LDS-DMA hazard.
__device__ __forceinline__ void dma16(const void* gptr, uint32_t lds_base) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off" ::"s"(lds_base), "v"(gptr)
               : "memory", "m0");
}
// The same with the address split into a wave-uniform base and a 32-bit byte offset per lane; the LDS target is lds + OFF.
template <int OFF>
__device__ __forceinline__ void dma16_sv(const void* sbase, uint32_t voff, uint32_t lds) {
  asm volatile("s_add_u32 m0, %0, %3\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" ::"s"(lds), "v"(voff), "s"(sbase), "n"(OFF)
               : "memory", "m0", "scc");
}
__device__ __forceinline__ uint32_t lds_addr(const void* p) {
  return (uint32_t)(uintptr_t)(BT_AS3 const void*)p;
}

// s_waitcnt vmcnt(n), other counters untouched (gfx9 encoding: vmcnt = [15:14|3:0]).
template <int N>
__device__ __forceinline__ void wait_vmcnt() {
  static_assert(N >= 0 && N < 64, "vmcnt is 6 bits");
  __builtin_amdgcn_s_waitcnt((N & 15) | ((N >> 4) << 14) | (7 << 4) | (15 << 8));
}

// Calls f(integral_constant<int, 0>) ... f(integral_constant<int, N-1>).
template <int N, int I = 0, class F>
__device__ __forceinline__ void static_for(F&& f) {
  if constexpr (I < N) {
    f(std::integral_constant<int, I>{});
    static_for<N, I + 1>(f);
  }
}

}  // namespace bt
