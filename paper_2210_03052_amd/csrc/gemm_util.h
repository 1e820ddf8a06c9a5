// What the product kernels share: activations, DMA into LDS, hand-written waits.
#pragma once
#include <type_traits>

#include "common.h"

namespace bt {

#define BT_AS1 __attribute__((address_space(1)))
#define BT_AS3 __attribute__((address_space(3)))

// Exact-form GELU, x * Phi(x).  With h(a) = Phi(-a) = 0.5 erfc(a / sqrt 2), a = |x|:
//   Phi(x) = x >= 0 ? 1 - h : h,  so  x Phi(x) = max(x, 0) - a h(a)  in both cases.
// log2 h(a) is smooth (-1 at a = 0, ~ -a^2/2 log2 e further out), so h = exp2(P(a)) with P a degree-7
// polynomial fitted (weighted least squares iterated to minimax) to log2 h on [0, 6]: |P - log2 h| <=
// 4.8e-6 there, i.e. h to 3.3e-6 RELATIVE, and the small negative outputs keep their fp16 digits
// too.  In fp32 arithmetic the result is within 6e-7 of x Phi(x) everywhere and rounds to the same
// fp16 value as the fp64 definition for 99.9 % of inputs (1 ulp otherwise).  The leading
// coefficient is negative and P decreases monotonically, so beyond the fitted range exp2(P)
// underflows to 0 (a h(a) < 3e-9 there anyway).  Nine VALU instructions, one transcendental; the
// epilogue runs once per output element and is not overlapped with MFMA work.
__device__ __forceinline__ float gelu_erf(float x) {
  const float a = fabsf(x);
  float p = __builtin_fmaf(a, -1.83486475e-06f, 6.15994941e-05f);
  p = __builtin_fmaf(a, p, -0.000930535374f);
  p = __builtin_fmaf(a, p, 0.00850793719f);
  p = __builtin_fmaf(a, p, -0.0539601706f);
  p = __builtin_fmaf(a, p, -0.458464265f);
  p = __builtin_fmaf(a, p, -1.15125108f);
  p = __builtin_fmaf(a, p, -0.999995291f);
  return __builtin_fmaf(-a, __builtin_amdgcn_exp2f(p), fmaxf(x, 0.f));
}
// tanh form: 0.5 x (1 + tanh u) = x / (1 + exp(-2u)),  u = sqrt(2/pi) (x + 0.044715 x^3).
__device__ __forceinline__ float gelu_tanh(float x) {
  constexpr float k1 = -2.0f * 1.4426950408889634f * 0.7978845608028654f, k3 = k1 * 0.044715f;
  const float e = __builtin_amdgcn_exp2f(x * __builtin_fmaf(x * x, k3, k1));
  return x * __builtin_amdgcn_rcpf(1.0f + e);
}

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
