// What the matrix-core kernels share: memory straight to LDS, waits on single
// counters, and fp32 values as bf16 planes.
#pragma once

#include "device.hpp"

namespace cats {

// Plane p of a value as two bf16 planes: the nearest hi, the nearest lo.
__device__ __forceinline__ uint32_t split2_plane(float f, int p) {
  const uint32_t h = bf16_bits(f);
  return p == 0 ? h : bf16_bits(f - __uint_as_float(h << 16));
}

// Plane p of a value as three bf16 planes of 8 significand bits each, cut (not
// rounded), whose sum is the value.  An infinity or NaN is its first plane
// alone, so products make of it what fp32 products do.
__device__ __forceinline__ uint32_t split3_plane(float f, int p) {
  const uint32_t u = __float_as_uint(f);
  const bool special = (u & 0x7f800000u) == 0x7f800000u;
  const float r1 = special ? 0.f : f - __uint_as_float(u & 0xffff0000u);
  const uint32_t u1 = __float_as_uint(r1);
  if (p == 0) return (u >> 16) | (special && (u & 0x007fffffu) ? 0x40u : 0u);
  if (p == 1) return u1 >> 16;
  return __float_as_uint(r1 - __uint_as_float(u1 & 0xffff0000u)) >> 16;
}

__device__ __forceinline__ bool is_finite(float f) {
  return (__float_as_uint(f) & 0x7f800000u) != 0x7f800000u;
}
// Sums of three-plane products: lower[t] becomes first[t] (the first plane's
// sum) plus lower[t] (the other two's) where the first is finite, the first
// alone where it is not.  An infinite weight makes of the first plane (which
// has the value's sign, and is zero only where the value is zero or below
// 2^-126) what it makes of the value itself, but a NaN of a lower plane that is
// zero.  The choice costs most where it is made for each sum (0.55 us at the end
// of a 15 us kernel), so a wave looks for infinities and NaN among its sums
// first.
template <int N>
__device__ __forceinline__ void add_lower_planes(const f32x4 (&first)[N], f32x4 (&lower)[N]) {
  f32x4 zero = {0.f, 0.f, 0.f, 0.f};  // NaN where a sum is infinite or NaN
#pragma unroll
  for (int t = 0; t < N; ++t) {
    lower[t] = first[t] + lower[t];
#pragma unroll
    for (int e = 0; e < 4; ++e) zero[e] = fmaf(lower[t][e], 0.f, zero[e]);
  }
  if (__builtin_expect(__any((zero.x + zero.y) + (zero.z + zero.w) != 0.f), 0)) {
#pragma unroll
    for (int t = 0; t < N; ++t)
#pragma unroll
      for (int e = 0; e < 4; ++e)
        if (!is_finite(first[t][e])) lower[t][e] = first[t][e];
  }
}

// A number known to the compiler, as an argument.
template <int V> struct Const { static constexpr int v = V; };

// Wait until at most N of this wave's memory operations are outstanding
// (they complete in order); no other counter is waited for.
template <int N> __device__ __forceinline__ void wait_vm() {
  static_assert(N >= 0 && N < 64, "vmcnt is six bits");
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_waitcnt((N & 15) | ((N >> 4) << 14) | 0x0f70);
  asm volatile("" ::: "memory");
}
// Wait until this wave's LDS reads and writes are done.
__device__ __forceinline__ void wait_lds() {
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_waitcnt(0xc07f);
  asm volatile("" ::: "memory");
}

// 16 bytes per lane from memory to LDS (lane l's at dst + 16 l).
template <int POLICY = 0>
__device__ __forceinline__ void dma16(__amdgpu_buffer_rsrc_t r, uint8_t* dst, uint32_t off) {
  __builtin_amdgcn_raw_ptr_buffer_load_lds(r, (__attribute__((address_space(3))) void*)dst, 16, (int)off, 0, 0, POLICY);
}

}  // namespace cats
