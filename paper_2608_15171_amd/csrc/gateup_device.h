// What the projection's kernels share (device code).
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

namespace ppas {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef __attribute__((address_space(3))) void lds_void;

__device__ __forceinline__ u32x4 lds16(const char* p) { return *reinterpret_cast<const u32x4*>(p); }
__device__ __forceinline__ bf16x8 as_bf16x8(u32x4 v) { return __builtin_bit_cast(bf16x8, v); }

__device__ __forceinline__ uint32_t pack_bf16x2(float a, float b) {
  const f32x2 v = {a, b};
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2));
}

// silu(g) = g / (1 + e^-g) in fp32 (e^-g through the hardware base-2 exponential;
// +inf for large negative g, which gives -0).
__device__ __forceinline__ float silu_f32(float g) {
  return g / (1.f + __builtin_amdgcn_exp2f(-g * 1.4426950408889634f));
}

// Wait until at most N of this wave's transfers (and stores) are in flight
// (vmcnt: bits 3:0 and 15:14 of the s_waitcnt immediate; they complete in order).
template <int N>
__device__ __forceinline__ void wait_vmcnt() {
  static_assert(N >= 0 && N < 64, "vmcnt range");
  __builtin_amdgcn_s_waitcnt(0x0F70 | (N & 15) | ((N >> 4) << 14));
}

// Workgroup barrier without a memory fence (the fence of __syncthreads would wait
// for every transfer in flight). The LDS data it guards is written only by the
// transfers, whose completion each wave waits for explicitly before it; the empty
// asm keeps the compiler from moving memory accesses across it.
__device__ __forceinline__ void bare_barrier() {
  asm volatile("" ::: "memory");
  __builtin_amdgcn_sched_barrier(0);
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_sched_barrier(0);
  asm volatile("" ::: "memory");
}

// fp32 partial sums: columns n .. n + 3 of a token row, valid below `lim`.
__device__ __forceinline__ void store_part(float* row, int n, int lim, bool vec, f32x4 v) {
  if (n + 4 <= lim && vec) {
    *reinterpret_cast<f32x4*>(row + n) = v;
  } else {
#pragma unroll
    for (int e = 0; e < 4; ++e)
      if (n + e < lim) row[n + e] = v[e];
  }
}

}  // namespace
}  // namespace ppas
