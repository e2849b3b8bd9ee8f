// Small device-side helpers shared by the gfx950 kernels: vector types, bf16 conversion, GELU.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "kernels.h"

namespace wf {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

// float -> bf16 with round-to-nearest-even (gfx950 has the conversion in hardware).
__device__ __forceinline__ bf16x4 to_bf16x4(f32x4 v) { return __builtin_convertvector(v, bf16x4); }
__device__ __forceinline__ float bf16_to_float(__bf16 v) { return (float)v; }

// Exact-form GELU, z/2 (1 + erf(z / sqrt 2)), for the fp32 debug path.
__device__ __forceinline__ float gelu_erf(float z) { return 0.5f * z * (1.0f + erff(z * 0.70710678118654752f)); }

// GELU for the bf16 path, z Phi(z) = z (1/2 + erf(z / sqrt 2) / 2), without transcendental instructions: its cost
// sits in the GEMM epilogue while the matrix pipe idles.  erf(z / sqrt 2) / 2 ~ c Q(c^2) with c = z clamped to
// +-2.8 sqrt 2 and Q a degree-7 near-minimax polynomial (|erf error| <= 7.5e-5; erf(2.8) = 0.99992 beyond the clamp):
// 11 instructions per value (clamp, square, 7 fused multiply-adds, one more, one multiply).
// Relative error of the result <= 4.7e-4 wherever |GELU| > 0.05, i.e. 8 times below the half-ulp of the
// bf16 value it is rounded to; absolute error <= 1.5e-4 for |z| <= 4 and <= 6e-5 |z| beyond (past the clamp
// Phi saturates at 0.99994 / 0.00006 instead of 1 / 0).
__host__ __device__ __forceinline__ float gelu_fast(float z) {
  const float c = fminf(fmaxf(z, -3.959797975f), 3.959797975f);
  const float t = c * c;
  float q = -1.672331698e-09f;
  q = q * t + 1.267176756e-07f;
  q = q * t - 4.209586276e-06f;
  q = q * t + 8.185916601e-05f;
  q = q * t - 1.055126184e-03f;
  q = q * t + 9.685237790e-03f;
  q = q * t - 6.620135098e-02f;
  q = q * t + 3.988568696e-01f;
  return z * (c * q + 0.5f);              // z (1/2 + erf(z / sqrt 2) / 2)
}

// Sums and maxima over the lanes of a wave in the vector unit: rotations inside a row of 16 lanes, swaps of rows and of halves.
// A step takes about 10 cycles where a shuffle through the LDS takes about 100, and these steps lie on the critical chain of every
// kernel that uses them (LayerNorm of 425 x 1280 4.0 -> 3.2 us a launch, 6420 x 1280 11.4 -> 9.7, 75 x 384 2.6 -> 2.3; an encoder call of 31 694 rows
// 40.08 -> 39.58 ms).
template <int N>
__device__ __forceinline__ float row_rotate(float v) {
  return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), 0x120 + N, 0xF, 0xF, true));
}
struct Pair { float a, b; };
// a: the even rows' values in every pair of rows (the lower half's in both halves), b: the odd rows' (the upper half's)
__device__ __forceinline__ Pair row_pair(float v) {
  const unsigned u = __builtin_bit_cast(unsigned, v);
  const auto r = __builtin_amdgcn_permlane16_swap(u, u, false, false);
  return {__builtin_bit_cast(float, (unsigned)r[0]), __builtin_bit_cast(float, (unsigned)r[1])};
}
__device__ __forceinline__ Pair half_pair(float v) {
  const unsigned u = __builtin_bit_cast(unsigned, v);
  const auto r = __builtin_amdgcn_permlane32_swap(u, u, false, false);
  return {__builtin_bit_cast(float, (unsigned)r[0]), __builtin_bit_cast(float, (unsigned)r[1])};
}
__device__ __forceinline__ float row_sum(float v) {          // over the 16 lanes of a row
  v += row_rotate<8>(v);
  v += row_rotate<4>(v);
  v += row_rotate<2>(v);
  return v + row_rotate<1>(v);
}
__device__ __forceinline__ float half_sum(float v) { const Pair p = half_pair(v); return p.a + p.b; }         // of lanes l and l + 32
__device__ __forceinline__ float half_max(float v) { const Pair p = half_pair(v); return fmaxf(p.a, p.b); }
// (lanes 32 apart first, then 16, .. 1: bit for bit the sum that shuffles of the lane number's bits from the highest down give)
__device__ __forceinline__ float wave_sum(float v) {
  const Pair p = row_pair(half_sum(v));
  return row_sum(p.a + p.b);
}
__device__ __forceinline__ float wave_max(float v) {
  v = fmaxf(v, row_rotate<8>(v));
  v = fmaxf(v, row_rotate<4>(v));
  v = fmaxf(v, row_rotate<2>(v));
  v = fmaxf(v, row_rotate<1>(v));
  const Pair p = row_pair(v);
  return half_max(fmaxf(p.a, p.b));
}
__device__ __forceinline__ float wave_min(float v) { return -wave_max(-v); }

// The share of workgroup `block` of f.blocks (256 threads or more, the first 256 take part) in fetching f: loads into 4 KB of
// LDS that nobody reads.
__device__ __forceinline__ void prefetch_block(const Prefetch &f, int block, unsigned char *lds) {
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  if (wave >= 4) return;
  const uint32_t share = ((f.bytes + f.blocks * 4096u - 1) / (f.blocks * 4096u)) * 4096, begin = block * share;
  const uint32_t end = begin + share < f.bytes ? begin + share : f.bytes;
  for (uint32_t off = begin + threadIdx.x * 16; off < end; off += 4096)
    __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void *)((const unsigned char *)f.p + off),
                                     (__attribute__((address_space(3))) void *)(lds + wave * 1024), 16, 0, 0);
  __builtin_amdgcn_s_waitcnt(0x0F70);            // vmcnt(0): the LDS is this workgroup's until they have landed
}

// First stream index i with cu[i+1] > r, for a row r in [0, cu[B]).
__device__ __forceinline__ int find_stream(const int32_t *cu, int B, int r) {
  int lo = 0, hi = B - 1;
  while (lo < hi) {
    int mid = (lo + hi) >> 1;
    if (cu[mid + 1] > r) hi = mid; else lo = mid + 1;
  }
  return lo;
}

}  // namespace wf
