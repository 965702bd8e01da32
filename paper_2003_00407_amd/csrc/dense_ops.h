// Device helpers shared by the dense kernels: column codes, small-matrix slots,
// global-address-space accesses, FP64 and FP32 matrix instructions, block reductions.
#pragma once

#include "dg_internal.h"
#include "wave_ops.h"

namespace dg {

// column-count codes: > 0 explicit, 0 -> E.K, -1 -> E.J
__device__ __forceinline__ int kcode(int k, const ElemDev& E) { return k > 0 ? k : (k == 0 ? E.K : E.J); }
// small-matrix offsets: >= 0 explicit, -1-w -> SmallLayout slot w for this element
__device__ __forceinline__ long long soff(long long o, const ElemDev& E) {
  if (o >= 0) return o;
  const int KP = E.kmax3 + 2;
  switch (-1 - (int)o) {
    case 0: return SmallLayout::G(KP);
    case 1: return SmallLayout::A(KP);
    case 2: return SmallLayout::U(KP);
    case 3: return SmallLayout::V(KP);
    default: return SmallLayout::C(KP);
  }
}
// rows of the blocks a kernel works on: 0 -> N (Q_k grid), 1 -> |E_k|
__device__ __forceinline__ int nrows_of(const ElemDev& E, int rows_e) {
  return rows_e ? E.en[0] * E.en[1] * E.en[2] : E.N;
}

// Loads through a global-address-space pointer: the block pointers come from tables
// in memory, so the compiler cannot infer the address space and would otherwise use
// flat loads, which also count against the LDS counter and get conservative waits.
typedef double gd2 __attribute__((ext_vector_type(2)));
template <typename V>
__device__ __forceinline__ V gload(const void* p) {
  return *(const __attribute__((address_space(1))) V*)(p);
}
__device__ __forceinline__ double2 gload2(const void* p) {
  const gd2 v = *(const __attribute__((address_space(1))) gd2*)(p);
  return double2{v.x, v.y};
}
// store through a global-address-space pointer (a flat store would make later LDS waits
// wait for its completion)
template <typename V>
__device__ __forceinline__ void gstore(V* p, V v) { *(__attribute__((address_space(1))) V*)(p) = v; }
typedef float gf2 __attribute__((ext_vector_type(2)));
typedef float gf4 __attribute__((ext_vector_type(4)));
__device__ __forceinline__ float2 gload2f(const void* p) {
  const gf2 v = *(const __attribute__((address_space(1))) gf2*)(p);
  return float2{v.x, v.y};
}
__device__ __forceinline__ void gstore2f(void* p, float x, float y) {
  *(__attribute__((address_space(1))) gf2*)(p) = gf2{x, y};
}
__device__ __forceinline__ void gstore2(void* p, double x, double y) {
  *(__attribute__((address_space(1))) gd2*)(p) = gd2{x, y};
}

typedef double d4v __attribute__((ext_vector_type(4)));
typedef float f4v __attribute__((ext_vector_type(4)));

// v_mfma_f64_16x16x4f64 lane layout (checked on the device): lane l supplies
// A[l%16][l/16] and B[l/16][l%16]; result register q of lane l is D[l/16 + 4q][l%16].
__device__ __forceinline__ d4v mfma16x16x4(double a, double b, d4v c) {
  return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
}

// ---------------------------------------------------------------------------
// block reductions
// ---------------------------------------------------------------------------
__device__ __forceinline__ double wave_sum(double v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
  return v;
}

// sum over the block, result broadcast to every thread (fixed order)
__device__ inline double block_sum(double v, double* sh) {
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, nw = (blockDim.x + 63) >> 6;
  v = wave_sum(v);
  __syncthreads();
  if (lane == 0) sh[w] = v;
  __syncthreads();
  double s = 0.0;
  for (int i = 0; i < nw; ++i) s += sh[i];
  __syncthreads();
  return s;
}

__device__ inline double block_max(double v, double* sh) {
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, nw = (blockDim.x + 63) >> 6;
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v = fmax(v, __shfl_xor(v, o));
  __syncthreads();
  if (lane == 0) sh[w] = v;
  __syncthreads();
  double s = sh[0];
  for (int i = 1; i < nw; ++i) s = fmax(s, sh[i]);
  __syncthreads();
  return s;
}

// Workgroup barrier that orders LDS only: __syncthreads() also waits for every global
// store in flight (about a microsecond), which a step that only hands on LDS need not.
__device__ __forceinline__ void lds_barrier() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

}  // namespace dg
