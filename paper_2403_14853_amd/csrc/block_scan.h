// Workgroup-wide sums and prefix sums of the integer bookkeeping kernels (256 threads).
#pragma once
#include "isp_internal.h"

namespace isp_dev {

constexpr int BS_THREADS = 256;

// Orders this wave's earlier LDS writes before its later LDS reads (other lanes' data).  The LDS
// unit executes one wave's operations in order, so only the compiler has to be held back.
__device__ inline void wave_lds_sync() {
  __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

template <typename T>
__device__ inline T wave_inclusive_scan(T v, int lane) {
#pragma unroll
  for (int o = 1; o < ISP_WAVE; o <<= 1) {
    T t = __shfl_up(v, o);
    if (lane >= o) v += t;
  }
  return v;
}

// Exclusive scan of one value per thread across the workgroup; returns the exclusive prefix and
// writes the workgroup total to *total (same value in every thread).
template <typename T>
__device__ inline T block_exclusive_scan(T v, T* total) {
  __shared__ T wave_tot[BS_THREADS / ISP_WAVE];
  const int lane = threadIdx.x & (ISP_WAVE - 1), w = threadIdx.x / ISP_WAVE;
  T inc = wave_inclusive_scan(v, lane);
  __syncthreads();  // protect wave_tot against a previous call's readers
  if (lane == ISP_WAVE - 1) wave_tot[w] = inc;
  __syncthreads();
  T base = 0, tot = 0;
#pragma unroll
  for (int i = 0; i < BS_THREADS / ISP_WAVE; ++i) {
    if (i < w) base += wave_tot[i];
    tot += wave_tot[i];
  }
  *total = tot;
  return base + inc - v;
}

// Sum of a[0 .. n) by the whole workgroup, same value in every thread.
template <typename T>
__device__ inline T block_sum_of(const T* __restrict__ a, int n) {
  T s = 0;
#pragma unroll 8
  for (int i = threadIdx.x; i < n; i += BS_THREADS) s += a[i];
  T tot;
  block_exclusive_scan<T>(s, &tot);
  return tot;
}

}  // namespace isp_dev
