// The scan of a radix sort's pass, whose table holds the digit counts of every tile, digit by digit (transpose.hip, csr_build.hip).
#pragma once
#include "block_scan.h"

namespace isp_dev {

// One workgroup per digit: exclusive prefix of its counts over the tiles, in place, and the digit's total.  (The prefix
// over the digits is a few hundred numbers, which every scatter workgroup adds up for itself: one launch instead of
// the three of a device-wide scan.)
static __global__ void __launch_bounds__(BS_THREADS) k_digit_scan(int32_t* __restrict__ table, int n_tiles,
                                                           int32_t* __restrict__ digit_total) {
  int32_t* __restrict__ t = table + (int64_t)blockIdx.x * n_tiles;
  int carry = 0;
  constexpr int PER = 8;
  for (int base = 0; base < n_tiles; base += BS_THREADS * PER) {
    int v[PER], sum = 0;
#pragma unroll
    for (int k = 0; k < PER; ++k) {
      const int i = base + (int)threadIdx.x * PER + k;
      v[k] = i < n_tiles ? t[i] : 0;
      sum += v[k];
    }
    int tot;
    int run = carry + block_exclusive_scan<int>(sum, &tot);
#pragma unroll
    for (int k = 0; k < PER; ++k) {
      const int i = base + (int)threadIdx.x * PER + k;
      if (i < n_tiles) t[i] = run;
      run += v[k];
    }
    carry += tot;
  }
  if (threadIdx.x == 0) digit_total[blockIdx.x] = carry;
}

}  // namespace isp_dev
