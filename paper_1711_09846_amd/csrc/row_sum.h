// Sum of a member's per-row values (losses) by one workgroup.
#pragma once
#include "common.h"

namespace pbt {

// Sum of p[0 .. rows) by the first n = row_sum_threads(rows) threads of a workgroup (64, or all of it); the total is valid in thread 0.  wsum: 16 floats
// of LDS.
inline int row_sum_threads(int rows) { return rows > 1024 ? 1024 : 64; }
__device__ __forceinline__ float member_row_sum(const float* __restrict__ p, int rows, float* wsum, int n) {
  float acc = 0.f;
  int r = threadIdx.x;
  for (; r + 7 * n < rows; r += 8 * n) {
    float v[8];
#pragma unroll
    for (int q = 0; q < 8; ++q) v[q] = p[r + q * n];
#pragma unroll
    for (int q = 0; q < 8; ++q) acc += v[q];
  }
  for (; r < rows; r += n) acc += p[r];
  acc = wave_sum(acc);
  if (n > 64) {
    if ((threadIdx.x & 63) == 0) wsum[threadIdx.x >> 6] = acc;
    __syncthreads();
    if (threadIdx.x == 0)
      for (int w = 1; w < n / 64; ++w) acc += wsum[w];
  }
  return acc;
}
}  // namespace pbt
