// Fixed-order sums of fp32 partials: the split weight gradients' and the
// LayerNorm column sums.  Shared by the per-kernel reductions and by the
// layer backward's last launch, which runs all of a layer's in one grid.
#pragma once

#include "common.hpp"
#include "geometry.hpp"

namespace optimus {

// out[i] = (accumulate ? out[i] : 0) + part[0][i] + part[1][i] + ... in split
// order, for the i-th of n4 float4s.
__device__ __forceinline__ void split_sum_at(long i, long n4, float *out, const float *part, int splits,
                                             int accumulate) {
  f32x4_t v = accumulate ? reinterpret_cast<const f32x4_t *>(out)[i] : f32x4_t{0.f, 0.f, 0.f, 0.f};
  for (int sp = 0; sp < splits; ++sp) v += reinterpret_cast<const f32x4_t *>(part)[sp * n4 + i];
  reinterpret_cast<f32x4_t *>(out)[i] = v;
}

// Columns [64 * bx, 64 * bx + 64) of out (+)= the fixed-order sum of the nblk
// rows of part.  Block = 64 columns (8 chunks of 8) x 32 groups of partial
// rows; the 32 group sums are added in a fixed order through LDS.
constexpr int kRedCols = 64, kRedGroups = 32;

__device__ __forceinline__ void column_sum_block(int bx, int nblk, int cols, const float *__restrict__ part,
                                                 float *__restrict__ out, int accumulate,
                                                 float (*red)[kRedCols + 1]) {
  const int chunk = threadIdx.x & 7, grp = threadIdx.x >> 3;
  const int c0 = bx * kRedCols + chunk * 8;
  float v[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  if (c0 < cols) {
#pragma unroll 4
    for (int b = grp; b < nblk; b += kRedGroups) {
      const float *q = part + static_cast<size_t>(b) * cols + c0;
      const f32x4_t a = *reinterpret_cast<const f32x4_t *>(q);
      const f32x4_t c = *reinterpret_cast<const f32x4_t *>(q + 4);
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        v[e] += a[e];
        v[4 + e] += c[e];
      }
    }
  }
#pragma unroll
  for (int e = 0; e < 8; ++e) red[grp][chunk * 8 + e] = v[e];
  __syncthreads();
  if (threadIdx.x < kRedCols) {
    const int col = bx * kRedCols + threadIdx.x;
    float tsum = 0.f;
#pragma unroll 8
    for (int q = 0; q < kRedGroups; ++q) tsum += red[q][threadIdx.x];
    if (col < cols) out[col] = accumulate ? out[col] + tsum : tsum;
  }
}

}  // namespace optimus
