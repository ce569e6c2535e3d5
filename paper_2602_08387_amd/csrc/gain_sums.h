// Column sums of the partial rows that the RMSNorm backward leaves, for a kernel of its own (elementwise.hip) and as workgroups of
// another launch (gemm_tile.hip).
#pragma once
#include "common.h"
#include "kernels.h"

namespace dl {

// workgroups: one per 32 columns of each norm
inline __host__ __device__ int gain_sum_blocks(const GainSums& s) { return (s.D + 31) / 32 * (s.pb ? 2 : 1); }

// Workgroup `block` of NT threads: 32 columns in 32 row groups, folded through LDS (red: 32 x 33 floats).  Four loads in flight per thread
// and 32 groups: the work is a chain of load latencies (512 rows: 7 us with 8 groups, 5 us with 32).  A column's sum has the same
// bits whatever NT.
template <int NT>
__device__ __forceinline__ void gain_sums(const GainSums& s, int block, float* red) {
  const int per_norm = (s.D + 31) / 32;
  const bool second = block >= per_norm;
  const float* partial = second ? s.pb : s.pa;
  bf16_t* out = static_cast<bf16_t*>(second ? s.outb : s.outa);
  const int cl = threadIdx.x & 31, c = (second ? block - per_norm : block) * 32 + cl;
  for (int rg = threadIdx.x >> 5; rg < 32; rg += NT / 32) {
    float s0 = 0.f, s1 = 0.f, s2 = 0.f, s3 = 0.f;
    if (c < s.D) {
      int r = rg;
      for (; r + 96 < s.nrows; r += 128) {
        s0 += partial[(int64_t)r * s.D + c];
        s1 += partial[(int64_t)(r + 32) * s.D + c];
        s2 += partial[(int64_t)(r + 64) * s.D + c];
        s3 += partial[(int64_t)(r + 96) * s.D + c];
      }
      for (; r < s.nrows; r += 32) s0 += partial[(int64_t)r * s.D + c];
    }
    red[rg * 33 + cl] = (s0 + s1) + (s2 + s3);
  }
  __syncthreads();
  if (threadIdx.x < 32 && c < s.D) {
    float t = 0.f;
#pragma unroll
    for (int g = 0; g < 32; ++g) t += red[g * 33 + cl];
    if (s.accumulate) t += (float)out[c];
    out[c] = (bf16_t)t;
  }
}

}  // namespace dl
