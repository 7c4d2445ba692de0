// Adding up the partial rows of LayerNorm gradients (FinalizeJob in kernels.h) inside a weight-gradient launch.
#pragma once

#include "device_util.h"
#include "kernels.h"

namespace hanayo {
namespace k {

// Columns a workgroup of NT threads takes: 256 threads own 32, eight groups of them running down the rows.
template <int NT>
constexpr int finalize_cols() { return NT / 256 * 32; }
inline int finalize_blocks(const FinalizeJob& j, int cols) { return (j.n + cols - 1) / cols; }

// out[c] += sum_r partial[r][c] for the `block`-th group of columns, in the order of finalize_kernel (32 row groups, each
// every 32nd row, added in order), whatever NT is: the same bits in every kernel.  `lds`: NT / 256 * 4 KiB.
template <int NT>
__device__ __forceinline__ void finalize_columns(const FinalizeJob& j, int block, void* lds) {
  const int sub = threadIdx.x >> 8, cl = threadIdx.x & 31, rg = (threadIdx.x & 255) >> 5;
  float(*red)[32] = reinterpret_cast<float(*)[32]>(lds) + sub * 32;
  const int c = (block * (NT / 256) + sub) * 32 + cl;
  float t[4] = {0.f, 0.f, 0.f, 0.f};
  if (c < j.n) {
#pragma unroll 4
    for (int r0 = 0; r0 < j.rows; r0 += 32)
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int r = r0 + rg + 8 * u;
        if (r < j.rows) t[u] += j.partial[(size_t)r * j.ld + c];
      }
  }
#pragma unroll
  for (int u = 0; u < 4; ++u) red[rg + 8 * u][cl] = t[u];
  __syncthreads();
  if (rg == 0 && c < j.n) {
    float total = 0.f;
#pragma unroll
    for (int g = 0; g < 32; ++g) total += red[g][cl];
    float* dst = c < j.split ? j.out0 + c : j.out1 + (c - j.split);
    *dst += total;
  }
}

}  // namespace k
}  // namespace hanayo
