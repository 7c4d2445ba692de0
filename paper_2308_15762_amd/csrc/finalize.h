// Adding up partial rows (FinalizeJob in kernels.h), in launches of their own and inside a weight-gradient launch.
#pragma once

#include "device_util.h"
#include "kernels.h"

namespace hanayo {
namespace k {

// A group of 32 columns is added up by 1024 / U threads.  Columns a workgroup of NT threads takes:
template <int NT, int U>
constexpr int finalize_cols() { return NT * U / 1024 * 32; }
inline int finalize_blocks(const FinalizeJob& j, int cols) { return (j.n + cols - 1) / cols; }

// out[c] += sum_r partial[r][c] for the `block`-th share of the columns, without atomics and in one fixed order, whatever NT and
// U are: 32 row groups each run down every 32nd partial row (32 lanes x 4 bytes = one 128-byte line per row), U of them in a
// thread, and their sums are added in order through LDS.  Columns >= split go to out1.  U = 1, where the launch does nothing
// else: 256 partial rows are 8 loads per thread, all in flight at once; U = 4 in the workgroups of a GEMM.
// `lds`: NT * U / 1024 * 4 KiB.
template <int NT, int U>
__device__ __forceinline__ void finalize_columns(const FinalizeJob& j, int block, void* lds) {
  constexpr int kThreads = 1024 / U, kStep = 32 / U;
  const int sub = threadIdx.x / kThreads, cl = threadIdx.x % 32, rg = threadIdx.x % kThreads / 32;
  float(*red)[32] = reinterpret_cast<float(*)[32]>(lds) + sub * 32;
  const int c = (block * (NT / kThreads) + sub) * 32 + cl;
  float t[U];
#pragma unroll
  for (int u = 0; u < U; ++u) t[u] = 0.f;
  if (c < j.n) {
    int r = rg;
    const int whole = j.rows - (32 - kStep);
#pragma unroll (U == 1 ? 8 : 4)
    for (; r < whole; r += 32)
#pragma unroll
      for (int u = 0; u < U; ++u) t[u] += j.partial[(size_t)(r + kStep * u) * j.ld + c];
#pragma unroll
    for (int u = 0; u < U - 1; ++u)  // the last partial row of each group, where not every group has it
      if (r + kStep * u < j.rows) t[u] += j.partial[(size_t)(r + kStep * u) * j.ld + c];
  }
#pragma unroll
  for (int u = 0; u < U; ++u) red[rg + kStep * u][cl] = t[u];
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
