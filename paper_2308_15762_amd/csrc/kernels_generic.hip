// A GEMM on the ALU for the shapes that the matrix-instruction kernels do not take (extents or leading dimensions that
// are no multiple of a 16-byte vector, unaligned bases), and the row sums of the bf16 attention backward pass.
#include "device_util.h"
#include "epilogue.h"
#include "kernels.h"

namespace hanayo {
namespace k {

namespace {

// ---------------------------------------------------------------- GEMM 64x64x16
template <typename T, int EPI>
__global__ __launch_bounds__(256) void gemm_alu_kernel(const T* __restrict__ A, const T* __restrict__ B, int M, int N,
                                                       int K, int lda, int ldb, bool a_t, bool b_t,
                                                       const int* __restrict__ live, int live_dim, EpiParams<T> ep) {
  __shared__ float As[16][64 + 4];
  __shared__ float Bs[16][64 + 4];
  const int tx = threadIdx.x & 15, ty = threadIdx.x >> 4;
  const int tiles_n = (N + 63) / 64, m0 = (int)(blockIdx.x / tiles_n) * 64, n0 = (int)(blockIdx.x % tiles_n) * 64;
  if (live) {
    (live_dim == LIVE_K ? K : M) = live[0];
    if (live[0] < 1 || m0 >= M) return;
  }
  float acc[4][4], sum[4][4];  // of the last 65536 contraction elements, of all before: in one sum over a vocabulary of millions
                               // the later terms would be lost
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j) acc[i][j] = sum[i][j] = 0.f;
  for (int k0 = 0; k0 < K; k0 += 16) {
    if (k0 && k0 % 65536 == 0) {
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) sum[i][j] += acc[i][j], acc[i][j] = 0.f;
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int idx = threadIdx.x + i * 256;
      int mm, kk;
      if (a_t) { kk = idx >> 6; mm = idx & 63; } else { mm = idx >> 4; kk = idx & 15; }
      const int gm = m0 + mm, gk = k0 + kk;
      float v = 0.f;
      if (gm < M && gk < K) v = ld(A + (a_t ? (size_t)gk * lda + gm : (size_t)gm * lda + gk));
      As[kk][mm] = v;
      int nn;
      if (b_t) { kk = idx >> 6; nn = idx & 63; } else { nn = idx >> 4; kk = idx & 15; }
      const int gn = n0 + nn, gk2 = k0 + kk;
      v = 0.f;
      if (gn < N && gk2 < K) v = ld(B + (b_t ? (size_t)gk2 * ldb + gn : (size_t)gn * ldb + gk2));
      Bs[kk][nn] = v;
    }
    __syncthreads();
#pragma unroll
    for (int kk = 0; kk < 16; ++kk) {
      float a[4], b[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) a[i] = As[kk][ty * 4 + i];
#pragma unroll
      for (int j = 0; j < 4; ++j) b[j] = Bs[kk][tx * 4 + j];
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) acc[i][j] += a[i] * b[j];
    }
    __syncthreads();
  }
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int m = m0 + ty * 4 + i, n = n0 + tx * 4 + j;
      if (m < M && n < N) epilogue_one<T, EPI>(ep, m, n, sum[i][j] + acc[i][j]);
    }
}

// ---------------------------------------------------------------- attention
// delta[n][h][i] = sum_c dctx[i][c] * ctx[i][c].  ctx and dctx are read as one stream of 8-element
// vectors (d / 8 consecutive vectors make one (row, head) group); a workgroup takes kDeltaGroups
// groups, parks the per-vector sums in LDS and adds each group up.
constexpr int kDeltaGroups = 64;
__global__ __launch_bounds__(256) void attn_delta_kernel(const bf16* __restrict__ ctx, const bf16* __restrict__ dctx,
                                                         float* __restrict__ delta, long groups, int s, int heads, int d) {
  __shared__ float part[kDeltaGroups * 16];
  const int vpg = d / 8;  // vectors per group, at most 16
  const long g0 = (long)blockIdx.x * kDeltaGroups;
  const int ng = (int)(groups - g0 < kDeltaGroups ? groups - g0 : kDeltaGroups);
  for (int v = threadIdx.x; v < ng * vpg; v += 256) {
    float a[8], b[8];
    load8(ctx + (g0 * vpg + v) * 8, a);
    load8(dctx + (g0 * vpg + v) * 8, b);
    float t = 0.f;
#pragma unroll
    for (int e = 0; e < 8; ++e) t += a[e] * b[e];
    part[v] = t;
  }
  __syncthreads();
  if ((int)threadIdx.x < ng) {
    float t = 0.f;
    for (int j = 0; j < vpg; ++j) t += part[threadIdx.x * vpg + j];
    const long g = g0 + threadIdx.x;  // = row * heads + head
    const long row = g / heads;
    const int h = (int)(g - row * heads);
    delta[((row / s) * heads + h) * s + row % s] = t;
  }
}

template <typename T>
int gemm_alu_t(const GemmArgs& g, hipStream_t stream) {
  EpiParams<T> ep{(T*)g.C, (float*)g.C, (const T*)g.bias, (const T*)g.aux, (T*)g.aux_out, g.ldc};
  const long tiles = (long)((g.N + 63) / 64) * ((g.M + 63) / 64);  // in one dimension: the others end at 65535 workgroups
  if (tiles >= 1L << 24) return set_error(HANAYO_EUNSUPPORTED, "gemm_alu: too many tiles");
  if (g.live && g.live_dim == LIVE_M_SPLIT) return set_error(HANAYO_EUNSUPPORTED, "gemm_alu: split contraction");
  const dim3 grid((unsigned)tiles), block(256);
#define LAUNCH(E)                                                                                                    \
  case E:                                                                                                            \
    launch_kernel((gemm_alu_kernel<T, E>), grid, block, 0, stream, (const T*)g.A, (const T*)g.B, g.M, g.N, g.K, \
                       g.lda, g.ldb, g.a_t, g.b_t, g.live, g.live_dim, ep);                                                          \
    break
  switch (g.epi) {
    LAUNCH(EPI_NONE);
    LAUNCH(EPI_BIAS);
    LAUNCH(EPI_BIAS_GELU);
    LAUNCH(EPI_BIAS_RES);
    LAUNCH(EPI_MUL_DGELU);
    LAUNCH(EPI_ADD);
    LAUNCH(EPI_ACCUM_F32);
    default: return set_error(HANAYO_EUNSUPPORTED, "gemm_alu: epilogue");
  }
#undef LAUNCH
  return check_launch("gemm_alu");
}

}  // namespace

int gemm_alu(int dtype, const GemmArgs& g, hipStream_t stream) {
  return dtype == HANAYO_BF16 ? gemm_alu_t<bf16>(g, stream) : gemm_alu_t<float>(g, stream);
}
int attn_delta(const AttnArgs& a, hipStream_t stream) {
  if (a.d % 8 || a.d > 128) return set_error(HANAYO_EUNSUPPORTED, "attn_delta: head dim %d", a.d);
  const long groups = (long)a.b * a.s * a.heads;
  launch_kernel(attn_delta_kernel, dim3((unsigned)((groups + kDeltaGroups - 1) / kDeltaGroups)), dim3(256), 0, stream,
                     (const bf16*)a.ctx, (const bf16*)a.dctx, a.delta, groups, a.s, a.heads, a.d);
  return check_launch("attn_delta");
}

}  // namespace k
}  // namespace hanayo
