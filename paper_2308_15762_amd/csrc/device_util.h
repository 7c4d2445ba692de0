// Device-side helpers shared by the HIP kernels: storage types, 8-wide row
// access, wavefront (64-lane) reductions, GELU.
#pragma once

#include <hip/hip_runtime.h>

namespace hanayo {

typedef __bf16 bf16;
typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(4))) __bf16 bf16x4;
typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((ext_vector_type(16))) float f32x16;

constexpr int kWave = 64;

// Eight consecutive elements <-> eight floats.
__device__ __forceinline__ void load8(const float* p, float (&v)[8]) {
  const f32x4 a = *reinterpret_cast<const f32x4*>(p);
  const f32x4 b = *reinterpret_cast<const f32x4*>(p + 4);
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    v[i] = a[i];
    v[4 + i] = b[i];
  }
}
__device__ __forceinline__ void load8(const bf16* p, float (&v)[8]) {
  const bf16x8 a = *reinterpret_cast<const bf16x8*>(p);
#pragma unroll
  for (int i = 0; i < 8; ++i) v[i] = (float)a[i];
}
__device__ __forceinline__ void store8(float* p, const float (&v)[8]) {
  f32x4 a, b;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    a[i] = v[i];
    b[i] = v[4 + i];
  }
  *reinterpret_cast<f32x4*>(p) = a;
  *reinterpret_cast<f32x4*>(p + 4) = b;
}
__device__ __forceinline__ void store8(bf16* p, const float (&v)[8]) {
  bf16x8 a;
#pragma unroll
  for (int i = 0; i < 8; ++i) a[i] = (bf16)v[i];
  *reinterpret_cast<bf16x8*>(p) = a;
}

__device__ __forceinline__ float ld(const float* p) { return *p; }
__device__ __forceinline__ float ld(const bf16* p) { return (float)*p; }
__device__ __forceinline__ void st(float* p, float v) { *p = v; }
__device__ __forceinline__ void st(bf16* p, float v) { *p = (bf16)v; }

// Butterfly reductions over lanes l ^ 32, l ^ 16, ... l ^ 1 without the LDS crossbar that __shfl_xor goes through (about 100
// cycles a step): the swaps exchange halves and 16-lane rows between two registers, and inside a row a rotation by 8 is l ^ 8,
// after which lanes that differ by 8 agree and a rotation by 4 is as good as l ^ 4, and so on.  The same additions in the same
// tree: the bits of the shuffles.  All 64 lanes have to be active.
template <typename Op>
__device__ __forceinline__ float reduce_halves(float v, Op op) {  // over l and l ^ 32
  const unsigned u = __float_as_uint(v);
  const auto r = __builtin_amdgcn_permlane32_swap(u, u, false, false);
  return op(__uint_as_float(r[0]), __uint_as_float(r[1]));
}
template <int N, typename Op>
__device__ __forceinline__ float reduce_rotated(float v, Op op) {
  const int u = (int)__float_as_uint(v);
  return op(v, __uint_as_float((unsigned)__builtin_amdgcn_update_dpp(u, u, 0x120 + N, 0xf, 0xf, false)));  // row_ror:N
}
template <typename Op>
__device__ __forceinline__ float reduce_half(float v, Op op) {  // over the 32 lanes of each half
  const unsigned u = __float_as_uint(v);
  const auto r = __builtin_amdgcn_permlane16_swap(u, u, false, false);
  v = op(__uint_as_float(r[0]), __uint_as_float(r[1]));
  v = reduce_rotated<8>(v, op);
  v = reduce_rotated<4>(v, op);
  v = reduce_rotated<2>(v, op);
  return reduce_rotated<1>(v, op);
}
struct AddOp {
  __device__ __forceinline__ float operator()(float a, float b) const { return a + b; }
};
struct MaxOp {
  __device__ __forceinline__ float operator()(float a, float b) const { return fmaxf(a, b); }
};
__device__ __forceinline__ float halves_sum(float v) { return reduce_halves(v, AddOp()); }
__device__ __forceinline__ float halves_max(float v) { return reduce_halves(v, MaxOp()); }
__device__ __forceinline__ float wave_sum(float v) { return reduce_half(reduce_halves(v, AddOp()), AddOp()); }
__device__ __forceinline__ float wave_max(float v) { return reduce_half(reduce_halves(v, MaxOp()), MaxOp()); }

// Workgroup -> output tile, XCD-aware.  The dispatcher hands consecutive workgroup ids to the chip's
// 8 XCDs in turn, and each XCD has an L2 of its own, so workgroup w runs on XCD w % 8 as that XCD's
// (w / 8)-th.  Each XCD therefore gets one contiguous run of tile numbers, and tile numbers walk the
// tile grid in bands of kTileBand tile rows, column by column within a band: the workgroups resident
// on one XCD at a time then cover a compact patch of the output and share their operand panels in
// that L2 instead of each XCD fetching every panel.  Any bijection is correct; this one is fast.  A band
// of 8 makes the patch of 32 workgroups 8 x 4 tiles; tiles twice as tall as wide take bands of 4, so that
// the patch is as many rows as columns: 16 panels of a 2048 x 4096 x 16384 product then cross the fabric
// instead of 20 per XCD (see kernels_gemm_dma.hip for what that measured).
constexpr int kXcds = 8;
template <int kTileBand = 8>
__device__ __forceinline__ void xcd_tile(int w, int tiles_m, int tiles_n, int& tm, int& tn) {
  const int total = tiles_m * tiles_n, per = total / kXcds, rem = total % kXcds;
  const int xcd = w % kXcds;
  const int t = xcd * per + (xcd < rem ? xcd : rem) + w / kXcds;
  const int band = t / (kTileBand * tiles_n), first = band * kTileBand;
  const int rows = tiles_m - first < kTileBand ? tiles_m - first : kTileBand;
  const int r = t - band * kTileBand * tiles_n;
  tm = first + r % rows;
  tn = r / rows;
}

// One wavefront-wide 16-byte-per-lane load from global memory into LDS: lane L's vector lands at lds_byte_addr + 16 L.
// `voff` is the lane's byte offset from `base`.  M0 carries the LDS address; it is written and consumed inside the statement,
// and nothing else in these kernels lives in M0 (gfx950 LDS instructions do not use it).
__device__ __forceinline__ void dma16(const void* base, unsigned voff, unsigned lds_byte_addr) {
  asm volatile(
      "s_mov_b32 m0, %2\n\t"
      "s_nop 0\n\t"
      "global_load_lds_dwordx4 %0, %1"
      :
      : "v"(voff), "s"(base), "s"(lds_byte_addr)
      : "memory");
}
// Waits until at most N vector-memory operations of the wavefront are outstanding.
template <int N>
__device__ __forceinline__ void wait_vmcnt() {
  asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
}

constexpr float kLog2e = 1.4426950408889634f;
constexpr float kLn2 = 0.6931471805599453f;
__device__ __forceinline__ f32x16 zero16() {
  f32x16 z;
#pragma unroll
  for (int r = 0; r < 16; ++r) z[r] = 0.f;
  return z;
}
// Row of accumulator register r of a 32 x 32 MFMA inside its tile, for half wavefront `half`.
__device__ __forceinline__ int acc_row(int r, int half) { return 8 * (r >> 2) + 4 * half + (r & 3); }

// GELU(h) = h/2 (1 + erf(h / sqrt 2)) and its derivative Phi(h) + h phi(h).
__device__ __forceinline__ float gelu_f(float h) { return 0.5f * h * (1.0f + erff(h * 0.70710678118654752f)); }
__device__ __forceinline__ float gelu_grad_f(float h) {
  const float cdf = 0.5f * (1.0f + erff(h * 0.70710678118654752f));
  const float pdf = 0.39894228040143268f * __expf(-0.5f * h * h);
  return cdf + h * pdf;
}

// The same two functions from one exponential and a rational erfc approximation
// (Abramowitz & Stegun 7.1.26, absolute error of erf below 1.5e-7): used in the
// bf16 MFMA epilogues, where the result is rounded to bf16 anyway.
//   Phi(|h|) = 1 - 0.5 t (a1 + t (a2 + t (a3 + t (a4 + t a5)))) exp(-h^2 / 2),  t = 1 / (1 + p |h| / sqrt 2)
__device__ __forceinline__ void phi_fast(float h, float& cdf, float& pdf) {
  const float ah = fabsf(h);
  const float t = __frcp_rn(1.0f + 0.3275911f * 0.70710678118654752f * ah);
  const float e = exp2f(-0.72134752044448170f * h * h);  // exp(-h^2 / 2)
  const float poly = t * (0.254829592f + t * (-0.284496736f + t * (1.421413741f + t * (-1.453152027f + t * 1.061405429f))));
  const float tail = 0.5f * poly * e;  // 1 - Phi(|h|)
  cdf = h >= 0.f ? 1.0f - tail : tail;
  pdf = 0.39894228040143268f * e;
}
__device__ __forceinline__ float gelu_fast(float h) {
  float cdf, pdf;
  phi_fast(h, cdf, pdf);
  return h * cdf;
}
__device__ __forceinline__ float gelu_grad_fast(float h) {
  float cdf, pdf;
  phi_fast(h, cdf, pdf);
  return cdf + h * pdf;
}

}  // namespace hanayo
