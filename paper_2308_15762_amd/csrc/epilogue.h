// GEMM epilogues: the ALU kernel's, and the row access of the MFMA kernels'.
#pragma once

#include "device_util.h"
#include "kernels.h"

namespace hanayo {
namespace k {

template <typename T>
struct EpiParams {
  T* C;
  float* Cf;  // EPI_ACCUM_F32 target
  const T* bias;
  const T* aux;
  T* aux_out;
  int ldc;
};

// Eight elements of a row of C, aux or aux_out: rows start on 8-byte boundaries only where ldc is no multiple of 8.  (The
// chip takes such 16-byte accesses; the type keeps the compiler from assuming more than there is.)
typedef bf16x8 bf16x8_row __attribute__((aligned(8)));
__device__ __forceinline__ void load8_row(const bf16* p, float (&v)[8]) {
  const bf16x8 a = *reinterpret_cast<const bf16x8_row*>(p);
#pragma unroll
  for (int i = 0; i < 8; ++i) v[i] = (float)a[i];
}
__device__ __forceinline__ void store8_row(bf16* p, const float (&v)[8]) {
  bf16x8 a;
#pragma unroll
  for (int i = 0; i < 8; ++i) a[i] = (bf16)v[i];
  *reinterpret_cast<bf16x8_row*>(p) = a;
}

// The distance between rows of C, a multiple of 4, and the kind of counted dimension in one kernel argument, for every distance.
inline unsigned pack_ldc(int ldc, int live_dim) { return (unsigned)ldc >> 2 | (unsigned)live_dim << 29; }
__device__ __forceinline__ int ldc_of(unsigned packed) { return (int)((packed & 0x1fffffffu) << 2); }
__device__ __forceinline__ int live_dim_of(unsigned packed) { return (int)(packed >> 29); }

// One output element (m, n) with accumulator value `acc`.
template <typename T, int EPI>
__device__ __forceinline__ void epilogue_one(const EpiParams<T>& p, int m, int n, float acc) {
  const size_t at = (size_t)m * p.ldc + n;
  if constexpr (EPI == EPI_NONE) {
    st(p.C + at, acc);
  } else if constexpr (EPI == EPI_BIAS) {
    st(p.C + at, acc + ld(p.bias + n));
  } else if constexpr (EPI == EPI_BIAS_GELU) {
    const float h = acc + ld(p.bias + n);
    st(p.aux_out + at, h);
    st(p.C + at, gelu_f(h));
  } else if constexpr (EPI == EPI_BIAS_RES) {
    st(p.C + at, acc + ld(p.bias + n) + ld(p.aux + at));
  } else if constexpr (EPI == EPI_MUL_DGELU) {
    st(p.C + at, acc * gelu_grad_f(ld(p.aux + at)));
  } else if constexpr (EPI == EPI_ADD) {
    st(p.C + at, acc + ld(p.aux + at));
  } else {
    p.Cf[at] += acc;
  }
}

}  // namespace k
}  // namespace hanayo
