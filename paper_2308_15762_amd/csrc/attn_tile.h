// What the bf16 attention kernels share: fragments, the direct-to-LDS tile layout, the argument block.
#pragma once

#include "device_util.h"
#include "kernels.h"

namespace hanayo {
namespace k {

typedef __attribute__((ext_vector_type(4))) short s16x4;
typedef __attribute__((address_space(3))) s16x4* lds_s16x4_ptr;

// 16-byte fragment straight from global memory (row pointer given): contraction elements 16 kk + 8 (lane / 32) .. +7,
// zero outside [0, d).
__device__ __forceinline__ bf16x8 frag_global(const bf16* row, bool row_ok, int kk, int lane, int d) {
  const int c = kk * 16 + 8 * (lane >> 5);
  bf16x8 z = {0, 0, 0, 0, 0, 0, 0, 0};
  return (row_ok && c < d) ? *reinterpret_cast<const bf16x8*>(row + c) : z;
}

// Accumulator registers 8t .. 8t+7 as a bf16 MFMA operand.
__device__ __forceinline__ bf16x8 pack_half(const f32x16& a, int t) {
  bf16x8 o;
#pragma unroll
  for (int j = 0; j < 8; ++j) o[j] = (bf16)a[8 * t + j];
  return o;
}

struct AttnDev {
  const bf16* qkv;
  const int32_t* valid_len;
  bf16* ctx;
  float* lse;
  const bf16* dctx;
  bf16* dqkv;
  float* delta;  // written by attn_delta or by the pipelined dQ kernel, read by the others
  int s, heads, d, causal;
};

// A kernel's parameters one by one and the block made of them: the first 14 words of them are in scalar registers when the
// kernel starts (see the build flags), a struct would have to be read from memory first.
#define ATTN_PARAMS                                                                                                    \
  const bf16 *qkv, const int32_t *valid_len, float *lse, int s, int heads, int d, int causal, const bf16 *dctx, bf16 *ctx, \
      bf16 *dqkv, float *delta
#define ATTN_BLOCK AttnDev{qkv, valid_len, ctx, lse, dctx, dqkv, delta, s, heads, d, causal}
#define ATTN_ARGS(p) p.qkv, p.valid_len, p.lse, p.s, p.heads, p.d, p.causal, p.dctx, p.ctx, p.dqkv, p.delta

__device__ __forceinline__ int seq_len(const AttnDev& p, int n) {
  if (!p.valid_len) return p.s;
  const int v = p.valid_len[n];
  return v < 1 ? 1 : (v > p.s ? p.s : v);
}

__device__ __forceinline__ void dma4(const void* base, unsigned voff, unsigned lds_byte_addr) {
  asm volatile(
      "s_mov_b32 m0, %2\n\t"
      "s_nop 0\n\t"
      "global_load_lds_dword %0, %1"
      :
      : "v"(voff), "s"(base), "s"(lds_byte_addr)
      : "memory");
}
// LDS rows are unpadded and XOR-swizzled in 16-byte slots so that both access patterns are
// bank-conflict free:
//   16-byte fragment reads: 16 consecutive rows at one slot;
//   transpose reads: 4 consecutive rows x 4 consecutive slots per half wavefront.
// DP = 64 (8 slots/row, two rows per 256-byte bank line): slot' = slot ^ (r1<<2 | r3<<1 | r2)
// DP = 128 (16 slots/row, one row per bank line):         slot' = slot ^ (r1<<3 | r0<<2 | r3<<1 | r2)
// with r0..r3 the low bits of the row.
template <int DP>
struct SwTile {
  static_assert(DP == 64 || DP == 128, "swizzled tiles exist for head dims 64 and 128");
  static constexpr int SPR = DP / 8;
  static constexpr int kRowsPerInstr = 64 / SPR;
  static constexpr int kInstr = 64 / kRowsPerInstr;  // per 64-row tile
  static constexpr int kPerWave = kInstr / 4;
  static constexpr int kBytes = 64 * DP * 2;

  __device__ static int swz(int row) {
    return DP == 64 ? ((((row >> 1) & 1) << 2) | ((row >> 2) & 3)) : (((row & 3) << 2) | ((row >> 2) & 3));
  }
  // This wavefront's share of the tile whose first row is row0 (rows clamped to s-1).  D = the row
  // length actually present in memory: for D < DP the slots past it are left as they are (every
  // instruction still has active lanes, so the load counts per wavefront do not change); their
  // contents only ever reach output columns >= D, which are not stored.
  template <int D = DP>
  __device__ static void issue(const bf16* gbase, int ld, int row0, int s, unsigned lds_addr, int wave, int lane) {
    issue_range<D, kPerWave>(gbase, ld, row0, s, lds_addr, wave * kPerWave, lane);
  }
  // The first 32 rows of a tile, all by one wavefront.
  static constexpr int kInstr32 = kInstr / 2;
  template <int D = DP>
  __device__ static void issue32(const bf16* gbase, int ld, int row0, int s, unsigned lds_addr, int lane) {
    issue_range<D, kInstr32>(gbase, ld, row0, s, lds_addr, 0, lane);
  }
  template <int D, int N>
  __device__ static void issue_range(const bf16* gbase, int ld, int row0, int s, unsigned lds_addr, int first, int lane) {
    static_assert(D % 16 == 0 && D <= DP, "row length for this layout");
#pragma unroll
    for (int i = 0; i < N; ++i) {
      const int q = first + i;
      const int lr = q * kRowsPerInstr + lane / SPR, sp = lane % SPR;
      const int row = min(row0 + lr, s - 1);
      const int src = sp ^ swz(lr);  // the global slot that lands in LDS slot sp of this row
      if (D == DP || src < D / 8) dma16(gbase, (unsigned)((row * ld + (src << 3)) * 2), lds_addr + q * 1024);
    }
  }
  // Per-lane byte offsets of every fragment read inside a tile, computed once per kernel.  The swizzle
  // depends on the row's low four bits only, so a fragment that starts r0 rows further down (r0 a
  // multiple of 16) is the same offset plus r0 * SPR * 16, an immediate in the LDS instruction.
  struct Offsets {
    unsigned rows[DP / 16];     // 16-byte fragment of contraction step kk (rows = lane % 32)
    unsigned cols_lo[DP / 32];  // transpose reads of column tile dt: tile rows 4 (lane/32) + 0..3
    unsigned cols_hi[DP / 32];  //                                   and those rows + 8
  };
  __device__ static void init(Offsets& f, int lane) {
#pragma unroll
    for (int kk = 0; kk < DP / 16; ++kk) {
      const int row = lane & 31, slot = 2 * kk + (lane >> 5);
      f.rows[kk] = (unsigned)((row * SPR + (slot ^ swz(row))) * 16);
    }
#pragma unroll
    for (int dt = 0; dt < DP / 32; ++dt) {
      const int row = 4 * (lane >> 5) + ((lane & 15) >> 2);
      const int col = 32 * dt + 16 * ((lane >> 4) & 1) + (lane & 3) * 4;
      const int slot = col >> 3, sub = (col & 7) * 2;
      f.cols_lo[dt] = (unsigned)((row * SPR + (slot ^ swz(row))) * 16 + sub);
      f.cols_hi[dt] = (unsigned)(((row + 8) * SPR + (slot ^ swz(row + 8))) * 16 + sub);
    }
  }
  // rows r0 + lane % 32 (r0 multiple of 16), contraction step kk
  __device__ static bf16x8 frag_rows(const char* lds, const Offsets& f, int r0, int kk) {
    return *reinterpret_cast<const bf16x8*>(lds + f.rows[kk] + r0 * SPR * 16);
  }
  // columns 32 dt + lane % 32; contraction rows r0 + {0..3, 8..11} + 4 (lane / 32) (r0 multiple of 16)
  __device__ static bf16x8 frag_cols(const char* lds, const Offsets& f, int r0, int dt) {
    union {
      struct { s16x4 lo, hi; } s;
      bf16x8 v;
    } u;
    u.s.lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4_ptr)(lds + f.cols_lo[dt] + r0 * SPR * 16));
    u.s.hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4_ptr)(lds + f.cols_hi[dt] + r0 * SPR * 16));
    return u.v;
  }
};

}  // namespace k
}  // namespace hanayo
