// GEMM for the shapes that large tiles serve badly: few output tiles (small models, short micro-batches), ragged
// extents (any token count), and fp32 storage, whose matrix instruction is 16 times slower than bf16's, so that
// tiles have to be small for a launch to reach every CU.
//
// The wavefronts of a workgroup all own the SAME output tile and split the contraction: wavefront w takes K tiles
// w, w + 4, w + 8, ...  Each fills an LDS ring of its own with direct loads and waits for its own loads only, so the
// main loop has no barrier and the chain of dependent K tiles, which bounds a launch of few tiles, is four times
// shorter than with an output split.  A 64 x 64 tile then costs one fragment read per MFMA, half of what four
// wavefronts of 32 x 32 each would read.  The partial tiles are added in a fixed order through LDS at the end.
//
// What a workgroup loads sets its pace (44 bytes per clock and CU), so a launch is as long as the busiest CU's loads: tiles
// of 96 x 64 and 32 x 64 (bf16; not for weight gradients, whose operands run the other way) fill the gaps between 64 x 64 and
// 32 x 32 where these need one round of the CUs more (see wave_choice in chunk.cpp).
//
// Measured (us per launch, MI355X): bf16 512 x 256 x 1024: 11.6 in one 128 x 128 tile per 8 CUs, 4.1 here; bf16 weight
// gradient 1024 x 1024 x 2048: 26.5 and 12.3; bf16 1527 x 768 x 3072, which only the ALU kernel took: 551 and 20.4;
// fp32 256 x 256 x 1024: 206 on the ALU and 8.1, 2048 x 1024 x 1024: 103 TFLOP/s of the 157 that fp32 MFMAs issue at.
//
// Edges: rows and columns outside the operands are read from inside instead (their products reach only outputs that
// are not stored); what lies past K in the last K tile is overwritten with zeros in LDS once the tile has landed.
//
// A K tile is 128 bytes of a contraction-contiguous row for both types (64 bf16, 32 floats).  LDS tiles are unpadded
// and XOR-swizzled in 16-byte slots; a direct load writes 64 consecutive slots, so the swizzle is applied by choosing
// which vector a lane fetches:
//   contraction-contiguous, [EXT rows][8 slots]:         slot' = slot ^ (row / 2 mod 8): 16 rows at one slot, all banks
//   contraction-strided bf16, [64 k][EXT / 8 slots]:     EXT = 64: slot' = slot ^ 4 (k / 2 mod 2); EXT = 32: none needed
//     (a transpose read takes 4 consecutive k x 4 consecutive slots per half wavefront: all banks)
//   contraction-strided fp32, [32 k][EXT / 4 slots]:     EXT = 64: slot' = slot ^ 8 (k / 4 mod 2): the two half wavefronts
//     read 32 consecutive columns of k and of k + 4
#include <type_traits>

#include "device_util.h"
#include "epilogue.h"
#include "finalize.h"
#include "kernels.h"

namespace hanayo {
namespace k {

namespace {

typedef __attribute__((ext_vector_type(4))) short s16x4;
typedef __attribute__((address_space(3))) s16x4* lds_s16x4_ptr;

constexpr int kMaxGroup = 4;
constexpr int NW = 4;  // wavefronts per workgroup

template <typename T>
struct WaveGemm {
  const T* A;
  const T* B;
  T* C;
  float* Cf;
  const T* bias;
  const T* aux;
  T* aux_out;
  int M, N, K;
  int lda, ldb, ldc;
  float* colsum;  // see GemmArgs
  const int* live;
  int live_dim;
};
template <typename T>
struct WaveGemmGroup {
  WaveGemm<T> prob[kMaxGroup];
  int first[kMaxGroup + 1];  // workgroups first[i] .. first[i + 1] - 1 are the tiles of problem i
  int count;
  FinalizeJob job[kMaxJobs];  // the workgroups behind the tiles: job_blocks of each job
  int job_blocks;
};

// VEC = elements of a 16-byte vector, BK = elements of a K tile (4 MFMA steps), Frag = what a lane feeds per step:
// VEC contraction elements, 2 VEC per step over the two halves of the wavefront.
template <typename T>
struct Prec;
template <>
struct Prec<bf16> {
  static constexpr int VEC = 8, BK = 64;
  typedef bf16x8 Frag;
  __device__ static f32x16 mma(Frag b, Frag a, f32x16 acc) { return __builtin_amdgcn_mfma_f32_32x32x16_bf16(b, a, acc, 0, 0, 0); }
  __device__ static float gelu(float h) { return gelu_fast(h); }
  __device__ static float gelu_grad(float h) { return gelu_grad_fast(h); }
};
template <>
struct Prec<float> {
  static constexpr int VEC = 4, BK = 32;
  typedef f32x4 Frag;
  __device__ static f32x16 mma(Frag b, Frag a, f32x16 acc) {
#pragma unroll
    for (int j = 0; j < 4; ++j) acc = __builtin_amdgcn_mfma_f32_32x32x2f32(b[j], a[j], acc, 0, 0, 0);
    return acc;
  }
  __device__ static float gelu(float h) { return gelu_f(h); }
  __device__ static float gelu_grad(float h) { return gelu_grad_f(h); }
};
constexpr int kSteps = 4;


// Operand tile of EXT rows (columns, if the contraction is strided in memory: TR).
template <typename T, int EXT, bool TR>
struct WaveOperand {
  static constexpr int VEC = Prec<T>::VEC;
  static constexpr int SPR = TR ? EXT / VEC : 8;  // slots per LDS row
  static constexpr int kInstr = EXT / 8;          // wavefront-wide loads per K tile
  static constexpr int kBytes = kInstr * 1024;

  __device__ static int swizzle(int row, int slot) {
    if (!TR) return slot ^ ((row >> 1) & 7);
    if (EXT != 64) return slot;
    return sizeof(T) == 2 ? slot ^ (((row >> 1) & 1) << 2) : slot ^ (((row >> 2) & 1) << 3);
  }
  // Tile row and logical slot of the vector that lands in LDS slot 64 i + lane.
  __device__ static void where(int i, int lane, int& row, int& slot) {
    row = i * (64 / SPR) + lane / SPR;
    slot = swizzle(row, lane % SPR);
  }
  __device__ static bool past_k(int row, int slot, int k_left) { return TR ? row >= k_left : slot * VEC >= k_left; }
  // Byte offset of a vector from the tile's first element; `inside` = rows (columns) of the operand from there on.
  __device__ static unsigned offset(int row, int slot, int ld, int inside) {
    if (TR) return (unsigned)((row * ld + (slot * VEC < inside ? slot * VEC : 0)) * (int)sizeof(T));
    return (unsigned)(((row < inside ? row : inside - 1) * ld + slot * VEC) * (int)sizeof(T));
  }
  // The part of that offset that runs along K: without it the vector lies in the K tile's first row (slot).
  __device__ static unsigned k_part(int row, int slot, int ld) {
    return (unsigned)((TR ? row * ld : slot * VEC) * (int)sizeof(T));
  }
  __device__ static typename Prec<T>::Frag frag(const char* lds, int c0, int step, int lane) {
    if constexpr (!TR) {
      const int row = c0 + (lane & 31), slot = 2 * step + (lane >> 5);
      return *reinterpret_cast<const typename Prec<T>::Frag*>(lds + (row * 8 + swizzle(row, slot)) * 16);
    } else if constexpr (sizeof(T) == 2) {
      const int krow = step * 16 + 8 * (lane >> 5) + ((lane & 15) >> 2);
      const int col = c0 + 16 * ((lane >> 4) & 1) + (lane & 3) * 4;
      // rows krow and krow + 4 have the same swizzle (it looks at bit 1 of the row)
      const char* p = lds + (krow * SPR + swizzle(krow, col >> 3)) * 16 + (col & 7) * 2;
      union {
        struct { s16x4 lo, hi; } s;
        bf16x8 v;
      } u;
      u.s.lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4_ptr)(p));
      u.s.hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4_ptr)(p + 4 * SPR * 16));
      return u.v;
    } else {
      const int krow = step * 8 + 4 * (lane >> 5), col = c0 + (lane & 31);
      const float* p = reinterpret_cast<const float*>(lds + (krow * SPR + swizzle(krow, col >> 2)) * 16) + (col & 3);
      f32x4 v;
#pragma unroll
      for (int j = 0; j < 4; ++j) v[j] = p[j * SPR * 4];
      return v;
    }
  }
};

// Four or eight consecutive elements <-> floats
__device__ __forceinline__ void loadv(const bf16* p, float (&v)[4]) {
  const bf16x4 a = *reinterpret_cast<const bf16x4*>(p);
#pragma unroll
  for (int i = 0; i < 4; ++i) v[i] = (float)a[i];
}
__device__ __forceinline__ void storev(bf16* p, const float (&v)[4]) {
  bf16x4 a;
#pragma unroll
  for (int i = 0; i < 4; ++i) a[i] = (bf16)v[i];
  *reinterpret_cast<bf16x4*>(p) = a;
}
__device__ __forceinline__ void loadv(const bf16* p, float (&v)[8]) { load8_row(p, v); }
__device__ __forceinline__ void loadv(const float* p, float (&v)[8]) { load8(p, v); }
__device__ __forceinline__ void loadv(const float* p, float (&v)[4]) {
  const f32x4 a = *reinterpret_cast<const f32x4*>(p);
#pragma unroll
  for (int i = 0; i < 4; ++i) v[i] = a[i];
}
__device__ __forceinline__ void storev(bf16* p, const float (&v)[8]) { store8_row(p, v); }
__device__ __forceinline__ void storev(float* p, const float (&v)[8]) { store8(p, v); }
__device__ __forceinline__ void storev(float* p, const float (&v)[4]) {
  f32x4 a;
#pragma unroll
  for (int i = 0; i < 4; ++i) a[i] = v[i];
  *reinterpret_cast<f32x4*>(p) = a;
}

template <int BM, int BN>
constexpr size_t wave_lds_bytes(int nst) {
  const size_t ring = (size_t)NW * nst * (BM + BN) / 8 * 1024, parts = (size_t)NW * BM * (BN + 4) * 4 + 2 * NW * BN * 4;
  return ring > parts ? ring : parts;
}

// NST = stages of a wavefront's ring.  One (64 KiB of LDS at 64 x 64: two workgroups per CU, whose wavefronts cover each
// other's waits) for launches with more tiles than CUs, two for launches of at most one tile per CU.  Even with one
// stage the next tile's loads run under the MFMAs of this one: its fragments are in registers by then.
template <typename T, int BM, int BN, int NST, bool A_T, bool B_T, int EPI>
__device__ __forceinline__ void gemm_wave_body(WaveGemm<T> p, int wg) {
  using P = Prec<T>;
  using OpA = WaveOperand<T, BM, A_T>;
  using OpB = WaveOperand<T, BN, B_T>;
  using Frag = typename P::Frag;
  constexpr int TM = BM / 32, TN = BN / 32, VEC = P::VEC, BK = P::BK;
  constexpr int STAGE = OpA::kBytes + OpB::kBytes, LOADS = OpA::kInstr + OpB::kInstr;
  if (p.live_dim) {
    const int live = __builtin_amdgcn_readfirstlane(*p.live);
    if (live < 1) return;
    if (p.live_dim == LIVE_K) p.K = live;
    else p.M = live;
    if (wg >= (p.M + BM - 1) / BM * ((p.N + BN - 1) / BN)) return;
  }
  extern __shared__ __attribute__((aligned(1024))) char smem[];
  const unsigned lds0 = (unsigned)(unsigned long)((__attribute__((address_space(3))) char*)smem);
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  int tile_m, tile_n;
  xcd_tile(wg, (p.M + BM - 1) / BM, (p.N + BN - 1) / BN, tile_m, tile_n);
  const int m0 = __builtin_amdgcn_readfirstlane(tile_m) * BM, n0 = __builtin_amdgcn_readfirstlane(tile_n) * BN;
  const int nk = (p.K + BK - 1) / BK, k_tail = p.K - (nk - 1) * BK;  // k_tail = BK: the last K tile is whole

  // The operand an epilogue reads is fetched first of all, from clamped places (what is outside is not stored).
  constexpr int OV = BM * BN / (NW * 64) < VEC ? BM * BN / (NW * 64) : VEC;  // elements of an output vector
  constexpr int kVecPerRow = BN / OV, kOut = BM * kVecPerRow / (NW * 64);
  static_assert(BM * kVecPerRow % (NW * 64) == 0 && (NW * 64) % kVecPerRow == 0, "outputs divide among the threads");
  constexpr bool kBias = EPI == EPI_BIAS || EPI == EPI_BIAS_GELU || EPI == EPI_BIAS_RES;
  constexpr bool kReadsAux = EPI == EPI_BIAS_RES || EPI == EPI_ADD || EPI == EPI_MUL_DGELU;
  constexpr bool kReadsC = EPI == EPI_ACCUM_F32;
  const int col = (threadIdx.x % kVecPerRow) * OV, row0 = threadIdx.x / kVecPerRow;
  constexpr int kRowStep = NW * 64 / kVecPerRow;
  const int n = n0 + col, n_in = n < p.N ? n : 0;
  float pre[kReadsAux || kReadsC ? kOut : 1][OV], bias[OV];
  if constexpr (kReadsAux || kReadsC) {
#pragma unroll
    for (int u = 0; u < kOut; ++u) {
      const int m = m0 + row0 + u * kRowStep;
      const size_t at = (size_t)(m < p.M ? m : p.M - 1) * p.ldc + n_in;
      if constexpr (kReadsAux) loadv(p.aux + at, pre[u]);
      else loadv(p.Cf + at, pre[u]);
    }
  }
  if constexpr (kBias) loadv(p.bias + n_in, bias);

  unsigned voff_a[OpA::kInstr], voff_b[OpB::kInstr];
#pragma unroll
  for (int i = 0; i < OpA::kInstr; ++i) {
    int row, slot;
    OpA::where(i, lane, row, slot);
    voff_a[i] = OpA::offset(row, slot, p.lda, p.M - m0);
  }
#pragma unroll
  for (int i = 0; i < OpB::kInstr; ++i) {
    int row, slot;
    OpB::where(i, lane, row, slot);
    voff_b[i] = OpB::offset(row, slot, p.ldb, p.N - n0);
  }
  const size_t a_step = (A_T ? (size_t)BK * p.lda : (size_t)BK), b_step = (B_T ? (size_t)BK * p.ldb : (size_t)BK);
  const T* a_next = (A_T ? p.A + m0 : p.A + (size_t)m0 * p.lda) + wave * a_step;
  const T* b_next = (B_T ? p.B + n0 : p.B + (size_t)n0 * p.ldb) + wave * b_step;
  const unsigned ring = lds0 + wave * NST * STAGE;
  const char* ring_ptr = smem + wave * NST * STAGE;
  const int mine = nk > wave ? (nk - wave + NW - 1) / NW : 0;  // K tiles of this wavefront
  auto issue = [&](int j) {
    const unsigned st = ring + (NST == 1 ? 0 : (unsigned)(j % NST) * STAGE);
    const bool partial = k_tail < BK && wave + j * NW == nk - 1;
#pragma unroll
    for (int i = 0; i < OpA::kInstr; ++i) {
      unsigned v = voff_a[i];
      if (partial) {
        int row, slot;
        OpA::where(i, lane, row, slot);
        if (OpA::past_k(row, slot, k_tail)) v -= OpA::k_part(row, slot, p.lda);
      }
      dma16(a_next, v, st + i * 1024);
    }
#pragma unroll
    for (int i = 0; i < OpB::kInstr; ++i) {
      unsigned v = voff_b[i];
      if (partial) {
        int row, slot;
        OpB::where(i, lane, row, slot);
        if (OpB::past_k(row, slot, k_tail)) v -= OpB::k_part(row, slot, p.ldb);
      }
      dma16(b_next, v, st + OpA::kBytes + i * 1024);
    }
    a_next += NW * a_step;
    b_next += NW * b_step;
  };
  auto clear_past_k = [&](const char* st) {
    const f32x4 z = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int i = 0; i < OpA::kInstr; ++i) {
      int row, slot;
      OpA::where(i, lane, row, slot);
      if (OpA::past_k(row, slot, k_tail)) *reinterpret_cast<f32x4*>(const_cast<char*>(st) + (i * 64 + lane) * 16) = z;
    }
#pragma unroll
    for (int i = 0; i < OpB::kInstr; ++i) {
      int row, slot;
      OpB::where(i, lane, row, slot);
      if (OpB::past_k(row, slot, k_tail))
        *reinterpret_cast<f32x4*>(const_cast<char*>(st) + OpA::kBytes + (i * 64 + lane) * 16) = z;
    }
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
  };

#pragma unroll
  for (int j = 0; j < NST; ++j)
    if (j < mine) issue(j);

  f32x16 acc[TM][TN], csum[TN];  // fp32: csum[j][0] only
#pragma unroll
  for (int j = 0; j < TN; ++j)
#pragma unroll
    for (int r = 0; r < 16; ++r) {
#pragma unroll
      for (int i = 0; i < TM; ++i) acc[i][j][r] = 0.f;
      csum[j][r] = 0.f;
    }
  // Column sums of B (the bias gradient), by the workgroups of the first tile row: in bf16 they multiply their B fragments
  // by ones; in fp32, where that takes half as many MFMAs again (29.7 us against 23.4 without column sums for 512 x 2048 x
  // 1024), every lane adds up what it holds of its column.
  const bool sums_columns = kReadsC && p.colsum && m0 == 0;
  Frag ones;
#pragma unroll
  for (int e = 0; e < VEC; ++e) ones[e] = (T)1.0f;

  for (int j = 0; j < mine; ++j) {
    if (NST > 1 && j + 1 < mine) wait_vmcnt<LOADS>();
    else wait_vmcnt<0>();
    const char* st = ring_ptr + (NST == 1 ? 0 : (j % NST) * STAGE);
    if (k_tail < BK && wave + j * NW == nk - 1) clear_past_k(st);
    Frag fa[kSteps][TM], fb[kSteps][TN];
#pragma unroll
    for (int s = 0; s < kSteps; ++s) {
#pragma unroll
      for (int i = 0; i < TM; ++i) fa[s][i] = OpA::frag(st, i * 32, s, lane);
#pragma unroll
      for (int i = 0; i < TN; ++i) fb[s][i] = OpB::frag(st + OpA::kBytes, i * 32, s, lane);
    }
    __builtin_amdgcn_sched_barrier(0);
    auto steps = [&](int s0, int s1) {
#pragma unroll
      for (int s = s0; s < s1; ++s)
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
          for (int jn = 0; jn < TN; ++jn) acc[i][jn] = P::mma(fb[s][jn], fa[s][i], acc[i][jn]);
    };
    steps(0, 2);
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");  // the stage has been read: it takes the next tile
    __builtin_amdgcn_sched_barrier(0);
    if (j + NST < mine) issue(j + NST);
    steps(2, kSteps);
    if constexpr (kReadsC) {
      if (sums_columns) {
#pragma unroll
        for (int s = 0; s < kSteps; ++s)
#pragma unroll
          for (int jn = 0; jn < TN; ++jn) {
            if constexpr (sizeof(T) == 2) csum[jn] = P::mma(fb[s][jn], ones, csum[jn]);
            else csum[jn][0] += (fb[s][jn][0] + fb[s][jn][1]) + (fb[s][jn][2] + fb[s][jn][3]);
          }
      }
    }
  }

  // Partial tiles to LDS (a lane holds columns 8 q + 4 (lane / 32) .. + 3 of row lane % 32), then every thread adds the
  // four of its output vectors in order.
  constexpr int EP = BN + 4;
  float* parts = reinterpret_cast<float*>(smem);
  float* cparts = parts + NW * BM * EP;
  __syncthreads();  // the rings are no longer read
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        f32x4 v;
#pragma unroll
        for (int e = 0; e < 4; ++e) v[e] = acc[i][j][4 * q + e];
        *reinterpret_cast<f32x4*>(parts + (wave * BM + i * 32 + (lane & 31)) * EP + j * 32 + 8 * q + 4 * (lane >> 5)) = v;
      }
  if constexpr (kReadsC) {
    if (sizeof(T) == 4 && sums_columns) {
#pragma unroll
      for (int j = 0; j < TN; ++j) cparts[(wave * 2 + (lane >> 5)) * BN + j * 32 + (lane & 31)] = csum[j][0];
    }
    if (sizeof(T) == 2 && sums_columns && (lane & 31) == 0) {
#pragma unroll
      for (int j = 0; j < TN; ++j)
#pragma unroll
        for (int r = 0; r < 16; ++r) cparts[wave * BN + j * 32 + 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3)] = csum[j][r];
    }
  }
  __syncthreads();
  if constexpr (kReadsC) {
    if (sums_columns && (int)threadIdx.x < BN && n0 + (int)threadIdx.x < p.N) {
      float t = 0.f;
#pragma unroll
      for (int w = 0; w < (sizeof(T) == 4 ? 2 * NW : NW); ++w) t += cparts[w * BN + threadIdx.x];
      p.colsum[n0 + threadIdx.x] += t;
    }
  }
#pragma unroll
  for (int u = 0; u < kOut; ++u) {
    const int row = row0 + u * kRowStep, m = m0 + row;
    float v[OV];
    loadv(parts + row * EP + col, v);
#pragma unroll
    for (int w = 1; w < NW; ++w) {
      float t[OV];
      loadv(parts + (w * BM + row) * EP + col, t);
#pragma unroll
      for (int e = 0; e < OV; ++e) v[e] += t[e];
    }
    if (m >= p.M || n >= p.N) continue;
    const size_t at = (size_t)m * p.ldc + n;
    if constexpr (kReadsC) {
#pragma unroll
      for (int e = 0; e < OV; ++e) v[e] += pre[u][e];
      storev(p.Cf + at, v);
    } else {
      if constexpr (kBias) {
#pragma unroll
        for (int e = 0; e < OV; ++e) v[e] += bias[e];
      }
      if constexpr (EPI == EPI_BIAS_RES || EPI == EPI_ADD) {
#pragma unroll
        for (int e = 0; e < OV; ++e) v[e] += pre[u][e];
      }
      if constexpr (EPI == EPI_MUL_DGELU) {
#pragma unroll
        for (int e = 0; e < OV; ++e) v[e] *= P::gelu_grad(pre[u][e]);
      }
      if constexpr (EPI == EPI_BIAS_GELU) {
        storev(p.aux_out + at, v);
#pragma unroll
        for (int e = 0; e < OV; ++e) v[e] = P::gelu(v[e]);
      }
      storev(p.C + at, v);
    }
  }
}

// Weight gradients come with others of theirs and with jobs, other products in groups only where a caller sends them so: a single
// one is passed by itself.  Its fields are where the kernel expects them without a search, and a quarter of the bytes goes
// through the launch (1 us of host time).  Groups: four of 512 x 512 x 512 with a bias 5.3 us, one after the other 14.2; two of 2048 x
// 1024 x 1024 13.4 and 18.3.  The first 14 words of a kernel's arguments are in scalar registers when it starts (see the build
// flags); what the first loads depend on stands there, and live_dim with ldc, so that nothing at the start waits for the argument
// block in memory (0.3 us).
template <typename T, int BM, int BN, int NST, bool A_T, bool B_T, int EPI>
__global__ __launch_bounds__(NW * 64) void gemm_wave_kernel(const T* A, const T* B, T* C, const T* bias, int M, int N, int K,
                                                            int lda, int ldb, unsigned ldc_live, const T* aux, T* aux_out,
                                                            const int* live) {
  WaveGemm<T> p;
  p.A = A; p.B = B; p.C = C; p.Cf = nullptr; p.bias = bias; p.aux = aux; p.aux_out = aux_out;
  p.M = M; p.N = N; p.K = K; p.lda = lda; p.ldb = ldb; p.ldc = ldc_of(ldc_live);
  p.colsum = nullptr; p.live = live; p.live_dim = live_dim_of(ldc_live);
  gemm_wave_body<T, BM, BN, NST, A_T, B_T, EPI>(p, (int)blockIdx.x);
}
template <typename T, int BM, int BN, int NST, bool A_T, bool B_T, int EPI>
__global__ __launch_bounds__(NW * 64) void gemm_wave_group_kernel(WaveGemmGroup<T> grp) {
  if (EPI == EPI_ACCUM_F32 && (int)blockIdx.x >= grp.first[kMaxGroup]) {
    extern __shared__ __attribute__((aligned(1024))) char smem[];
    const int at = (int)blockIdx.x - grp.first[kMaxGroup], second = at >= grp.job_blocks;
    finalize_columns<NW * 64, 4>(grp.job[second], at - second * grp.job_blocks, smem);
    return;
  }
  int gi = 0;
#pragma unroll
  for (int j = 1; j < kMaxGroup; ++j)
    if (j < grp.count && (int)blockIdx.x >= grp.first[j]) gi = j;
  gemm_wave_body<T, BM, BN, NST, A_T, B_T, EPI>(grp.prob[gi], (int)blockIdx.x - grp.first[gi]);
}

template <typename T, int BM, int BN, int NST, bool A_T, bool B_T, int EPI>
int launch(WaveGemmGroup<T>& grp, unsigned workgroups, hipStream_t stream) {
  constexpr size_t lds = wave_lds_bytes<BM, BN>(NST);
  if constexpr (BM == BN) {
    if (EPI == EPI_ACCUM_F32 || grp.count > 1) {
      static thread_local uint64_t raised = 0;
      auto kern = gemm_wave_group_kernel<T, BM, BN, NST, A_T, B_T, EPI>;
      if (const int rc = raise_lds(reinterpret_cast<const void*>(kern), lds, raised)) return rc;
      launch_kernel(kern, dim3(workgroups), dim3(NW * 64), lds, stream, grp);
      return check_launch("gemm_wave");
    }
  }
  if constexpr (EPI != EPI_ACCUM_F32) {
    static thread_local uint64_t raised = 0;
    auto kern = gemm_wave_kernel<T, BM, BN, NST, A_T, B_T, EPI>;
    if (const int rc = raise_lds(reinterpret_cast<const void*>(kern), lds, raised)) return rc;
    const WaveGemm<T>& p = grp.prob[0];
    launch_kernel(kern, dim3(workgroups), dim3(NW * 64), lds, stream, p.A, p.B, p.C, p.bias, p.M, p.N, p.K, p.lda, p.ldb,
                       pack_ldc(p.ldc, p.live_dim), p.aux, p.aux_out, p.live);
  }
  return check_launch("gemm_wave");
}

template <typename T, int BM, int BN, int NST>
int launch_layout(const GemmArgs& g, WaveGemmGroup<T>& grp, unsigned workgroups, hipStream_t stream) {
  if (!g.a_t && g.b_t) {
    switch (g.epi) {
      case EPI_NONE: return launch<T, BM, BN, NST, false, true, EPI_NONE>(grp, workgroups, stream);
      case EPI_BIAS: return launch<T, BM, BN, NST, false, true, EPI_BIAS>(grp, workgroups, stream);
      case EPI_BIAS_GELU: return launch<T, BM, BN, NST, false, true, EPI_BIAS_GELU>(grp, workgroups, stream);
      case EPI_BIAS_RES: return launch<T, BM, BN, NST, false, true, EPI_BIAS_RES>(grp, workgroups, stream);
      default: break;
    }
  } else if (!g.a_t && !g.b_t) {
    switch (g.epi) {
      case EPI_NONE: return launch<T, BM, BN, NST, false, false, EPI_NONE>(grp, workgroups, stream);
      case EPI_MUL_DGELU: return launch<T, BM, BN, NST, false, false, EPI_MUL_DGELU>(grp, workgroups, stream);
      case EPI_ADD: return launch<T, BM, BN, NST, false, false, EPI_ADD>(grp, workgroups, stream);
      default: break;
    }
  } else if (g.a_t && g.b_t && g.epi == EPI_ACCUM_F32) {
    if constexpr (BM == BN) return launch<T, BM, BN, NST, true, true, EPI_ACCUM_F32>(grp, workgroups, stream);
  }
  return set_error(HANAYO_EUNSUPPORTED, "gemm_wave: layout/epilogue combination not built");
}


template <typename T>
int group_t(const GemmArgs* gs, int count, WaveTile tile, hipStream_t stream, const FinalizeJob* jobs, int n_jobs) {
  int bm, bn;
  wave_tile(tile, bm, bn);
  WaveGemmGroup<T> grp{};
  grp.count = count;
  long tiles = 0;
  for (int i = 0; i < count; ++i) {
    const GemmArgs& g = gs[i];
    WaveGemm<T>& p = grp.prob[i];
    p.A = (const T*)g.A; p.B = (const T*)g.B; p.C = (T*)g.C; p.Cf = (float*)g.C;
    p.bias = (const T*)g.bias; p.aux = (const T*)g.aux; p.aux_out = (T*)g.aux_out;
    p.M = g.M; p.N = g.N; p.K = g.K; p.lda = g.lda; p.ldb = g.ldb; p.ldc = g.ldc;
    p.colsum = g.epi == EPI_ACCUM_F32 ? g.colsum : nullptr;
    p.live = g.live; p.live_dim = g.live ? g.live_dim : LIVE_NONE;
    grp.first[i] = (int)tiles;
    tiles += (long)((g.M + bm - 1) / bm) * ((g.N + bn - 1) / bn);
  }
  for (int i = count; i <= kMaxGroup; ++i) grp.first[i] = (int)tiles;
  if (tiles > 0x7fff0000L) return set_error(HANAYO_EUNSUPPORTED, "gemm_wave: too many tiles");
  for (int i = 0; i < n_jobs; ++i) {
    grp.job[i] = jobs[i];
    const int blocks = finalize_blocks(jobs[i], finalize_cols<NW * 64, 4>());
    if (blocks > grp.job_blocks) grp.job_blocks = blocks;
  }
  const unsigned workgroups = (unsigned)(tiles + (long)n_jobs * grp.job_blocks);
  if (tile == WAVE_32x32) return launch_layout<T, 32, 32, 2>(gs[0], grp, workgroups, stream);
  if constexpr (sizeof(T) == 2) {
    if (tile == WAVE_96x64) return launch_layout<T, 96, 64, 2>(gs[0], grp, workgroups, stream);  // one to a CU either way
    if (tile == WAVE_32x64)
      return tiles > 256 ? launch_layout<T, 32, 64, 1>(gs[0], grp, workgroups, stream) : launch_layout<T, 32, 64, 2>(gs[0], grp, workgroups, stream);
  }
  return tiles > 256 ? launch_layout<T, 64, 64, 1>(gs[0], grp, workgroups, stream)
                     : launch_layout<T, 64, 64, 2>(gs[0], grp, workgroups, stream);
}

}  // namespace

// 16-byte vectors never straddle the end of a row and, in A and B, start on 16-byte boundaries (in C: see epilogue.h); lane
// offsets are 32-bit.
bool gemm_wave_supported(int dtype, const GemmArgs& g) {
  const int vec = dtype == HANAYO_BF16 ? 8 : 4, esz = dtype == HANAYO_BF16 ? 2 : 4;
  const bool combo = (!g.a_t && g.b_t && (g.epi == EPI_NONE || g.epi == EPI_BIAS || g.epi == EPI_BIAS_GELU || g.epi == EPI_BIAS_RES)) ||
                     (!g.a_t && !g.b_t && (g.epi == EPI_NONE || g.epi == EPI_MUL_DGELU || g.epi == EPI_ADD)) ||
                     (g.a_t && g.b_t && g.epi == EPI_ACCUM_F32);
  if (!combo || (g.colsum && g.epi != EPI_ACCUM_F32) || (g.live && g.live_dim == LIVE_M_SPLIT)) return false;
  const uintptr_t bits = (uintptr_t)g.A | (uintptr_t)g.B | (uintptr_t)g.C | (uintptr_t)g.bias | (uintptr_t)g.aux | (uintptr_t)g.aux_out;
  return bits % 16 == 0 && (g.a_t ? g.M : g.K) % vec == 0 && (g.b_t ? g.N : g.K) % vec == 0 && g.N % vec == 0 && g.lda % vec == 0 &&
         g.ldb % vec == 0 && g.ldc % 4 == 0 && (long)64 * g.lda * esz < (1L << 31) && (long)64 * g.ldb * esz < (1L << 31);
}

// A lane's offset reaches over the tile's rows where they are contiguous along the contraction; 64 rows are always within bounds.
bool gemm_wave_tile_fits(WaveTile t, int dtype, const GemmArgs& g) {
  int bm, bn;
  wave_tile(t, bm, bn);
  return g.a_t || bm <= 64 || (long)bm * g.lda * (dtype == HANAYO_BF16 ? 2 : 4) < (1L << 31);
}

int gemm_wave_group(int dtype, const GemmArgs* gs, int count, WaveTile tile, hipStream_t stream, const FinalizeJob* jobs, int n_jobs) {
  if (n_jobs < 0 || n_jobs > kMaxJobs || (n_jobs && gs[0].epi != EPI_ACCUM_F32)) return set_error(HANAYO_EINVAL, "gemm_wave: %d jobs", n_jobs);
  if (count < 1 || count > kMaxGroup || tile == WAVE_NONE) return set_error(HANAYO_EINVAL, "gemm_wave: group of %d", count);
  if (tile != WAVE_64x64 && tile != WAVE_32x32 && (dtype != HANAYO_BF16 || gs[0].epi == EPI_ACCUM_F32 || count > 1))
    return set_error(HANAYO_EUNSUPPORTED, "gemm_wave: tile not built");
  for (int i = 0; i < count; ++i)
    if (!gemm_wave_supported(dtype, gs[i]) || !gemm_wave_tile_fits(tile, dtype, gs[i]) || gs[i].a_t != gs[0].a_t || gs[i].b_t != gs[0].b_t || gs[i].epi != gs[0].epi)
      return set_error(HANAYO_EUNSUPPORTED, "gemm_wave: shape not supported");
  return dtype == HANAYO_BF16 ? group_t<bf16>(gs, count, tile, stream, jobs, n_jobs) : group_t<float>(gs, count, tile, stream, jobs, n_jobs);
}

}  // namespace k
}  // namespace hanayo
