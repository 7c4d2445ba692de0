// bf16 GEMM in large tiles: operand tiles go from global memory straight into LDS (global_load_lds_dwordx4, no VGPR
// staging and no LDS write instructions), through a ring of NSTAGE LDS buffers of 64-wide K tiles, so that loads for
// tiles t+1 .. t+NSTAGE-1 are in flight while tile t is multiplied.  One workgroup barrier per K tile.
//
// LDS layouts are unpadded and XOR-swizzled in units of 16 bytes ("slots"); a direct load writes 64 consecutive slots
// per wavefront instruction, so the swizzle is applied by choosing which global vector each lane fetches:
//   * contraction-contiguous operand, tile [rows][64]: 8 slots per row, slot' = slot ^ ((row >> 1) & 7)
//       (16-byte fragment reads of 16 consecutive rows then cover all 64 banks)
//   * contraction-strided operand, tile [64][cols]: cols/8 slots per row, slot' = slot ^ ((row & 3) << 2 | (row >> 3 & 1) << 1)
//       (the 8 rows x 2 slots one half wavefront touches in a transpose read cover all 64 banks)
//
// The matrix instruction is the 16x16x32 one.  What bounds the large launches is the chip's power: on random operands in
// registers, eight wavefronts per CU, 16x16x32 sustains 2055 TFLOP/s and 32x32x16 1823 (both issue 2500 at full clock).
// With 32x32x16 in this kernel: 8192^3 1340 TFLOP/s, now 1425; 4096 x 1024 x 4096 40.2 -> 34.5 us, 2048 x 10240 x 2560
// (160 tiles) 134 -> 132 us, 2048 x 16384 x 4096 233 -> 224 us, one after the other on one chip in its sustained state.
// The MFMAs compute the transposed tile, so a lane holds 4 consecutive columns of one row.  The epilogue goes through
// LDS (the idle load ring) so that stores are whole rows; a launch may carry several problems of one layout
// (DmaGemmGroup); workgroups take their tiles in an XCD-aware order (xcd_tile).
//
// EDGE kernels take any extents whose rows are whole 16-byte vectors: rows and columns outside the operands are read
// from inside instead (their products reach only outputs that are not stored), and what lies past K in the last K
// tile is overwritten with zeros in LDS by the wavefront that loaded it, before the barrier that admits the tile.
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
typedef __attribute__((address_space(3))) const bf16x8* lds_bf16x8_ptr;

struct DmaGemm {
  const bf16* A;
  const bf16* B;
  bf16* C;
  float* Cf;
  const bf16* bias;
  const bf16* aux;
  bf16* aux_out;
  int M, N, K;
  int lda, ldb, ldc;
  float* colsum;  // see GemmArgs; folded into the weight-gradient kernels
  const int* live;  // see GemmArgs; EDGE kernels only
  int live_dim;
};

// One launch covers up to kMaxGroup independent problems of one layout and epilogue: workgroups
// first[i] .. first[i + 1] - 1 are the tiles of problem i.  Four weight-gradient GEMMs of a block,
// none of which fills the chip alone, share one grid this way.
constexpr int kMaxGroup = 4;
struct DmaGemmGroup {
  DmaGemm prob[kMaxGroup];
  int first[kMaxGroup + 1];
  int count;
  FinalizeJob job[kMaxJobs];  // the workgroups behind the tiles: job_blocks of each of n_jobs jobs
  int n_jobs, job_blocks;
};

constexpr int kGeluN = 2048;  // intervals of the GELU epilogues' table

constexpr int kBK = 64;       // K tile
constexpr int KS = kBK / 32;  // MFMA steps per K tile

// Waits until at most `tiles_in_flight` tiles (0 to 2, LOADS instructions each) are still outstanding.
template <int LOADS>
__device__ __forceinline__ void wait_tiles(int tiles_in_flight) {
  switch (tiles_in_flight) {
    case 0: wait_vmcnt<0>(); break;
    case 1: wait_vmcnt<LOADS>(); break;
    default: wait_vmcnt<2 * LOADS>(); break;
  }
}

// Operand tile description.  T = contraction strided in memory (tile is [kBK][EXT]).
template <int EXT, bool T, int NW>
struct Operand {
  static constexpr int kSlotsPerRow = T ? EXT / 8 : kBK / 8;
  static constexpr int kRows = T ? kBK : EXT;
  static constexpr int kBytes = kRows * kSlotsPerRow * 16;
  static constexpr int kInstr = kBytes / 1024;      // wavefront-wide loads per tile
  static constexpr int kPerWave = kInstr / NW;      // issued by each wavefront
  static_assert(kInstr % NW == 0, "tile loads must divide evenly over the wavefronts");

  __device__ static int swizzle(int row, int slot) {
    return T ? slot ^ ((row & 3) << 2 | (row >> 3 & 1) << 1) : slot ^ ((row >> 1) & 7);
  }
  // Tile row and logical slot of the vector that lands in LDS slot 64 q + lane.
  __device__ static void where(int q, int lane, int& row, int& slot) {
    const int at = q * 64 + lane;
    row = at / kSlotsPerRow;
    slot = swizzle(row, at % kSlotsPerRow);
  }
  // Byte offset of that vector from the tile's first element; EDGE: `inside` rows (columns) of the operand are left
  // from there on.
  template <bool EDGE>
  __device__ static unsigned offset(int q, int lane, int ld, int inside) {
    int row, slot;
    where(q, lane, row, slot);
    if (EDGE) {
      if (T) slot = slot * 8 < inside ? slot : 0;
      else row = row < inside ? row : inside - 1;
    }
    return (unsigned)((row * ld + slot * 8) * 2);
  }
  // Is the vector past the last of k_left contraction elements?  Then it is fetched from the K tile's first row (slot).
  __device__ static bool past_k(int q, int lane, int k_left) {
    int row, slot;
    where(q, lane, row, slot);
    return (T ? row : slot * 8) >= k_left;
  }
  __device__ static unsigned k_part(int q, int lane, int ld) {
    int row, slot;
    where(q, lane, row, slot);
    return (unsigned)((T ? row * ld : slot * 8) * 2);
  }
  // What a lane feeds to one 16x16x32 MFMA step: row (column) 16 i + lane % 16 of the wavefront's share, contraction
  // elements 32 kk + 8 (lane / 16) .. + 7.  lane_at is where that is for i = kk = 0, in bytes from the tile's start, which
  // is a multiple of 1024; i and kk then only flip or add bits, so one register addresses every fragment of the operand.
  __device__ static unsigned lane_at(int first, int lane) {
    if (T) {
      const int row = 8 * (lane >> 4) + ((lane & 15) >> 2), col = first + (lane & 3) * 4;
      return (unsigned)((row * kSlotsPerRow + swizzle(row, col >> 3)) * 16 + (col & 7) * 2);
    }
    const int row = first + (lane & 15);
    return (unsigned)((row * kSlotsPerRow + swizzle(row, lane >> 4)) * 16);
  }
  __device__ static bf16x8 frag(unsigned at, int i, int kk) {
    if constexpr (T) {
      const unsigned p = (at ^ (unsigned)(i * 32)) + kk * 32 * kSlotsPerRow * 16;
      union {
        struct { s16x4 lo, hi; } s;
        bf16x8 v;
      } u;
      u.s.lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4_ptr)p);
      u.s.hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4_ptr)(p + 4 * kSlotsPerRow * 16));  // same swizzle
      return u.v;
    } else {
      return *(lds_bf16x8_ptr)((at ^ (unsigned)(kk * 64)) + i * 16 * kSlotsPerRow * 16);
    }
  }
};


// wg: tile number within the problem
template <int BM, int BN, int WGM, int WGN, int NSTAGE, bool A_T, bool B_T, int EPI, bool EDGE>
__device__ __forceinline__ void gemm_dma_body(DmaGemm p, int wg) {
  // A launch over rows counted on the device may have fewer workgroups than tiles (see launch): they take several each.
  // (By goto: with the tile's code in a function and a loop around it the other instances, which never loop, are scheduled
  // worse and one spills: 2048 x 16384 x 4096 with GELU' 222 -> 229 us.  With the goto only the 256 x 256 instance that loops
  // spills, 10 registers, 44 bytes per lane; with the function it does not, and the head of 460 rows x 30592 columns takes 201
  // us instead of 208.)
  constexpr bool kLoop = EDGE && EPI == EPI_NONE && !B_T;
  int step = 0, tiles_end = 0;
  if (EDGE && p.live_dim) {
    const int live = __builtin_amdgcn_readfirstlane(*p.live);
    if (live < 1) return;
    if (p.live_dim == LIVE_K) {
      p.K = live;
    } else {
      p.M = live;
      const int tiles_n = (p.N + BN - 1) / BN, tiles = (live + BM - 1) / BM * tiles_n;
      if (EPI == EPI_STORE_F32 && p.live_dim == LIVE_M_SPLIT) {
        int per;
        const int slices = split_plan(live, tiles_n, p.K, (int)gridDim.x, per), slice = wg / tiles;
        if (slice >= slices) return;
        wg -= slice * tiles;
        p.A += A_T ? (size_t)slice * per * p.lda : (size_t)slice * per;
        p.B += B_T ? (size_t)slice * per * p.ldb : (size_t)slice * per;
        p.Cf += (size_t)slice * live * p.ldc;
        p.K = min(per, p.K - slice * per);
      } else if (wg >= tiles) {
        return;
      }
      if (kLoop) step = (int)gridDim.x, tiles_end = tiles;
    }
  }
  constexpr int NW = WGM * WGN;                    // wavefronts in the workgroup
  constexpr int WM = BM / WGM, WN = BN / WGN, TM = WM / 16, TN = WN / 16;
  using OpA = Operand<BM, A_T, NW>;
  using OpB = Operand<BN, B_T, NW>;
  constexpr int STAGE_BYTES = OpA::kBytes + OpB::kBytes;
  constexpr int LOADS = OpA::kPerWave + OpB::kPerWave;  // per thread per tile
  static_assert((NSTAGE - 1) * LOADS <= 63, "vmcnt range");

  extern __shared__ __attribute__((aligned(1024))) char smem[];
  // LDS byte address of the ring (address-space-3 offset, what M0 takes)
  const unsigned lds0 = (unsigned)(unsigned long)((__attribute__((address_space(3))) char*)smem);

  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wm = wave / WGN, wn = wave % WGN;
next_tile:
  const int tiles_m = EDGE ? (p.M + BM - 1) / BM : p.M / BM, tiles_n = EDGE ? (p.N + BN - 1) / BN : p.N / BN;
  int tile_m, tile_n;
  // 256 x 128: patches of 1024 x 1024 outputs per XCD instead of 2048 x 512.  Steps with four and two lanes: H = 4096 164.6 ->
  // 164.0 ms, H = 2560 47.6 -> 46.2 ms (with band 8 in the same runs 164.5 and 47.5).
  xcd_tile<BM == 2 * BN ? 4 : 8>(wg, tiles_m, tiles_n, tile_m, tile_n);
  tile_m = __builtin_amdgcn_readfirstlane(tile_m);
  tile_n = __builtin_amdgcn_readfirstlane(tile_n);
  const int m0 = tile_m * BM, n0 = tile_n * BN;
  const int nk = EDGE ? (p.K + kBK - 1) / kBK : p.K / kBK;
  const int k_tail = EDGE ? p.K - (nk - 1) * kBK : kBK;  // contraction elements of the last K tile

  // GELU epilogues: Phi (forward) or GELU' (input gradient of FC2) comes from a table of kGeluN intervals over [-8, 8) behind
  // the ring, made with erff and read with linear interpolation (error below 1e-5, far under bf16 rounding).  It is made
  // while the first K tiles are on their way, each thread a run of neighbouring intervals, whose ends they share; between main
  // loop and epilogue, every end twice, it held up each tile: FC1 / FC2's input gradient 777 x 2560 x 640 13.5 / 12.1 us a launch
  // then and 12.5 / 11.0 now, 1527 x 3072 x 768 18.0 / 16.3 and 17.2 / 15.2, 4096 x 4096 x 1024 39.0 / 36.4 and 37.9 / 35.3.
  // Its 16 KiB stand behind the ring instead of in it: 256 x 256 tiles take 144 KiB and, as before, all registers of a CU; 256 x 128
  // tiles 160, beside which only kernels without LDS run; 128 x 128 tiles 80 (two on a CU, as before) and, with three stages, 112, beside
  // which another lane's 64 KiB no longer fit.  Steps of 18 shapes with two to four lanes, H = 512 - 2560, take 0.98 - 1.005 of
  // the time with the table in the ring.
  constexpr bool kGelu = EPI == EPI_BIAS_GELU || EPI == EPI_MUL_DGELU;
  float2* gelu_tab = reinterpret_cast<float2*>(smem + NSTAGE * STAGE_BYTES);
  auto build_table = [&]() {
    if constexpr (kGelu) {
      constexpr int PER = kGeluN / (NW * 64);  // neighbouring intervals of a thread
      auto value = [](int k) {
        const float x = -8.f + (float)k * (1.f / 128.f);
        return EPI == EPI_BIAS_GELU ? 0.5f * (1.0f + erff(x * 0.70710678118654752f)) : gelu_grad_f(x);
      };
      const int k0 = threadIdx.x * PER;
      float left = value(k0);
#pragma unroll
      for (int i = 0; i < PER; ++i) {
        const float right = value(k0 + i + 1);
        gelu_tab[k0 + i] = make_float2(left, right - left);
        left = right;
      }
    }
  };

  // Direct loads of one K tile.  The wavefront's i-th instruction for an operand covers the 64
  // slots q = wave * kPerWave + i of the tile; which rows that is goes into the lane's byte
  // offset (one VGPR per instruction, constant over the K loop), so every instruction of a tile
  // shares one uniform base pointer that just advances by a K tile.
  unsigned voff_a[OpA::kPerWave], voff_b[OpB::kPerWave];
#pragma unroll
  for (int i = 0; i < OpA::kPerWave; ++i)
    voff_a[i] = OpA::template offset<EDGE>(wave * OpA::kPerWave + i, lane, p.lda, p.M - m0);
#pragma unroll
  for (int i = 0; i < OpB::kPerWave; ++i)
    voff_b[i] = OpB::template offset<EDGE>(wave * OpB::kPerWave + i, lane, p.ldb, p.N - n0);
  // uniform running state of the loader: next tile's base pointers and LDS buffer
  const bf16* a_next = A_T ? p.A + m0 : p.A + (size_t)m0 * p.lda;
  const bf16* b_next = B_T ? p.B + n0 : p.B + (size_t)n0 * p.ldb;
  const size_t a_step = A_T ? (size_t)kBK * p.lda : (size_t)kBK;
  const size_t b_step = B_T ? (size_t)kBK * p.ldb : (size_t)kBK;
  unsigned stage_next = 0;  // buffer index the next issued tile goes to
  const unsigned wave_lds_a = lds0 + wave * OpA::kPerWave * 1024;
  const unsigned wave_lds_b = lds0 + OpA::kBytes + wave * OpB::kPerWave * 1024;
  // the i-th of the LOADS direct loads of the next tile (i is a compile-time constant at every call)
  auto issue_part = [&](int i) {
    const unsigned st = stage_next * STAGE_BYTES;
    if (i < OpA::kPerWave) dma16(a_next, voff_a[i], wave_lds_a + st + i * 1024);
    else dma16(b_next, voff_b[i - OpA::kPerWave], wave_lds_b + st + (i - OpA::kPerWave) * 1024);
  };
  // EDGE, before the first load of the last tile (nothing is started after it): what lies past K is fetched from inside
  auto stay_inside_k = [&](bool last) {
    if (!EDGE || !last || k_tail == kBK) return;
#pragma unroll
    for (int i = 0; i < OpA::kPerWave; ++i) {
      const int q = wave * OpA::kPerWave + i;
      if (OpA::past_k(q, lane, k_tail)) voff_a[i] -= OpA::k_part(q, lane, p.lda);
    }
#pragma unroll
    for (int i = 0; i < OpB::kPerWave; ++i) {
      const int q = wave * OpB::kPerWave + i;
      if (OpB::past_k(q, lane, k_tail)) voff_b[i] -= OpB::k_part(q, lane, p.ldb);
    }
  };
  // EDGE: zeros over what this wavefront loaded from past K into the stage of the last tile
  auto clear_past_k = [&]() {
    if (!EDGE || k_tail == kBK) return;
    char* st = smem + ((nk - 1) % NSTAGE) * STAGE_BYTES;
    const f32x4 z = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int i = 0; i < OpA::kPerWave; ++i) {
      const int q = wave * OpA::kPerWave + i;
      if (OpA::past_k(q, lane, k_tail)) *reinterpret_cast<f32x4*>(st + (q * 64 + lane) * 16) = z;
    }
#pragma unroll
    for (int i = 0; i < OpB::kPerWave; ++i) {
      const int q = wave * OpB::kPerWave + i;
      if (OpB::past_k(q, lane, k_tail)) *reinterpret_cast<f32x4*>(st + OpA::kBytes + (q * 64 + lane) * 16) = z;
    }
  };
  auto issue_done = [&]() {
    a_next += a_step;
    b_next += b_step;
    stage_next = stage_next + 1 == NSTAGE ? 0 : stage_next + 1;
  };
  auto issue = [&]() {
#pragma unroll
    for (int i = 0; i < LOADS; ++i) issue_part(i);
    issue_done();
  };

  f32x4 acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int r = 0; r < 4; ++r) acc[i][j][r] = 0.f;

  const unsigned at_a = lds0 + OpA::lane_at(wm * WM, lane), at_b = lds0 + OpA::kBytes + OpB::lane_at(wn * WN, lane);
  static_assert(WM <= 128 && WN <= 128 && STAGE_BYTES % 1024 == 0, "frag flips address bits below 256");

  // Column sums of B (bias gradient): the workgroup of tile row 0 sums every K tile of its tile column from
  // the B tiles that pass through LDS anyway (each thread adds 4 columns x (kBK / kColRowGroups) rows per
  // tile).  One workgroup per column and a fixed order of additions: the sums are the same bits every run.
  constexpr int kColGroups = BN / 4, kColRowGroups = NW * 64 / kColGroups, kColRows = kBK / kColRowGroups;
  float csum[4] = {0.f, 0.f, 0.f, 0.f};
  constexpr bool kColsum = EPI == EPI_ACCUM_F32;  // nothing else asks for them
  const bool sums_columns = kColsum && p.colsum && tile_m == 0;
  auto colsum_tile = [&](int kt) {
    if constexpr (kColsum) {
      if (sums_columns) {
        const char* b_lds = smem + (kt % NSTAGE) * STAGE_BYTES + OpA::kBytes;
        const int c = (threadIdx.x % kColGroups) * 4, rg = threadIdx.x / kColGroups;
#pragma unroll
        for (int r = 0; r < kColRows; ++r) {
          const int row = rg * kColRows + r;
          const int slot = OpB::swizzle(row, c >> 3);
          const bf16x4 v = *reinterpret_cast<const bf16x4*>(b_lds + (row * OpB::kSlotsPerRow + slot) * 16 + (c & 7) * 2);
#pragma unroll
          for (int e = 0; e < 4; ++e) csum[e] += (float)v[e];
        }
      }
    }
  };

  // Main loop over K tiles of two MFMA steps.  A wavefront holds the A fragments of one step, each replaced by the next
  // step's as soon as its row of MFMAs is out, and the B fragments of two:
  //   step 0                | LDS reads: the fragments of step 1
  //   step 1, kHead rows    | these cover the last of those reads
  //   everything of the tile is in registers: wait until the next tile has landed; barrier (everyone is there)
  //   step 1, other rows    | start the loads of tile kt + NSTAGE into the buffer of tile kt; LDS reads: step 0 of tile kt + 1
  // Behind each MFMA goes its share of the reads and loads, one or two instructions, held there by scheduling barriers:
  // every wavefront leaves the barrier in the same phase, so a run of loads between two MFMAs idles the matrix pipe of all
  // four SIMDs at once.  With three stages the second half of a tile's direct loads goes out in step 0 of the next tile
  // (with two it would have less than a tile's time to land).
  constexpr int kHead = 2, kLate = (TM - kHead) * TN, kMf = TM * TN;
  constexpr int kFirst = NSTAGE < 3 ? LOADS : LOADS / 2, kRest = LOADS - kFirst;
  static_assert(KS == 2 && kLate >= TN + kHead && kFirst <= 2 * kLate && kRest <= kMf, "slots for every read and load");
  bf16x8 fa[TM], fb[2][TN];
  // Loads [n0, n1) of the next tile that belong behind slot m of `slots`: evenly spread.
  auto issue_slot = [&](int m, int slots, int n0, int n1) {
#pragma unroll
    for (int u = 0; u < LOADS; ++u)
      if (n0 + u < n1 && u * slots / (n1 - n0) == m) issue_part(n0 + u);
  };
  // One K tile.  ISSUE: start the loads of tile kt + NSTAGE; `rest`: the previous tile left half of its loads; NEXT: there is
  // a tile kt + 1, admitted once at most `in_flight` younger tiles are outstanding.
  auto k_tile = [&](auto issue_tag, auto next_tag, int kt, bool rest, int in_flight) {
    constexpr bool ISSUE = decltype(issue_tag)::value, NEXT = decltype(next_tag)::value;
    const unsigned cur = (kt % NSTAGE) * STAGE_BYTES, nxt = ((kt + 1) % NSTAGE) * STAGE_BYTES;
    unsigned a_cur = at_a + cur, b_cur = at_b + cur, a_nxt = at_a + nxt, b_nxt = at_b + nxt;
    // left to itself the compiler keeps a register per fragment address and spills
    asm volatile("" : "+v"(a_cur), "+v"(b_cur));
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j) {
        acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fb[0][j], fa[i], acc[i][j], 0, 0, 0);
        if (i == 0) fb[1][j] = OpB::frag(b_cur, j, 1);
        if (j == TN - 1) fa[i] = OpA::frag(a_cur, i, 1);
        if (kRest > 0 && NEXT && rest) issue_slot(i * TN + j, kMf, kFirst, LOADS);
        __builtin_amdgcn_sched_barrier(0);
      }
    if (kRest > 0 && NEXT && rest) issue_done();
#pragma unroll
    for (int i = 0; i < kHead; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fb[1][j], fa[i], acc[i][j], 0, 0, 0);
    __builtin_amdgcn_sched_barrier(0);
    if constexpr (NEXT) {
      asm volatile("" : "+v"(a_nxt), "+v"(b_nxt));
      // the buffer of tile kt is overwritten right after the barrier: its last fragments must have arrived
      asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
      if constexpr (ISSUE) wait_vmcnt<(NSTAGE - 2) * LOADS>();
      else wait_tiles<LOADS>(in_flight);
      if (!ISSUE && kt + 2 == nk) clear_past_k();
      __syncthreads();
      if constexpr (ISSUE) stay_inside_k(kt + NSTAGE == nk - 1);
      __builtin_amdgcn_sched_barrier(0);
    }
#pragma unroll
    for (int i = kHead; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j) {
        const int m = (i - kHead) * TN + j;
        acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fb[1][j], fa[i], acc[i][j], 0, 0, 0);
        if constexpr (NEXT) {
          if (m < TN) fb[0][m] = OpB::frag(b_nxt, m, 0);
          else if (m < TN + kHead) fa[m - TN] = OpA::frag(a_nxt, m - TN, 0);
          if (j == TN - 1) fa[i] = OpA::frag(a_nxt, i, 0);
        }
        if constexpr (ISSUE) issue_slot(m, kLate, 0, kFirst);
        __builtin_amdgcn_sched_barrier(0);
      }
    if constexpr (ISSUE && kRest == 0) issue_done();
    if constexpr (NEXT) colsum_tile(kt + 1);
  };
  {
#pragma unroll
    for (int t = 0; t < NSTAGE - (kRest > 0); ++t)
      if (t < nk) {
        stay_inside_k(t == nk - 1);
        issue();
      }
    const bool filled = kRest > 0 && nk >= NSTAGE;
    if (filled) {
      stay_inside_k(NSTAGE == nk);
#pragma unroll
      for (int i = 0; i < kFirst; ++i) issue_part(i);
    }
    build_table();
    if (filled) wait_vmcnt<(NSTAGE - 1) * LOADS - kRest>();
    else wait_tiles<LOADS>(min(NSTAGE - 1, nk - 1));
    if (nk == 1) clear_past_k();
    __syncthreads();
    colsum_tile(0);
#pragma unroll
    for (int j = 0; j < TN; ++j) fb[0][j] = OpB::frag(at_b, j, 0);
#pragma unroll
    for (int i = 0; i < TM; ++i) fa[i] = OpA::frag(at_a, i, 0);
    const std::true_type yes;
    const std::false_type no;
    int kt = 0;
    for (; kt + NSTAGE < nk; ++kt) k_tile(yes, yes, kt, true, 0);
    // The last tiles: nothing left to start.
    for (; kt + 1 < nk; ++kt) k_tile(no, yes, kt, kt + NSTAGE == nk, min(NSTAGE - 2, nk - 2 - kt));
    k_tile(no, no, kt, false, 0);
  }

  if constexpr (kColsum) {
    if (sums_columns) {  // combine the row groups through LDS (the ring is idle now); this workgroup alone owns the columns
      __syncthreads();
      float* red = reinterpret_cast<float*>(smem);
      const int c = (threadIdx.x % kColGroups) * 4, rg = threadIdx.x / kColGroups;
#pragma unroll
      for (int e = 0; e < 4; ++e) red[rg * BN + c + e] = csum[e];
      __syncthreads();
      if (threadIdx.x < BN && (!EDGE || n0 + (int)threadIdx.x < p.N)) {
        float t = 0.f;
#pragma unroll
        for (int g = 0; g < kColRowGroups; ++g) t += red[g * BN + threadIdx.x];
        p.colsum[n0 + threadIdx.x] += t;
      }
    }
  }

  // Epilogue through LDS.  In registers a lane holds 4 consecutive columns of one row, and 16
  // consecutive lanes hold 16 different rows: stores (and the reads of the residual or
  // pre-activation operand) straight from that layout touch 16 bytes per row.  Instead, one band
  // of 32 rows per wavefront row (WGM * 32 rows x BN columns, fp32) at a time is parked in LDS and
  // taken out again with each thread owning 8 consecutive columns, so every global access of the
  // epilogue is a run of full rows: 16 bytes per lane, whole 128-byte lines.
  constexpr int EP = BN + 4;  // fp32 row pitch in LDS: +4 keeps the register-layout writes conflict-free
  constexpr int kBands = WM / 32;
  float* stage = reinterpret_cast<float*>(smem);
  constexpr int kBandRows = WGM * 32, kVecPerRow = BN / 8, kVecs = kBandRows * kVecPerRow;
  static_assert((size_t)kBandRows * EP * 4 <= (size_t)NSTAGE * STAGE_BYTES, "epilogue band must fit the load ring");
  // 8 VALU operations and one LDS read per element instead of an exponential, a reciprocal and a polynomial, which at one
  // workgroup per CU nothing else would overlap.
  auto gelu_lookup = [&](float x) {
    const float t = fminf(fmaxf(fmaf(x, 128.f, 1024.f), 0.f), 2047.99f);
    const int k = (int)t;
    const float2 e = gelu_tab[k];
    return fmaf(t - (float)k, e.y, e.x);
  };
  // The operand an epilogue reads from global memory (residual, pre-activation, or the fp32 sums it
  // accumulates into) is fetched one band ahead into registers, so that its latency runs under the
  // staging of the band before instead of in front of every band's arithmetic.
  constexpr int VPT = kVecs / (NW * 64);  // 8-column vectors per thread per band
  static_assert(kVecs % (NW * 64) == 0, "band vectors divide among the threads");
  constexpr bool kReadsAux = EPI == EPI_BIAS_RES || EPI == EPI_ADD || EPI == EPI_MUL_DGELU;
  constexpr bool kReadsC = EPI == EPI_ACCUM_F32;
  bf16x8 pre_aux[2][kReadsAux ? VPT : 1];
  f32x4 pre_c[2][kReadsC ? VPT : 1][2];
  auto where = [&](int i, int u, int& br, int& c, size_t& at, int& n) {
    const int vi = threadIdx.x + u * NW * 64;
    br = vi / kVecPerRow;          // band row
    c = (vi % kVecPerRow) * 8;     // first column
    const int m = m0 + (br >> 5) * WM + i * 32 + (br & 31);
    n = n0 + c;
    at = (size_t)m * p.ldc + n;
    return !EDGE || (m < p.M && n < p.N);
  };
  auto prefetch = [&](int i, int buf) {
#pragma unroll
    for (int u = 0; u < VPT; ++u) {
      const int vi = threadIdx.x + u * NW * 64, br = vi / kVecPerRow;
      int m = m0 + (br >> 5) * WM + i * 32 + (br & 31), n = n0 + (vi % kVecPerRow) * 8;
      if (EDGE) m = min(m, p.M - 1), n = n < p.N ? n : n0;  // from inside: what is outside is not stored
      const size_t at = (size_t)m * p.ldc + n;
      if constexpr (kReadsAux) pre_aux[buf][u] = *reinterpret_cast<const bf16x8_row*>(p.aux + at);
      if constexpr (kReadsC) {
        pre_c[buf][u][0] = *reinterpret_cast<const f32x4*>(p.Cf + at);
        pre_c[buf][u][1] = *reinterpret_cast<const f32x4*>(p.Cf + at + 4);
      }
    }
  };
  if constexpr (kReadsAux || kReadsC) prefetch(0, 0);
#pragma unroll
  for (int i = 0; i < kBands; ++i) {
    __syncthreads();  // the ring (first band) or the previous band is no longer being read
    {
      float* dst = stage + (wm * 32 + (lane & 15)) * EP + wn * WN + 4 * (lane >> 4);
#pragma unroll
      for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int j = 0; j < TN; ++j) *reinterpret_cast<f32x4*>(dst + h * 16 * EP + j * 16) = acc[2 * i + h][j];
    }
    if constexpr (kReadsAux || kReadsC) {
      if (i + 1 < kBands) prefetch(i + 1, (i + 1) & 1);
    }
    __syncthreads();
#pragma unroll
    for (int u = 0; u < VPT; ++u) {
      int br, c, n;
      size_t at;
      if (!where(i, u, br, c, at, n)) continue;
      float v[8];
      load8(stage + br * EP + c, v);
      if constexpr (EPI == EPI_ACCUM_F32) {
        float cur[8];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          cur[e] = pre_c[i & 1][u][0][e] + v[e];
          cur[4 + e] = pre_c[i & 1][u][1][e] + v[4 + e];
        }
        store8(p.Cf + at, cur);
      } else if constexpr (EPI == EPI_STORE_F32) {
        store8(p.Cf + at, v);
      } else {
        if constexpr (EPI == EPI_BIAS || EPI == EPI_BIAS_GELU || EPI == EPI_BIAS_RES) {
          float b[8];
          load8(p.bias + n, b);
#pragma unroll
          for (int e = 0; e < 8; ++e) v[e] += b[e];
        }
        if constexpr (EPI == EPI_BIAS_RES || EPI == EPI_ADD) {
#pragma unroll
          for (int e = 0; e < 8; ++e) v[e] += (float)pre_aux[i & 1][u][e];
        }
        if constexpr (EPI == EPI_MUL_DGELU) {
#pragma unroll
          for (int e = 0; e < 8; ++e) v[e] *= gelu_lookup((float)pre_aux[i & 1][u][e]);
        }
        if constexpr (EPI == EPI_BIAS_GELU) {
          store8_row(p.aux_out + at, v);
#pragma unroll
          for (int e = 0; e < 8; ++e) v[e] *= gelu_lookup(v[e]);
        }
        store8_row(p.C + at, v);
      }
    }
  }
  if constexpr (kLoop) {
    wg += step;
    if (step && wg < tiles_end) {
      wait_vmcnt<0>();
      __syncthreads();  // the last band is no longer being read
      goto next_tile;
    }
  }
}

// A single product, unless it is a weight gradient, is passed by itself: what its first loads depend on stands in the first 14 words of
// the kernel's arguments, which are in scalar registers when it starts (see the build flags); live_dim stands beside ldc.
template <int BM, int BN, int WGM, int WGN, int NSTAGE, bool A_T, bool B_T, int EPI, bool EDGE>
__global__ __launch_bounds__(WGM* WGN * 64) __attribute__((amdgpu_waves_per_eu(2, 2))) void gemm_dma_kernel(
    const bf16* A, const bf16* B, void* C, const bf16* bias, int M, int N, int K, int lda, int ldb, unsigned ldc_live, const bf16* aux,
    bf16* aux_out, const int* live) {
  DmaGemm p;
  p.A = A; p.B = B; p.C = (bf16*)C; p.Cf = (float*)C; p.bias = bias; p.aux = aux; p.aux_out = aux_out;
  p.M = M; p.N = N; p.K = K; p.lda = lda; p.ldb = ldb; p.ldc = ldc_of(ldc_live);
  p.colsum = nullptr; p.live = live; p.live_dim = live_dim_of(ldc_live);
  gemm_dma_body<BM, BN, WGM, WGN, NSTAGE, A_T, B_T, EPI, EDGE>(p, (int)blockIdx.x);
}
template <int BM, int BN, int WGM, int WGN, int NSTAGE, bool A_T, bool B_T, int EPI, bool EDGE>
__global__ __launch_bounds__(WGM* WGN * 64) __attribute__((amdgpu_waves_per_eu(2, 2))) void gemm_dma_group_kernel(DmaGemmGroup grp) {
  if (EPI == EPI_ACCUM_F32 && (int)blockIdx.x >= grp.first[kMaxGroup]) {
    extern __shared__ __attribute__((aligned(1024))) char smem[];
    const int at = (int)blockIdx.x - grp.first[kMaxGroup], second = at >= grp.job_blocks;
    finalize_columns<WGM * WGN * 64, 4>(grp.job[second], at - second * grp.job_blocks, smem);
    return;
  }
  int gi = 0;
#pragma unroll
  for (int j = 1; j < kMaxGroup; ++j)
    if (j < grp.count && (int)blockIdx.x >= grp.first[j]) gi = j;
  gemm_dma_body<BM, BN, WGM, WGN, NSTAGE, A_T, B_T, EPI, EDGE>(grp.prob[gi], (int)blockIdx.x - grp.first[gi]);
}

template <int BM, int BN, int WGM, int WGN, int NSTAGE, bool A_T, bool B_T, int EPI, bool EDGE>
int launch(DmaGemmGroup& grp, hipStream_t stream) {
  constexpr int NW = WGM * WGN;
  constexpr size_t lds = (size_t)NSTAGE * (Operand<BM, A_T, NW>::kBytes + Operand<BN, B_T, NW>::kBytes) +
                         (EPI == EPI_BIAS_GELU || EPI == EPI_MUL_DGELU ? kGeluN * sizeof(float2) : 0);
  long tiles = 0;
  for (int i = 0; i < grp.count; ++i) {
    grp.first[i] = (int)tiles;
    tiles += (long)((grp.prob[i].N + BN - 1) / BN) * ((grp.prob[i].M + BM - 1) / BM);
    if (grp.prob[i].live_dim == LIVE_M_SPLIT && tiles < kSplitGrid) tiles = kSplitGrid;
  }
  if (tiles > 0x7fff0000L) return set_error(HANAYO_EUNSUPPORTED, "gemm_dma: too many tiles");
  // Rows counted on the device: of the workgroups that all M rows would need, those past the count have nothing to do, but
  // each waits for a CU with room for its LDS (460 of 4096 rows x 30592 columns, 1680 of 1920 workgroups idle: 50 us; 31
  // for a launch of 460 rows).  Alone on the chip, as many workgroups as fit at once take the tiles in turn; next to other
  // lanes, where some would start late, the dispatcher deals out one tile each.
  if (EDGE && EPI == EPI_NONE && !B_T && grp.count == 1 && grp.prob[0].live && grp.prob[0].live_dim == LIVE_M && gemm_sharing() <= 0.0) {
    const long fit = 256L * (long)(160 * 1024 / lds);
    if (tiles > fit) tiles = fit;
  }
  for (int i = grp.count; i <= kMaxGroup; ++i) grp.first[i] = (int)tiles;
  const dim3 block(NW * 64);
  if constexpr (EPI != EPI_STORE_F32) {
    if (EPI == EPI_ACCUM_F32 || grp.count > 1) {
      auto kern = gemm_dma_group_kernel<BM, BN, WGM, WGN, NSTAGE, A_T, B_T, EPI, EDGE>;
      static thread_local uint64_t raised = 0;
      if (const int rc = raise_lds(reinterpret_cast<const void*>(kern), lds, raised)) return rc;
      grp.job_blocks = 0;
      for (int i = 0; i < grp.n_jobs; ++i) {
        const int blocks = finalize_blocks(grp.job[i], finalize_cols<NW * 64, 4>());
        if (blocks > grp.job_blocks) grp.job_blocks = blocks;
      }
      launch_kernel(kern, dim3((unsigned)(tiles + (long)grp.n_jobs * grp.job_blocks)), block, lds, stream, grp);
      return check_launch("gemm_dma");
    }
  }
  if constexpr (EPI != EPI_ACCUM_F32) {
    auto kern = gemm_dma_kernel<BM, BN, WGM, WGN, NSTAGE, A_T, B_T, EPI, EDGE>;
    static thread_local uint64_t raised = 0;
    if (const int rc = raise_lds(reinterpret_cast<const void*>(kern), lds, raised)) return rc;
    const DmaGemm& p = grp.prob[0];
    launch_kernel(kern, dim3((unsigned)tiles), block, lds, stream, p.A, p.B, (void*)p.C, p.bias, p.M, p.N, p.K, p.lda, p.ldb,
                  pack_ldc(p.ldc, p.live_dim), p.aux, p.aux_out, p.live);
  }
  return check_launch("gemm_dma");
}

template <int BM, int BN, int WGM, int WGN, int NSTAGE, bool EDGE>
int launch_layout(const GemmArgs& g, DmaGemmGroup& grp, hipStream_t stream) {
  if (!g.a_t && g.b_t) {
    switch (g.epi) {
      case EPI_NONE: return launch<BM, BN, WGM, WGN, NSTAGE, false, true, EPI_NONE, EDGE>(grp, stream);
      case EPI_BIAS: return launch<BM, BN, WGM, WGN, NSTAGE, false, true, EPI_BIAS, EDGE>(grp, stream);
      case EPI_BIAS_GELU: return launch<BM, BN, WGM, WGN, NSTAGE, false, true, EPI_BIAS_GELU, EDGE>(grp, stream);
      case EPI_BIAS_RES: return launch<BM, BN, WGM, WGN, NSTAGE, false, true, EPI_BIAS_RES, EDGE>(grp, stream);
      case EPI_STORE_F32:  // the split contraction of LIVE_M_SPLIT only
        if constexpr (BM == 256 && BN == 256 && EDGE) return launch<BM, BN, WGM, WGN, NSTAGE, false, true, EPI_STORE_F32, EDGE>(grp, stream);
        break;
      default: break;
    }
  } else if (!g.a_t && !g.b_t) {
    switch (g.epi) {
      case EPI_NONE: return launch<BM, BN, WGM, WGN, NSTAGE, false, false, EPI_NONE, EDGE>(grp, stream);
      case EPI_MUL_DGELU: return launch<BM, BN, WGM, WGN, NSTAGE, false, false, EPI_MUL_DGELU, EDGE>(grp, stream);
      case EPI_ADD: return launch<BM, BN, WGM, WGN, NSTAGE, false, false, EPI_ADD, EDGE>(grp, stream);
      default: break;
    }
  } else if (g.a_t && g.b_t && g.epi == EPI_ACCUM_F32) {
    return launch<BM, BN, WGM, WGN, NSTAGE, true, true, EPI_ACCUM_F32, EDGE>(grp, stream);
  }
  return set_error(HANAYO_EUNSUPPORTED, "gemm_dma: layout/epilogue combination not built");
}

bool whole_tiles(const GemmArgs& g, int config) {
  int bm, bn;
  gemm_dma_tile(config, bm, bn);
  return g.M % bm == 0 && g.N % bn == 0 && g.K % kBK == 0;
}

}  // namespace

// Tile configurations: 7 = 256 x 256 with 8 wavefronts (2 x 4, 128 x 64 each: two per SIMD that cover each other's
// stalls), two stages; 9 = 128 x 128 with 4 wavefronts, two stages (64 KiB: two workgroups per CU); 10 = 256 x 128 with 8
// wavefronts (4 x 2, 64 x 64 each), three stages (with 4 wavefronts of 128 x 64 the same time where every CU has a tile and
// 3 - 7 % more where some idle: 2048 x 2560 x 2560 34.1 us, here 31.6); 11 = 128 x 128 with 4 wavefronts, three stages (96
// KiB, one workgroup per CU: for launches whose single wavefront per SIMD has nothing else to cover a late load).
bool gemm_dma_config_exists(int config) { return config == 7 || (config >= 9 && config <= 11); }
void gemm_dma_tile(int config, int& bm, int& bn) {
  bm = config == 9 || config == 11 ? 128 : 256;
  bn = config == 7 ? 256 : 128;
}

bool gemm_dma_supported(const GemmArgs& g, int config) {
  const bool combo = (!g.a_t && g.b_t && (g.epi == EPI_NONE || g.epi == EPI_BIAS || g.epi == EPI_BIAS_GELU || g.epi == EPI_BIAS_RES ||
                                             (g.epi == EPI_STORE_F32 && config == 7 && g.live && g.live_dim == LIVE_M_SPLIT))) ||
                     (!g.a_t && !g.b_t && (g.epi == EPI_NONE || g.epi == EPI_MUL_DGELU || g.epi == EPI_ADD)) ||
                     (g.a_t && g.b_t && g.epi == EPI_ACCUM_F32);
  if (!combo || !gemm_dma_config_exists(config) || (g.colsum && g.epi != EPI_ACCUM_F32)) return false;
  int bm, bn;
  gemm_dma_tile(config, bm, bn);
  // lane offsets are 32-bit byte offsets from the tile origin
  const long span_a = (long)(g.a_t ? kBK : bm) * g.lda * 2, span_b = (long)(g.b_t ? kBK : bn) * g.ldb * 2;
  // operands on 16-byte boundaries with every row of A and B on one too (those of C: see epilogue.h)
  const uintptr_t bits = (uintptr_t)g.A | (uintptr_t)g.B | (uintptr_t)g.C | (uintptr_t)g.bias | (uintptr_t)g.aux | (uintptr_t)g.aux_out;
  if (bits % 16 || g.lda % 8 || g.ldb % 8 || g.ldc % 4 || span_a >= (1L << 31) || span_b >= (1L << 31)) return false;
  if (whole_tiles(g, config)) return true;
  // edges: whole 16-byte vectors along every row
  return (g.a_t ? g.M : g.K) % 8 == 0 && (g.b_t ? g.N : g.K) % 8 == 0 && g.N % 8 == 0;
}

// The problems of a group share layout and epilogue (those of gs[0]); each must pass gemm_dma_supported.
int gemm_dma_group(const GemmArgs* gs, int count, int config, hipStream_t stream, const FinalizeJob* jobs, int n_jobs) {
  if (n_jobs < 0 || n_jobs > kMaxJobs || (n_jobs && gs[0].epi != EPI_ACCUM_F32)) return set_error(HANAYO_EINVAL, "gemm_dma: %d jobs", n_jobs);
  if (count < 1 || count > kMaxGroup) return set_error(HANAYO_EINVAL, "gemm_dma: group of %d", count);
  DmaGemmGroup grp{};
  grp.count = count;
  grp.n_jobs = n_jobs;
  for (int i = 0; i < n_jobs; ++i) grp.job[i] = jobs[i];
  bool edge = false;
  for (int i = 0; i < count; ++i) {
    const GemmArgs& g = gs[i];
    if (!gemm_dma_supported(g, config) || g.a_t != gs[0].a_t || g.b_t != gs[0].b_t || g.epi != gs[0].epi)
      return set_error(HANAYO_EUNSUPPORTED, "gemm_dma: shape not supported");
    edge = edge || !whole_tiles(g, config);
    DmaGemm& p = grp.prob[i];
    p.A = (const bf16*)g.A; p.B = (const bf16*)g.B; p.C = (bf16*)g.C; p.Cf = (float*)g.C;
    p.bias = (const bf16*)g.bias; p.aux = (const bf16*)g.aux; p.aux_out = (bf16*)g.aux_out;
    p.M = g.M; p.N = g.N; p.K = g.K; p.lda = g.lda; p.ldb = g.ldb; p.ldc = g.ldc;
    p.colsum = g.b_t ? g.colsum : nullptr;
    p.live = g.live; p.live_dim = g.live ? g.live_dim : LIVE_NONE;
    edge = edge || g.live;
    if (g.live && g.live_dim == LIVE_M_SPLIT && (config != 7 || count != 1 || g.epi != EPI_STORE_F32))
      return set_error(HANAYO_EUNSUPPORTED, "gemm_dma: a split contraction takes one problem of 256 x 256 tiles");
  }
  const GemmArgs& g = gs[0];
  switch (config) {
    case 7: return edge ? launch_layout<256, 256, 2, 4, 2, true>(g, grp, stream) : launch_layout<256, 256, 2, 4, 2, false>(g, grp, stream);
    case 9: return edge ? launch_layout<128, 128, 2, 2, 2, true>(g, grp, stream) : launch_layout<128, 128, 2, 2, 2, false>(g, grp, stream);
    case 10: return edge ? launch_layout<256, 128, 4, 2, 3, true>(g, grp, stream) : launch_layout<256, 128, 4, 2, 3, false>(g, grp, stream);
    default: return edge ? launch_layout<128, 128, 2, 2, 3, true>(g, grp, stream) : launch_layout<128, 128, 2, 2, 3, false>(g, grp, stream);
  }
}

int gemm_dma(const GemmArgs& g, int config, hipStream_t stream) { return gemm_dma_group(&g, 1, config, stream); }

}  // namespace k
}  // namespace hanayo
