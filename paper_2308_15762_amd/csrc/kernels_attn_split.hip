// bf16 attention for launches of few rows: the 128-row workgroups of kernels_attn_mfma.hip leave most CUs idle there, and
// each walks its keys (queries) in one serial chain, which is what such a launch lasts.
//
// A workgroup owns 32 rows and its four wavefronts take every fourth 32-row tile of the other side: four times the
// workgroups, chains a quarter as long.  Every wavefront fills an LDS ring of its own with direct loads and waits for its
// own loads only, so there is no barrier before the end, where the partial results (forward: each with its own running
// maximum and sum) are merged in a fixed order through LDS.  dQ and dK / dV share one launch: the latter forms delta =
// rowsum(dC * C) of a query tile itself instead of waiting for the former.  The price is four times the K and V (Q, dC)
// traffic through L2 and LDS, which is why launches that fill the chip keep the 128-row kernels.
//
// What bounds a launch here is the chain of one wavefront (loads of a tile, two products, exponentials, one or two more
// products), hence the split.  us, forward / backward, with 128-row workgroups and here: one sequence of 777, 8 heads of 80,
// causal, 23.2 / 64.0 and 11.9 / 19.6; two of 256, 4 heads of 64, 7.4 / 19.8 and 5.0 / 7.1.
//
// Orientation and fragments as in kernels_attn_mfma.hip.
#include "attn_tile.h"
#include "kernels.h"

namespace hanayo {
namespace k {

namespace {

constexpr int NW = 4;   // wavefronts per workgroup
constexpr int NST = 2;  // stages of a wavefront's ring

template <int DP>
constexpr int kTile32 = 32 * DP * 2;  // bytes of a 32-row tile
template <int DP>
constexpr int kPart = 32 * (DP + 4);  // floats of a wavefront's parked 32 x DP partial result
template <int DP>
constexpr size_t lds_bytes(int stage, int stages = NST) {
  const size_t ring = (size_t)NW * stages * stage, parts = (size_t)NW * kPart<DP> * 4 + NW * 32 * sizeof(float2);
  return ring > parts ? ring : parts;
}

// Workgroup -> (tile, head, sequence): consecutive workgroups are heads, so that all of a head's tiles share an XCD where
// the (sequence, head) pairs are a multiple of 8, and the long tiles of a causal grid, which come first, start together.
__device__ __forceinline__ void place(const AttnDev& p, int w, int pairs, int& tile, int& h, int& n) {
  const int hn = w % pairs;
  tile = w / pairs;
  h = hn % p.heads;
  n = hn / p.heads;
}

// A wavefront's partial result to LDS: lane holds row lane % 32, columns 32 dt + acc_row(r).
template <int DP, int DT>
__device__ __forceinline__ void park(float* part, const f32x16 (&o)[DT], int lane) {
#pragma unroll
  for (int dt = 0; dt < DT; ++dt)
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      f32x4 v;
#pragma unroll
      for (int e = 0; e < 4; ++e) v[e] = o[dt][4 * q + e];
      *reinterpret_cast<f32x4*>(part + (lane & 31) * (DP + 4) + 32 * dt + 8 * q + 4 * (lane >> 5)) = v;
    }
}
// Sum of the four parked results, times `scale`, to rows row0 .. of `out` (row pitch ld).
template <int DP, int D>
__device__ __forceinline__ void sum_parts(const float* parts, float scale, bf16* out, size_t ld, int row0, int s) {
  for (int i = threadIdx.x; i < 32 * (D / 8); i += NW * 64) {
    const int row = i / (D / 8), c = (i % (D / 8)) * 8;
    if (row0 + row >= s) continue;
    float v[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int w = 0; w < NW; ++w) {
      float t[8];
      load8(parts + w * kPart<DP> + row * (DP + 4) + c, t);
#pragma unroll
      for (int e = 0; e < 8; ++e) v[e] += t[e];
    }
#pragma unroll
    for (int e = 0; e < 8; ++e) v[e] *= scale;
    store8(out + (size_t)(row0 + row) * ld + c, v);
  }
}

template <int DP, int D>
__global__ __launch_bounds__(NW * 64) void attn_fwd_split_kernel(int pairs, int /* tiles */, ATTN_PARAMS) {
  const AttnDev p = ATTN_BLOCK;
  using Tile = SwTile<DP>;
  constexpr int KS = D / 16, DT = (D + 31) / 32, STAGE = 2 * kTile32<DP>, LOADS = 2 * Tile::kInstr32;
  extern __shared__ __attribute__((aligned(1024))) char smem[];
  const unsigned lds0 = (unsigned)(unsigned long)((__attribute__((address_space(3))) char*)smem);
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), half = lane >> 5;
  typename Tile::Offsets fo;
  Tile::init(fo, lane);
  int qt, h, n;
  place(p, blockIdx.x, pairs, qt, h, n);
  qt = gridDim.x / pairs - 1 - qt;
  const int H = p.heads * p.d, ld3 = 3 * H, q0 = qt * 32, q = q0 + (lane & 31);
  const bf16* base = p.qkv + (size_t)n * p.s * ld3 + h * p.d;
  const int len = seq_len(p, n);
  const int kv_end = p.causal ? min(len, q0 + 32) : len;
  const int nt = (kv_end + 31) / 32, mine = nt > wave ? (nt - wave + NW - 1) / NW : 0;
  const float c2 = rsqrtf((float)p.d) * kLog2e;
  const unsigned ring = lds0 + wave * NST * STAGE;
  const char* ring_ptr = smem + wave * NST * STAGE;
  auto issue = [&](int j) {
    const unsigned st = ring + (unsigned)(j % NST) * STAGE;
    const int k0 = (wave + j * NW) * 32;
    Tile::template issue32<D>(base + H, ld3, k0, p.s, st, lane);
    Tile::template issue32<D>(base + 2 * H, ld3, k0, p.s, st + kTile32<DP>, lane);
  };
#pragma unroll
  for (int j = 0; j < NST; ++j)
    if (j < mine) issue(j);

  bf16x8 qf[KS];
#pragma unroll
  for (int kk = 0; kk < KS; ++kk) qf[kk] = frag_global(base + (size_t)q * ld3, q < p.s, kk, lane, p.d);
  f32x16 o[DT];
#pragma unroll
  for (int dt = 0; dt < DT; ++dt) o[dt] = zero16();
  float m = -INFINITY, lsum = 0.f;  // m in units of raw (unscaled) scores
  for (int j = 0; j < mine; ++j) {
    if (j + 1 < mine) wait_vmcnt<LOADS>();
    else wait_vmcnt<0>();
    const char* Ks = ring_ptr + (j % NST) * STAGE;
    const char* Vs = Ks + kTile32<DP>;
    const int k0 = (wave + j * NW) * 32;
    f32x16 sc = zero16();
#pragma unroll
    for (int kk = 0; kk < KS; ++kk)
      sc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(Tile::frag_rows(Ks, fo, 0, kk), qf[kk], sc, 0, 0, 0);
    if ((p.causal && k0 + 31 > q0) || k0 + 32 > len) {
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int key = k0 + acc_row(r, half);
        if (!(key < len && (!p.causal || key <= q))) sc[r] = -INFINITY;
      }
    }
    float mloc = sc[0];
#pragma unroll
    for (int r = 1; r < 16; ++r) mloc = fmaxf(mloc, sc[r]);
    mloc = halves_max(mloc);
    const float m_new = fmaxf(m, mloc);  // finite: the first key of every tile walked is allowed for every row
    const float alpha = __builtin_amdgcn_exp2f((m - m_new) * c2), shift = -m_new * c2;
    float rs = 0.f;
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      sc[r] = __builtin_amdgcn_exp2f(fmaf(sc[r], c2, shift));
      rs += sc[r];
    }
    rs = halves_sum(rs);
    lsum = lsum * alpha + rs;
    m = m_new;
    if (__builtin_amdgcn_ballot_w64(alpha != 1.0f)) {
#pragma unroll
      for (int dt = 0; dt < DT; ++dt)
#pragma unroll
        for (int r = 0; r < 16; ++r) o[dt][r] *= alpha;
    }
#pragma unroll
    for (int tt = 0; tt < 2; ++tt) {
      const bf16x8 pf = pack_half(sc, tt);
#pragma unroll
      for (int dt = 0; dt < DT; ++dt)
        o[dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(Tile::frag_cols(Vs, fo, 16 * tt, dt), pf, o[dt], 0, 0, 0);
    }
    if (j + NST < mine) {
      asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");  // the stage has been read: it takes another tile
      issue(j + NST);
    }
  }
  __syncthreads();  // the rings are no longer read
  float* parts = reinterpret_cast<float*>(smem);
  float2* stats = reinterpret_cast<float2*>(parts + NW * kPart<DP>);
  park<DP>(parts + wave * kPart<DP>, o, lane);
  if (half == 0) stats[wave * 32 + lane] = make_float2(m, lsum);
  __syncthreads();
  for (int i = threadIdx.x; i < 32 * (D / 8); i += NW * 64) {
    const int row = i / (D / 8), c = (i % (D / 8)) * 8;
    if (q0 + row >= p.s) continue;
    float mx = -INFINITY, total = 0.f;
#pragma unroll
    for (int w = 0; w < NW; ++w) mx = fmaxf(mx, stats[w * 32 + row].x);
    float v[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int w = 0; w < NW; ++w) {
      const float2 st = stats[w * 32 + row];
      const float f = __builtin_amdgcn_exp2f((st.x - mx) * c2);  // 0 for a wavefront that had no tile
      total += st.y * f;
      float t[8];
      load8(parts + w * kPart<DP> + row * (DP + 4) + c, t);
#pragma unroll
      for (int e = 0; e < 8; ++e) v[e] += t[e] * f;
    }
    const float inv = 1.f / total;
#pragma unroll
    for (int e = 0; e < 8; ++e) v[e] *= inv;
    store8(p.ctx + ((size_t)n * p.s + q0 + row) * H + h * p.d + c, v);
    if (c == 0) p.lse[((size_t)n * p.heads + h) * p.s + q0 + row] = (mx * c2 + log2f(total)) * kLn2;
  }
}

// Bytes of a stage of the backward kernel's ring: two tiles, and behind them for dK / dV the 64 log-sum-exps (32 needed)
// of the query tile and its 32 deltas.
template <int DP>
constexpr int kBwdStage = 2 * kTile32<DP> + 512;
// Stages of the backward kernel's rings.  One, and at most 256 registers, leave room for a second workgroup on a CU (for more
// below d = 80), whose wavefronts cover the loads better than a second stage does: us with two and with one: d = 64, s = 256, 8
// pairs 6.5 and 5.9; s = 509, 36 pairs, no mask 27.7 and 25.6; s = 1024, 8 heads 16.8 and 15.2; d = 32, s = 500, 8 heads 7.9 and 7.1; d =
// 80, s = 1024, 4 heads 19.2 and 17.4; s = 777, 8 heads 19.2 and 18.7; s = 96, 16 pairs 6.5 and 6.4; d = 96, s = 384, 10 heads 10.6 and 10.0,
// s = 1024, 4 and 8 heads 19.5 and 18.0, 25.3 and 21.6, s = 700, 6 heads, no mask 25.3 and 17.8.  A few more workgroups than CUs under a
// causal mask go the other way, the last ones being short: d = 96, s = 700, 6 heads 16.2 and 16.5, s = 600, 8 heads 14.6 and 15.4; twice the
// kernels for that are not worth it.  d = 128 does not fit 256 registers (s = 512, 8 heads 15.1 and 23.4).
template <int D>
constexpr int kBwdStages = D == 128 ? 2 : 1;

// dQ of 32 query rows.
template <int DP, int D>
__device__ __forceinline__ void bwd_dq(const AttnDev& p, char* smem, int qt, int h, int n) {
  using Tile = SwTile<DP>;
  constexpr int KS = D / 16, DT = (D + 31) / 32, NB = kBwdStages<D>, STAGE = kBwdStage<DP>, LOADS = 2 * Tile::kInstr32;
  const unsigned lds0 = (unsigned)(unsigned long)((__attribute__((address_space(3))) char*)smem);
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), half = lane >> 5;
  typename Tile::Offsets fo;
  Tile::init(fo, lane);
  const int H = p.heads * p.d, ld3 = 3 * H, q0 = qt * 32, q = q0 + (lane & 31);
  const bf16* base = p.qkv + (size_t)n * p.s * ld3 + h * p.d;
  const int len = seq_len(p, n);
  const int kv_end = p.causal ? min(len, q0 + 32) : len;
  const int nt = (kv_end + 31) / 32, mine = nt > wave ? (nt - wave + NW - 1) / NW : 0;
  const float scale = rsqrtf((float)p.d), c2 = scale * kLog2e;
  const unsigned ring = lds0 + wave * NB * STAGE;
  const char* ring_ptr = smem + wave * NB * STAGE;
  auto issue = [&](int j) {
    const unsigned st = ring + (unsigned)(j % NB) * STAGE;
    const int k0 = (wave + j * NW) * 32;
    Tile::template issue32<D>(base + H, ld3, k0, p.s, st, lane);
    Tile::template issue32<D>(base + 2 * H, ld3, k0, p.s, st + kTile32<DP>, lane);
  };
#pragma unroll
  for (int j = 0; j < NB; ++j)
    if (j < mine) issue(j);

  const bool in = q < p.s;
  const float my_lse2 = in ? p.lse[((size_t)n * p.heads + h) * p.s + q] * kLog2e : 0.f;
  bf16x8 qf[KS], cf[KS];
  float delta = 0.f;
#pragma unroll
  for (int kk = 0; kk < KS; ++kk) {
    const size_t at = ((size_t)n * p.s + q) * H + h * p.d;
    qf[kk] = frag_global(base + (size_t)q * ld3, in, kk, lane, p.d);
    cf[kk] = frag_global(p.dctx + at, in, kk, lane, p.d);
    const bf16x8 of = frag_global(p.ctx + at, in, kk, lane, p.d);
#pragma unroll
    for (int e = 0; e < 8; ++e) delta += (float)cf[kk][e] * (float)of[e];
  }
  delta = halves_sum(delta);
  f32x16 dq[DT];
#pragma unroll
  for (int dt = 0; dt < DT; ++dt) dq[dt] = zero16();
  for (int j = 0; j < mine; ++j) {
    if (NB > 1 && j + 1 < mine) wait_vmcnt<LOADS>();
    else wait_vmcnt<0>();
    const char* Ks = ring_ptr + (j % NB) * STAGE;
    const char* Vs = Ks + kTile32<DP>;
    const int k0 = (wave + j * NW) * 32;
    f32x16 sc = zero16(), dp = zero16();
#pragma unroll
    for (int kk = 0; kk < KS; ++kk) {
      sc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(Tile::frag_rows(Ks, fo, 0, kk), qf[kk], sc, 0, 0, 0);
      dp = __builtin_amdgcn_mfma_f32_32x32x16_bf16(Tile::frag_rows(Vs, fo, 0, kk), cf[kk], dp, 0, 0, 0);
    }
    if ((p.causal && k0 + 31 > q0) || k0 + 32 > len) {  // masked scores give P = 0
      asm volatile("");  // kept a branch: as selects the masks would cost every tile
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int key = k0 + acc_row(r, half);
        if (!(key < len && (!p.causal || key <= q))) sc[r] = -INFINITY;
      }
    }
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const float pr = __builtin_amdgcn_exp2f(fmaf(sc[r], c2, -my_lse2));
      dp[r] = pr * (dp[r] - delta);
    }
#pragma unroll
    for (int tt = 0; tt < 2; ++tt) {
      const bf16x8 dsf = pack_half(dp, tt);
#pragma unroll
      for (int dt = 0; dt < DT; ++dt)
        dq[dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(Tile::frag_cols(Ks, fo, 16 * tt, dt), dsf, dq[dt], 0, 0, 0);
    }
    if (j + NB < mine) {
      asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
      issue(j + NB);
    }
  }
  __syncthreads();
  float* parts = reinterpret_cast<float*>(smem);
  park<DP>(parts + wave * kPart<DP>, dq, lane);
  __syncthreads();
  sum_parts<DP, D>(parts, scale, p.dqkv + (size_t)n * p.s * ld3 + h * p.d, ld3, q0, p.s);
}

// dK and dV of 32 keys.
template <int DP, int D>
__device__ __forceinline__ void bwd_dkv(const AttnDev& p, char* smem, int kt, int h, int n) {
  using Tile = SwTile<DP>;
  constexpr int KS = D / 16, DT = (D + 31) / 32, NB = kBwdStages<D>, STAGE = kBwdStage<DP>, LOADS = 2 * Tile::kInstr32 + 1;
  const unsigned lds0 = (unsigned)(unsigned long)((__attribute__((address_space(3))) char*)smem);
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), half = lane >> 5;
  typename Tile::Offsets fo;
  Tile::init(fo, lane);
  const int H = p.heads * p.d, ld3 = 3 * H, k0 = kt * 32, key = k0 + (lane & 31);
  const bf16* base = p.qkv + (size_t)n * p.s * ld3 + h * p.d;
  const bf16* dcb = p.dctx + (size_t)n * p.s * H + h * p.d;
  const bf16* ctb = p.ctx + (size_t)n * p.s * H + h * p.d;
  const float* lse = p.lse + ((size_t)n * p.heads + h) * p.s;
  const int len = seq_len(p, n);
  const float scale = rsqrtf((float)p.d), c2 = scale * kLog2e;
  const int t_begin = p.causal ? kt : 0;
  const int t_end = k0 < len ? (p.s + 31) / 32 : 0;  // a tile of masked keys gets zero gradients
  const int nt = t_end > t_begin ? t_end - t_begin : 0, mine = nt > wave ? (nt - wave + NW - 1) / NW : 0;
  const unsigned ring = lds0 + wave * NB * STAGE;
  char* ring_ptr = smem + wave * NB * STAGE;
  auto issue = [&](int j) {
    const unsigned st = ring + (unsigned)(j % NB) * STAGE;
    const int q0 = (t_begin + wave + j * NW) * 32;
    Tile::template issue32<D>(base, ld3, q0, p.s, st, lane);
    Tile::template issue32<D>(dcb, H, q0, p.s, st + kTile32<DP>, lane);
    dma4(lse, (unsigned)(min(q0 + lane, p.s - 1) * 4), st + 2 * kTile32<DP>);
  };
#pragma unroll
  for (int j = 0; j < NB; ++j)
    if (j < mine) issue(j);

  bf16x8 kf[KS], vf[KS];
#pragma unroll
  for (int kk = 0; kk < KS; ++kk) {
    kf[kk] = frag_global(base + H + (size_t)key * ld3, key < p.s, kk, lane, p.d);
    vf[kk] = frag_global(base + 2 * H + (size_t)key * ld3, key < p.s, kk, lane, p.d);
  }
  f32x16 dk[DT], dv[DT];
#pragma unroll
  for (int dt = 0; dt < DT; ++dt) dk[dt] = dv[dt] = zero16();
  for (int j = 0; j < mine; ++j) {
    const int q0 = (t_begin + wave + j * NW) * 32;
    // this lane's row of C, for delta (these loads are younger than the ring's, whose wait below covers them too)
    bf16x8 of[KS];
    const int qr = min(q0 + (lane & 31), p.s - 1);
#pragma unroll
    for (int kk = 0; kk < KS; ++kk) of[kk] = *reinterpret_cast<const bf16x8*>(ctb + (size_t)qr * H + kk * 16 + 8 * half);
    if (NB > 1 && j + 1 < mine) wait_vmcnt<LOADS + KS>();
    else wait_vmcnt<KS>();
    char* Qs = ring_ptr + (j % NB) * STAGE;
    const char* Cs = Qs + kTile32<DP>;
    const float* lse_s = reinterpret_cast<const float*>(Qs + 2 * kTile32<DP>);
    float* dlt_s = reinterpret_cast<float*>(Qs + 2 * kTile32<DP> + 256);
    f32x16 sc = zero16(), dp = zero16();
    float delta = 0.f;
#pragma unroll
    for (int kk = 0; kk < KS; ++kk) {
      sc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(Tile::frag_rows(Qs, fo, 0, kk), kf[kk], sc, 0, 0, 0);
      const bf16x8 cr = Tile::frag_rows(Cs, fo, 0, kk);
      dp = __builtin_amdgcn_mfma_f32_32x32x16_bf16(cr, vf[kk], dp, 0, 0, 0);
#pragma unroll
      for (int e = 0; e < 8; ++e) delta += (float)cr[e] * (float)of[kk][e];
    }
    delta = halves_sum(delta);
    if (half == 0) dlt_s[lane] = delta;  // read back below by the same wavefront: LDS operations of one keep their order
    asm volatile("" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      const int ql = 8 * g + 4 * half;
      const f32x4 l4 = *reinterpret_cast<const f32x4*>(lse_s + ql);
      const f32x4 d4 = *reinterpret_cast<const f32x4*>(dlt_s + ql);
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int r = 4 * g + e;
        const float pr = __builtin_amdgcn_exp2f(fmaf(sc[r], c2, -l4[e] * kLog2e));
        sc[r] = pr;
        dp[r] = pr * (dp[r] - d4[e]);
      }
    }
    if ((p.causal && q0 < k0 + 31) || k0 + 31 >= len || q0 + 31 >= p.s) {
      asm volatile("");  // kept a branch: as selects the masks would cost every tile
#pragma unroll
      for (int r = 0; r < 16; ++r) {  // P and dS themselves: a query whose log-sum-exp or delta is NaN must not reach keys behind the mask
        const int qq = q0 + acc_row(r, half);
        if (!(qq < p.s && key < len && (!p.causal || key <= qq))) sc[r] = dp[r] = 0.f;
      }
    }
#pragma unroll
    for (int tt = 0; tt < 2; ++tt) {
      const bf16x8 pf = pack_half(sc, tt), dsf = pack_half(dp, tt);
#pragma unroll
      for (int dt = 0; dt < DT; ++dt) {
        dv[dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(Tile::frag_cols(Cs, fo, 16 * tt, dt), pf, dv[dt], 0, 0, 0);
        dk[dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(Tile::frag_cols(Qs, fo, 16 * tt, dt), dsf, dk[dt], 0, 0, 0);
      }
    }
    if (j + NB < mine) {
      asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
      issue(j + NB);
    }
  }
  float* parts = reinterpret_cast<float*>(smem);
  bf16* out = p.dqkv + (size_t)n * p.s * ld3 + h * p.d;
  __syncthreads();
  park<DP>(parts + wave * kPart<DP>, dk, lane);
  __syncthreads();
  sum_parts<DP, D>(parts, scale, out + H, ld3, k0, p.s);
  __syncthreads();
  park<DP>(parts + wave * kPart<DP>, dv, lane);
  __syncthreads();
  sum_parts<DP, D>(parts, 1.f, out + 2 * H, ld3, k0, p.s);
}

// dK / dV of every key tile, then dQ of every query tile: the longer work first.
template <int DP, int D>
__device__ __forceinline__ void bwd_split(const AttnDev& p, int pairs, int tiles) {
  extern __shared__ __attribute__((aligned(1024))) char smem[];
  const int per_side = pairs * tiles, side = (int)blockIdx.x >= per_side;
  int t, h, n;
  place(p, (int)blockIdx.x - side * per_side, pairs, t, h, n);
  if (side) bwd_dq<DP, D>(p, smem, tiles - 1 - t, h, n);
  else bwd_dkv<DP, D>(p, smem, t, h, n);
}
template <int DP, int D>
__global__ __launch_bounds__(NW * 64) void attn_bwd_split_kernel(int pairs, int tiles, ATTN_PARAMS) {
  const AttnDev p = ATTN_BLOCK;
  bwd_split<DP, D>(p, pairs, tiles);
}
// The same in at most 256 registers, for two workgroups on a CU.
template <int DP, int D>
__global__ __launch_bounds__(NW * 64) __attribute__((amdgpu_waves_per_eu(2, 2))) void attn_bwd_split2_kernel(int pairs, int tiles,
                                                                                                          ATTN_PARAMS) {
  const AttnDev p = ATTN_BLOCK;
  bwd_split<DP, D>(p, pairs, tiles);
}

AttnDev to_dev(const AttnArgs& a) {
  AttnDev p;
  p.qkv = (const bf16*)a.qkv; p.valid_len = a.valid_len; p.ctx = (bf16*)a.ctx; p.lse = a.lse;
  p.dctx = (const bf16*)a.dctx; p.dqkv = (bf16*)a.dqkv; p.delta = a.delta;
  p.s = a.s; p.heads = a.heads; p.d = a.d; p.causal = a.causal ? 1 : 0;
  return p;
}

template <int DP, int D>
int forward_t(const AttnArgs& a, hipStream_t stream) {
  static thread_local uint64_t raised = 0;
  constexpr size_t lds = lds_bytes<DP>(2 * kTile32<DP>);
  if (const int rc = raise_lds(reinterpret_cast<const void*>(attn_fwd_split_kernel<DP, D>), lds, raised)) return rc;
  const AttnDev p = to_dev(a);
  const int pairs = a.heads * a.b, tiles = (a.s + 31) / 32;
  launch_kernel((attn_fwd_split_kernel<DP, D>), dim3(pairs * tiles), dim3(NW * 64), lds, stream, pairs, tiles, ATTN_ARGS(p));
  return check_launch("attn_fwd_split");
}
template <int DP, int D>
int backward_t(const AttnArgs& a, hipStream_t stream) {
  static thread_local uint64_t raised = 0;
  constexpr size_t lds = lds_bytes<DP>(kBwdStage<DP>, kBwdStages<D>);
  void (*kern)(int, int, ATTN_PARAMS);
  if constexpr (kBwdStages<D> == 1) kern = attn_bwd_split2_kernel<DP, D>;
  else kern = attn_bwd_split_kernel<DP, D>;
  if (const int rc = raise_lds(reinterpret_cast<const void*>(kern), lds, raised)) return rc;
  const AttnDev p = to_dev(a);
  const int pairs = a.heads * a.b, tiles = (a.s + 31) / 32;
  launch_kernel(kern, dim3(2 * pairs * tiles), dim3(NW * 64), lds, stream, pairs, tiles, ATTN_ARGS(p));
  return check_launch("attn_bwd_split");
}

}  // namespace

int attn_forward_split(const AttnArgs& a, hipStream_t stream) {
  switch (a.d) {
    case 32: return forward_t<64, 32>(a, stream);
    case 64: return forward_t<64, 64>(a, stream);
    case 80: return forward_t<128, 80>(a, stream);
    case 96: return forward_t<128, 96>(a, stream);
    case 128: return forward_t<128, 128>(a, stream);
  }
  return set_error(HANAYO_EUNSUPPORTED, "attn_split: head dim %d", a.d);
}

int attn_backward_split(const AttnArgs& a, hipStream_t stream) {
  switch (a.d) {
    case 32: return backward_t<64, 32>(a, stream);
    case 64: return backward_t<64, 64>(a, stream);
    case 80: return backward_t<128, 80>(a, stream);
    case 96: return backward_t<128, 96>(a, stream);
    case 128: return backward_t<128, 128>(a, stream);
  }
  return set_error(HANAYO_EUNSUPPORTED, "attn_split: head dim %d", a.d);
}

}  // namespace k
}  // namespace hanayo
