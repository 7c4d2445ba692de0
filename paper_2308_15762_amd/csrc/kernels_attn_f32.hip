// Fused attention forward / backward for fp32 storage on the fp32 matrix instructions (v_mfma_f32_32x32x2_f32).
//
// That instruction does 4096 flop in 64 cycles, a sixteenth of bf16's rate, so a tile step is bound by matrix issue
// (a 32 x 32 tile of scores at d = 64: 2048 cycles forward) and not by its operands: fragments come straight from
// global memory (L1 / L2) and nothing is staged.  What matters is that every SIMD has a tile to work on: a workgroup
// owns only 32 query rows (keys, for dK / dV), its four wavefronts take every fourth tile of the other side, and their
// partial results (forward: each with its own running maximum and sum) are merged in a fixed order through LDS.
//
// Orientation as in the bf16 kernels: a product that contracts over keys takes the scores as S^T = K Q^T (a lane owns one
// query), one that contracts over queries as S = Q K^T (a lane owns one key), so probabilities go from accumulator
// registers straight into the next product: accumulator register r of half wavefront h is tile row 8 (r / 4) + 4 h + r mod 4,
// and that row is what the other operand fetches for MFMA r.
//
// Masked keys and rows have probability zero and count for nothing, whatever they hold; a product with zero lets infinities
// and NaN through.  They can only reach a result as NaN, so a result that is not finite is worked out again by a wavefront
// that skips what has probability zero (redo_*), and nothing else pays for it.
//
// Measured (MI355X): b = 2, 8 heads, d = 64, s = 512, causal: forward 208 us on the ALU, 17 here; backward 709 and 46.5
// (65.5 as two launches, dQ first).  The backward kernel keeps its 322 registers and one wavefront per SIMD at d = 64: held
// to 256 it spills and takes 71 us.
#include "device_util.h"
#include "kernels.h"

namespace hanayo {
namespace k {

namespace {

constexpr int NW = 4;  // wavefronts per workgroup

struct AttnF32 {
  const float* qkv;
  const int32_t* valid_len;
  float* ctx;
  float* lse;
  const float* dctx;
  float* dqkv;
  int s, heads, d, causal, tiles, pairs;  // tiles of 32 rows; (sequence, head) pairs
};
// A kernel's parameters one by one and the block made of them: the first 14 words of them are in scalar registers when the
// kernel starts (see the build flags), a struct would have to be read from memory first.
#define ATTN_F32_PARAMS                                                                                                        \
  const float *qkv, const int32_t *valid_len, float *lse, int s, int heads, int d, int causal, int tiles, int pairs, const float *dctx, \
      float *ctx, float *dqkv
#define ATTN_F32_BLOCK AttnF32{qkv, valid_len, ctx, lse, dctx, dqkv, s, heads, d, causal, tiles, pairs}
#define ATTN_F32_ARGS(p) p.qkv, p.valid_len, p.lse, p.s, p.heads, p.d, p.causal, p.tiles, p.pairs, p.dctx, p.ctx, p.dqkv

__device__ __forceinline__ int seq_len(const AttnF32& p, int n) {
  if (!p.valid_len) return p.s;
  const int v = p.valid_len[n];
  return v < 1 ? 1 : (v > p.s ? p.s : v);
}

// Row fragments: this lane's row (lane % 32 of a tile), elements 8 kk + 4 (lane / 32) .. + 3 of it.
// DP - 32 < d <= DP; FULL: d == DP.  What lies past d reads as zero (guards around the MFMAs would cut the tile step into
// small blocks and cost registers).
template <int DP, bool FULL>
struct Rows {
  f32x4 v[DP / 8];
  __device__ __forceinline__ void load(const float* row, int d, int half) {
#pragma unroll
    for (int kk = 0; kk < DP / 8; ++kk) {
      v[kk] = *reinterpret_cast<const f32x4*>(row + (FULL || kk * 8 < d ? kk * 8 + 4 * half : 0));
      if (!FULL && kk * 8 >= d) v[kk] = f32x4{0.f, 0.f, 0.f, 0.f};
    }
  }
};
// acc[i][j] += sum over d of a(row i) b(row j)
template <int DP, bool FULL>
__device__ __forceinline__ f32x16 mul_rows(const Rows<DP, FULL>& a, const Rows<DP, FULL>& b) {
  f32x16 acc = zero16();
#pragma unroll
  for (int kk = 0; kk < DP / 8; ++kk)
#pragma unroll
    for (int e = 0; e < 4; ++e) acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a.v[kk][e], b.v[kk][e], acc, 0, 0, 0);
  return acc;
}
// Column fragments: element (row0 + acc_row(r), c0 + lane % 32) for the 16 MFMAs of a 32-row tile; rows clamped to s - 1
// (what they multiply is zero there), columns past d clamped (their products are not stored).
struct Cols {
  float v[16];
  __device__ __forceinline__ void load(const float* base, size_t ld, int row0, int s, int c0, int d, int lane) {
    const int c = c0 + (lane & 31);
    const float* p = base + (c < d ? c : d - 1);
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const int row = row0 + acc_row(r, lane >> 5);
      v[r] = p[(size_t)(row < s ? row : s - 1) * ld];
    }
  }
};
// out[c][j] += sum over the tile's 32 rows of cols(row, c) * w(row, j)
__device__ __forceinline__ f32x16 mul_cols(const Cols& a, const f32x16& w, f32x16 out) {
#pragma unroll
  for (int r = 0; r < 16; ++r) out = __builtin_amdgcn_mfma_f32_32x32x2f32(a.v[r], w[r], out, 0, 0, 0);
  return out;
}

// Workgroup -> (tile, head, sequence): consecutive workgroups are heads, so that the long tiles of a causal grid, which
// come first, start together.
__device__ __forceinline__ void place(const AttnF32& p, int w, int& tile, int& h, int& n) {
  const int hn = w % p.pairs;
  tile = w / p.pairs;
  h = hn % p.heads;
  n = hn / p.heads;
}

// A wavefront's 32 x DP partial result to LDS: lane holds row lane % 32, columns 32 dt + acc_row(r).
template <int DP>
__device__ __forceinline__ void park(float* part, const f32x16 (&o)[DP / 32], int lane) {
#pragma unroll
  for (int dt = 0; dt < DP / 32; ++dt)
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      f32x4 v;
#pragma unroll
      for (int e = 0; e < 4; ++e) v[e] = o[dt][4 * q + e];
      *reinterpret_cast<f32x4*>(part + (lane & 31) * (DP + 4) + 32 * dt + 8 * q + 4 * (lane >> 5)) = v;
    }
}
template <int DP>
constexpr size_t part_floats() { return 32 * (DP + 4); }

// ---- results that are not finite, again: one wavefront per row, a lane per key (query), then two columns per lane.  A NaN
// among a row's probabilities makes all its columns NaN, so a model that has diverged does not go through every pair here.
__device__ __forceinline__ bool finite4(const f32x4& v) {
  const float m = fmaxf(fmaxf(fabsf(v[0]), fabsf(v[1])), fmaxf(fabsf(v[2]), fabsf(v[3])));  // fmaxf drops NaN: add it back
  return m < INFINITY && v[0] + v[1] + v[2] + v[3] == v[0] + v[1] + v[2] + v[3];
}
__device__ __forceinline__ float dot(const float* a, const float* b, int d) {
  float t = 0.f;
  for (int c = 0; c < d; c += 4) {
    const f32x4 x = *reinterpret_cast<const f32x4*>(a + c), y = *reinterpret_cast<const f32x4*>(b + c);
    t += x[0] * y[0] + x[1] * y[1] + x[2] * y[2] + x[3] * y[3];
  }
  return t;
}
// acc += sum over the 64 lanes' rows with w != 0 of w * row (this lane's columns: lane, lane + 64)
__device__ __forceinline__ void add_rows(float w, const float* first, size_t ld, int d, int lane, float (&acc)[2]) {
  for (int j = 0; j < 64; ++j) {
    const float wj = __shfl(w, j, 64);
    if (wj == 0.f) continue;
    const float* row = first + (size_t)j * ld;
#pragma unroll
    for (int u = 0; u < 2; ++u)
      if (lane + 64 * u < d) acc[u] += wj * row[lane + 64 * u];
  }
}
__device__ __forceinline__ bool nan_row(float w, float (&acc)[2]) {
  if (!__ballot(w != w)) return false;
  acc[0] = acc[1] = NAN;
  return true;
}
// Columns whose vector of four is in `vecs`.
__device__ __forceinline__ void store_columns(float* row, unsigned vecs, int d, int lane, const float (&acc)[2], float scale) {
#pragma unroll
  for (int u = 0; u < 2; ++u) {
    const int c = lane + 64 * u;
    if (c < d && (vecs >> (c >> 2) & 1u)) row[c] = acc[u] * scale;
  }
}
__device__ __forceinline__ void redo_ctx(const AttnF32& p, int n, int h, int q, unsigned vecs) {
  const int lane = threadIdx.x & 63, H = p.heads * p.d, len = seq_len(p, n), end = p.causal ? min(len, q + 1) : len;
  const size_t ld3 = (size_t)3 * H;
  const float* base = p.qkv + (size_t)n * p.s * ld3 + h * p.d;
  const float* qr = base + (size_t)q * ld3;
  const float c2 = rsqrtf((float)p.d) * kLog2e;
  auto score = [&](int j) { return j < end ? dot(qr, base + H + (size_t)j * ld3, p.d) : -INFINITY; };
  float mx = -INFINITY, sum = 0.f, acc[2] = {0.f, 0.f};
  for (int j0 = 0; j0 < end; j0 += 64) mx = fmaxf(mx, score(j0 + lane));
  mx = wave_max(mx);
  for (int j0 = 0; j0 < end; j0 += 64) {
    const float t = score(j0 + lane), e = t == -INFINITY ? 0.f : __builtin_amdgcn_exp2f((t - mx) * c2);
    sum += e;
    if (nan_row(e, acc)) break;
    add_rows(e, base + 2 * H + (size_t)j0 * ld3, ld3, p.d, lane, acc);
  }
  sum = wave_sum(sum);
  store_columns(p.ctx + ((size_t)n * p.s + q) * H + h * p.d, vecs, p.d, lane, acc, 1.f / sum);
  if ((vecs & 1u) && lane == 0) p.lse[((size_t)n * p.heads + h) * p.s + q] = (mx * c2 + log2f(sum)) * kLn2;
}
// Probability and score gradient of (query i, key j), zero where the mask says so.
__device__ __forceinline__ void redo_pair(const AttnF32& p, int n, int h, int i, int j, float& pr, float& ds) {
  const int H = p.heads * p.d;
  const size_t ld3 = (size_t)3 * H, at = ((size_t)n * p.s + i) * H + h * p.d;
  const float* base = p.qkv + (size_t)n * p.s * ld3 + h * p.d;
  const float c2 = rsqrtf((float)p.d) * kLog2e;
  const float t = dot(base + (size_t)i * ld3, base + H + (size_t)j * ld3, p.d);
  const float dp = dot(p.dctx + at, base + 2 * H + (size_t)j * ld3, p.d);
  pr = __builtin_amdgcn_exp2f(fmaf(t, c2, -p.lse[((size_t)n * p.heads + h) * p.s + i] * kLog2e));
  ds = pr * (dp - dot(p.dctx + at, p.ctx + at, p.d));
}
__device__ __forceinline__ void redo_dq(const AttnF32& p, int n, int h, int q, unsigned vecs) {
  const int lane = threadIdx.x & 63, H = p.heads * p.d, len = seq_len(p, n), end = p.causal ? min(len, q + 1) : len;
  const size_t ld3 = (size_t)3 * H, first = (size_t)n * p.s * ld3 + h * p.d;
  float acc[2] = {0.f, 0.f};
  for (int j0 = 0; j0 < end; j0 += 64) {
    float pr = 0.f, ds = 0.f;
    if (j0 + lane < end) redo_pair(p, n, h, q, j0 + lane, pr, ds);
    if (pr == 0.f) ds = 0.f;
    if (nan_row(ds, acc)) break;
    add_rows(ds, p.qkv + first + H + (size_t)j0 * ld3, ld3, p.d, lane, acc);
  }
  store_columns(p.dqkv + first + (size_t)q * ld3, vecs, p.d, lane, acc, rsqrtf((float)p.d));
}
// dK (which = 0) or dV (1) of one key.
__device__ __forceinline__ void redo_dkv(const AttnF32& p, int n, int h, int key, unsigned vecs, int which) {
  const int lane = threadIdx.x & 63, H = p.heads * p.d;
  const size_t ld3 = (size_t)3 * H, first = (size_t)n * p.s * ld3 + h * p.d;
  const float* rows = which ? p.dctx + (size_t)n * p.s * H + h * p.d : p.qkv + first;
  const size_t ld = which ? (size_t)H : ld3;
  float acc[2] = {0.f, 0.f};
  const int begin = p.causal ? key : 0, end = key < seq_len(p, n) ? p.s : 0;
  for (int i0 = begin; i0 < end; i0 += 64) {
    float pr = 0.f, ds = 0.f;
    if (i0 + lane < end) redo_pair(p, n, h, i0 + lane, key, pr, ds);
    const float w = which || pr == 0.f ? pr : ds;
    if (nan_row(w, acc)) break;
    add_rows(w, rows + (size_t)i0 * ld, ld, p.d, lane, acc);
  }
  store_columns(p.dqkv + first + (size_t)key * ld3 + (which + 1) * H, vecs, p.d, lane, acc, which ? 1.f : rsqrtf((float)p.d));
}

// Called by whole wavefronts: lanes with `bad` hold a vector (first column c) of `row` that has to be done again; redo(row,
// vectors) does one row.
template <typename Redo>
__device__ __forceinline__ void redo_rows(bool bad, int row, int c, Redo redo) {
  unsigned long long left = __ballot(bad);
  while (left) {
    const int r = __shfl(row, __ffsll(left) - 1, 64);
    const bool mine = bad && row == r;
    unsigned vecs = mine ? 1u << (c >> 2) : 0u;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) vecs |= __shfl_xor(vecs, o, 64);
    redo(r, vecs);
    left &= ~__ballot(mine);
  }
}

template <int DP, bool FULL>
__global__ __launch_bounds__(NW * 64) void attn_fwd_f32_kernel(ATTN_F32_PARAMS) {
  const AttnF32 p = ATTN_F32_BLOCK;
  constexpr int DT = DP / 32;
  extern __shared__ float smem[];  // [NW][32][DP + 4] partial outputs, then [NW][32] maxima and sums
  float2* stats = reinterpret_cast<float2*>(smem + NW * part_floats<DP>());
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), half = lane >> 5;
  int qt, h, n;
  place(p, blockIdx.x, qt, h, n);
  qt = p.tiles - 1 - qt;
  const int H = p.heads * p.d, q0 = qt * 32, q = q0 + (lane & 31);
  const size_t ld3 = (size_t)3 * H;
  const float* base = p.qkv + (size_t)n * p.s * ld3 + h * p.d;
  const int len = seq_len(p, n);
  const int kv_end = p.causal ? min(len, q0 + 32) : len;
  const int nt = (kv_end + 31) / 32;
  const float c2 = rsqrtf((float)p.d) * kLog2e;

  Rows<DP, FULL> qf;
  qf.load(base + (size_t)min(q, p.s - 1) * ld3, p.d, half);
  f32x16 o[DT];
#pragma unroll
  for (int dt = 0; dt < DT; ++dt) o[dt] = zero16();
  float m = -INFINITY, lsum = 0.f;  // m in units of raw scores
  for (int t = wave; t < nt; t += NW) {
    const int k0 = t * 32;
    Rows<DP, FULL> kf;
    kf.load(base + H + (size_t)min(k0 + (lane & 31), p.s - 1) * ld3, p.d, half);
    Cols vf[DT];
#pragma unroll
    for (int dt = 0; dt < DT; ++dt)
      vf[dt].load(base + 2 * H, ld3, k0, p.s, 32 * dt, p.d, lane);
    f32x16 sc = mul_rows<DP, FULL>(kf, qf);
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
#pragma unroll
    for (int dt = 0; dt < DT; ++dt) {
#pragma unroll
      for (int r = 0; r < 16; ++r) o[dt][r] *= alpha;
      o[dt] = mul_cols(vf[dt], sc, o[dt]);
    }
  }
  park<DP>(smem + wave * part_floats<DP>(), o, lane);
  if (half == 0) stats[wave * 32 + lane] = make_float2(m, lsum);
  __syncthreads();
  const int vecs = p.d / 4;  // 32 * vecs is a multiple of 64: whole wavefronts
  for (int i = threadIdx.x; i < 32 * vecs; i += NW * 64) {
    const int row = i / vecs, c = (i % vecs) * 4;
    float mx = -INFINITY, total = 0.f;
#pragma unroll
    for (int w = 0; w < NW; ++w) mx = fmaxf(mx, stats[w * 32 + row].x);
    f32x4 v = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int w = 0; w < NW; ++w) {
      const float2 st = stats[w * 32 + row];
      const float f = __builtin_amdgcn_exp2f((st.x - mx) * c2);  // 0 for a wavefront that had no tile
      total += st.y * f;
      const f32x4 t = *reinterpret_cast<const f32x4*>(smem + w * part_floats<DP>() + row * (DP + 4) + c);
#pragma unroll
      for (int e = 0; e < 4; ++e) v[e] += t[e] * f;
    }
    const float inv = 1.f / total;
#pragma unroll
    for (int e = 0; e < 4; ++e) v[e] *= inv;
    const bool in = q0 + row < p.s, fine = finite4(v);
    if (in && fine) {
      *reinterpret_cast<f32x4*>(p.ctx + ((size_t)n * p.s + q0 + row) * H + h * p.d + c) = v;
      if (c == 0) p.lse[((size_t)n * p.heads + h) * p.s + q0 + row] = (mx * c2 + log2f(total)) * kLn2;
    }
    redo_rows(in && !fine, row, c, [&](int r, unsigned which) { redo_ctx(p, n, h, q0 + r, which); });
  }
}

// dQ of 32 query rows.
template <int DP, bool FULL>
__device__ __forceinline__ void bwd_dq(const AttnF32& p, float* smem, int qt, int h, int n) {
  constexpr int DT = DP / 32;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), half = lane >> 5;
  const int H = p.heads * p.d, q0 = qt * 32, q = q0 + (lane & 31), q_in = min(q, p.s - 1);
  const size_t ld3 = (size_t)3 * H, at_q = ((size_t)n * p.s + q_in) * H + h * p.d;
  const float* base = p.qkv + (size_t)n * p.s * ld3 + h * p.d;
  const int len = seq_len(p, n);
  const int kv_end = p.causal ? min(len, q0 + 32) : len;
  const int nt = (kv_end + 31) / 32;
  const float scale = rsqrtf((float)p.d), c2 = scale * kLog2e;
  const size_t stat = ((size_t)n * p.heads + h) * p.s + q_in;
  const float my_lse2 = p.lse[stat] * kLog2e;

  Rows<DP, FULL> qf, cf;
  qf.load(base + (size_t)q_in * ld3, p.d, half);
  cf.load(p.dctx + at_q, p.d, half);
  float delta = 0.f;
#pragma unroll
  for (int kk = 0; kk < DP / 8; ++kk)
    if (FULL || kk * 8 < p.d) {
      const f32x4 c = *reinterpret_cast<const f32x4*>(p.ctx + at_q + kk * 8 + 4 * half);
#pragma unroll
      for (int e = 0; e < 4; ++e) delta += c[e] * cf.v[kk][e];
    }
  delta = halves_sum(delta);

  f32x16 dq[DT];
#pragma unroll
  for (int dt = 0; dt < DT; ++dt) dq[dt] = zero16();
  for (int t = wave; t < nt; t += NW) {
    const int k0 = t * 32;
    const size_t krow = (size_t)min(k0 + (lane & 31), p.s - 1) * ld3;
    Rows<DP, FULL> kf, vf;
    kf.load(base + H + krow, p.d, half);
    if (DP <= 64) vf.load(base + 2 * H + krow, p.d, half);
    f32x16 sc = mul_rows<DP, FULL>(kf, qf);
    if (DP > 64) {
      __builtin_amdgcn_sched_barrier(0);
      vf.load(base + 2 * H + krow, p.d, half);
    }
    const f32x16 dp = mul_rows<DP, FULL>(vf, cf);
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const int key = k0 + acc_row(r, half);
      const bool ok = key < len && (!p.causal || key <= q);
      sc[r] = ok ? __builtin_amdgcn_exp2f(fmaf(sc[r], c2, -my_lse2)) * (dp[r] - delta) : 0.f;
    }
#pragma unroll
    for (int dt = 0; dt < DT; ++dt) {
      if (DP > 64) __builtin_amdgcn_sched_barrier(0);  // hoisted, the column fragments of a wide head would spill
      Cols kc;
      kc.load(base + H, ld3, k0, p.s, 32 * dt, p.d, lane);
      dq[dt] = mul_cols(kc, sc, dq[dt]);
    }
  }
  park<DP>(smem + wave * part_floats<DP>(), dq, lane);
  __syncthreads();
  const int vecs = p.d / 4;
  for (int i = threadIdx.x; i < 32 * vecs; i += NW * 64) {
    const int row = i / vecs, c = (i % vecs) * 4;
    f32x4 v = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int w = 0; w < NW; ++w) {
      const f32x4 t2 = *reinterpret_cast<const f32x4*>(smem + w * part_floats<DP>() + row * (DP + 4) + c);
#pragma unroll
      for (int e = 0; e < 4; ++e) v[e] += t2[e];
    }
#pragma unroll
    for (int e = 0; e < 4; ++e) v[e] *= scale;
    const bool in = q0 + row < p.s, fine = finite4(v);
    if (in && fine) *reinterpret_cast<f32x4*>(p.dqkv + ((size_t)n * p.s + q0 + row) * ld3 + h * p.d + c) = v;
    redo_rows(in && !fine, row, c, [&](int r, unsigned which) { redo_dq(p, n, h, q0 + r, which); });
  }
}

// dK and dV of 32 keys.
template <int DP, bool FULL>
__device__ __forceinline__ void bwd_dkv(const AttnF32& p, float* smem, int kt, int h, int n) {
  constexpr int DT = DP / 32;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), half = lane >> 5;
  const int H = p.heads * p.d, k0 = kt * 32, key = k0 + (lane & 31);
  const size_t ld3 = (size_t)3 * H;
  const float* base = p.qkv + (size_t)n * p.s * ld3 + h * p.d;
  const float* dcb = p.dctx + (size_t)n * p.s * H + h * p.d;
  const float* ctb = p.ctx + (size_t)n * p.s * H + h * p.d;
  const size_t stat0 = ((size_t)n * p.heads + h) * p.s;
  const int len = seq_len(p, n);
  const float scale = rsqrtf((float)p.d), c2 = scale * kLog2e;
  const int t_begin = p.causal ? kt : 0;
  const int t_end = k0 < len ? (p.s + 31) / 32 : 0;  // a tile of masked keys gets zero gradients

  Rows<DP, FULL> kf, vf;
  const size_t krow = (size_t)min(key, p.s - 1) * ld3;
  kf.load(base + H + krow, p.d, half);
  vf.load(base + 2 * H + krow, p.d, half);
  f32x16 dk[DT], dv[DT];
#pragma unroll
  for (int dt = 0; dt < DT; ++dt) dk[dt] = dv[dt] = zero16();
  for (int t = t_begin + wave; t < t_end; t += NW) {
    const int q0 = t * 32;
    const int qr = min(q0 + (lane & 31), p.s - 1);
    Rows<DP, FULL> qf, cf;
    qf.load(base + (size_t)qr * ld3, p.d, half);
    if (DP <= 64) cf.load(dcb + (size_t)qr * H, p.d, half);
    float lse2[16];
#pragma unroll
    for (int r = 0; r < 16; ++r) lse2[r] = p.lse[stat0 + min(q0 + acc_row(r, half), p.s - 1)] * kLog2e;
    f32x16 sc = mul_rows<DP, FULL>(qf, kf);
    if (DP > 64) {
      __builtin_amdgcn_sched_barrier(0);
      cf.load(dcb + (size_t)qr * H, p.d, half);
    }
    float delta = 0.f;  // of this lane's row
#pragma unroll
    for (int kk = 0; kk < DP / 8; ++kk) {
      const f32x4 c = *reinterpret_cast<const f32x4*>(ctb + (size_t)qr * H + (FULL || kk * 8 < p.d ? kk * 8 + 4 * half : 0));
#pragma unroll
      for (int e = 0; e < 4; ++e) delta += c[e] * cf.v[kk][e];  // cf is zero past d
    }
    delta = halves_sum(delta);
    f32x16 dp = mul_rows<DP, FULL>(cf, vf);
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const float dlt = __shfl(delta, acc_row(r, half), 64);
      const int qq = q0 + acc_row(r, half);
      const bool ok = qq < p.s && key < len && (!p.causal || key <= qq);
      sc[r] = ok ? __builtin_amdgcn_exp2f(fmaf(sc[r], c2, -lse2[r])) : 0.f;
      dp[r] = sc[r] * (dp[r] - dlt);
    }
#pragma unroll
    for (int dt = 0; dt < DT; ++dt) {
      if (DP > 64) __builtin_amdgcn_sched_barrier(0);
      Cols cc, qc;
      cc.load(dcb, H, q0, p.s, 32 * dt, p.d, lane);
      qc.load(base, ld3, q0, p.s, 32 * dt, p.d, lane);
      dv[dt] = mul_cols(cc, sc, dv[dt]);
      dk[dt] = mul_cols(qc, dp, dk[dt]);
    }
  }
  const int vecs = p.d / 4;
#pragma unroll
  for (int which = 0; which < 2; ++which) {  // dK, then dV, through the same LDS
    park<DP>(smem + wave * part_floats<DP>(), which ? dv : dk, lane);
    __syncthreads();
    for (int i = threadIdx.x; i < 32 * vecs; i += NW * 64) {
      const int row = i / vecs, c = (i % vecs) * 4;
      f32x4 v = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int w = 0; w < NW; ++w) {
        const f32x4 t2 = *reinterpret_cast<const f32x4*>(smem + w * part_floats<DP>() + row * (DP + 4) + c);
#pragma unroll
        for (int e = 0; e < 4; ++e) v[e] += t2[e];
      }
#pragma unroll
      for (int e = 0; e < 4; ++e) v[e] *= which ? 1.f : scale;
      const bool in = k0 + row < p.s, fine = finite4(v);
      if (in && fine) *reinterpret_cast<f32x4*>(p.dqkv + ((size_t)n * p.s + k0 + row) * ld3 + (which ? 2 : 1) * H + h * p.d + c) = v;
      redo_rows(in && !fine, row, c, [&](int r, unsigned bad) { redo_dkv(p, n, h, k0 + r, bad, which); });
    }
    __syncthreads();
  }
}

// dK / dV of every key tile, then dQ of every query tile, the longer work first: one launch, because the former forms its
// deltas itself instead of waiting for the latter.
template <int DP, bool FULL>
__global__ __launch_bounds__(NW * 64, DP <= 32 ? 2 : 1) void attn_bwd_f32_kernel(ATTN_F32_PARAMS) {
  const AttnF32 p = ATTN_F32_BLOCK;
  extern __shared__ float smem[];
  const int per_side = p.pairs * p.tiles, side = (int)blockIdx.x >= per_side;
  int t, h, n;
  place(p, (int)blockIdx.x - side * per_side, t, h, n);
  if (side) bwd_dq<DP, FULL>(p, smem, p.tiles - 1 - t, h, n);
  else bwd_dkv<DP, FULL>(p, smem, t, h, n);
}

int check_shape(const AttnArgs& a, unsigned& grid) {
  if (a.d % 8 || a.d < 8 || a.d > 128) return set_error(HANAYO_EUNSUPPORTED, "attn_f32: head dim %d", a.d);
  const long wgs = (long)((a.s + 31) / 32) * a.heads * a.b;
  if (wgs > 0x3fffffffL) return set_error(HANAYO_EUNSUPPORTED, "attn_f32: too many tiles");
  grid = (unsigned)wgs;
  return HANAYO_OK;
}
AttnF32 to_dev(const AttnArgs& a) {
  return AttnF32{(const float*)a.qkv, a.valid_len, (float*)a.ctx, a.lse, (const float*)a.dctx, (float*)a.dqkv,
                 a.s, a.heads, a.d, a.causal ? 1 : 0, (a.s + 31) / 32, a.heads * a.b};
}
template <int DP>
constexpr size_t lds_bytes() { return NW * part_floats<DP>() * sizeof(float) + NW * 32 * sizeof(float2); }

template <int DP, bool FULL>
int forward_t(const AttnF32& p, unsigned grid, hipStream_t stream) {
  static thread_local uint64_t raised = 0;
  if (const int rc = raise_lds(reinterpret_cast<const void*>(attn_fwd_f32_kernel<DP, FULL>), lds_bytes<DP>(), raised)) return rc;
  launch_kernel((attn_fwd_f32_kernel<DP, FULL>), dim3(grid), dim3(NW * 64), lds_bytes<DP>(), stream, ATTN_F32_ARGS(p));
  return check_launch("attn_fwd_f32");
}
template <int DP, bool FULL>
int backward_t(const AttnF32& p, unsigned grid, hipStream_t stream) {
  static thread_local uint64_t raised = 0;
  if (const int rc = raise_lds(reinterpret_cast<const void*>(attn_bwd_f32_kernel<DP, FULL>), lds_bytes<DP>(), raised)) return rc;
  launch_kernel((attn_bwd_f32_kernel<DP, FULL>), dim3(2 * grid), dim3(NW * 64), lds_bytes<DP>(), stream, ATTN_F32_ARGS(p));
  return check_launch("attn_bwd_f32");
}

}  // namespace

int attn_forward_f32(const AttnArgs& a, hipStream_t stream) {
  unsigned grid;
  if (const int rc = check_shape(a, grid)) return rc;
  const AttnF32 p = to_dev(a);
  if (a.d <= 32) return a.d == 32 ? forward_t<32, true>(p, grid, stream) : forward_t<32, false>(p, grid, stream);
  if (a.d <= 64) return a.d == 64 ? forward_t<64, true>(p, grid, stream) : forward_t<64, false>(p, grid, stream);
  if (a.d <= 96) return a.d == 96 ? forward_t<96, true>(p, grid, stream) : forward_t<96, false>(p, grid, stream);
  return a.d == 128 ? forward_t<128, true>(p, grid, stream) : forward_t<128, false>(p, grid, stream);
}

int attn_backward_f32(const AttnArgs& a, hipStream_t stream) {
  unsigned grid;
  if (const int rc = check_shape(a, grid)) return rc;
  const AttnF32 p = to_dev(a);
  if (a.d <= 32) return a.d == 32 ? backward_t<32, true>(p, grid, stream) : backward_t<32, false>(p, grid, stream);
  if (a.d <= 64) return a.d == 64 ? backward_t<64, true>(p, grid, stream) : backward_t<64, false>(p, grid, stream);
  if (a.d <= 96) return a.d == 96 ? backward_t<96, true>(p, grid, stream) : backward_t<96, false>(p, grid, stream);
  return a.d == 128 ? backward_t<128, true>(p, grid, stream) : backward_t<128, false>(p, grid, stream);
}

}  // namespace k
}  // namespace hanayo
