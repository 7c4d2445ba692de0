// chunk_forward / chunk_backward: the fixed kernel sequence of n_blocks
// transformer blocks for one micro-batch (the paper's T_F / 2W and T_B / 2W
// units of work), plus the dispatch between the MFMA and the ALU kernels.
#include <hip/hip_runtime.h>

#include <cstdio>
#include <cstring>

#include <vector>

#include "kernels.h"

namespace hanayo {

namespace {

// gfx950 check, cached per device.
int check_device() {
  static thread_local int ok_device = -1;
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return set_error(HANAYO_EHIP, "hipGetDevice: %s", hipGetErrorString(e));
  if (dev == ok_device) return HANAYO_OK;
  hipDeviceProp_t prop;
  e = hipGetDeviceProperties(&prop, dev);
  if (e != hipSuccess) return set_error(HANAYO_EHIP, "hipGetDeviceProperties: %s", hipGetErrorString(e));
  if (std::strncmp(prop.gcnArchName, "gfx950", 6) != 0)
    return set_error(HANAYO_EUNSUPPORTED, "device %d is %s, this library is built for gfx950 only", dev, prop.gcnArchName);
  ok_device = dev;
  return HANAYO_OK;
}

bool misaligned(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 255u) != 0; }

struct BlockPtrs {
  const char* w[HANAYO_N_PARAMS];
  float* g[HANAYO_N_PARAMS];
};

BlockPtrs block_ptrs(const Shape& sh, const ParamOffsets& po, const void* weights, float* grads, int blk) {
  BlockPtrs bp;
  for (int i = 0; i < HANAYO_N_PARAMS; ++i) {
    const size_t e = (size_t)blk * po.block_elems + po.off[i];
    bp.w[i] = static_cast<const char*>(weights) + e * sh.esz;
    bp.g[i] = grads ? grads + e : nullptr;
  }
  return bp;
}

enum { P_LN1G, P_LN1B, P_WQKV, P_BQKV, P_WO, P_BO, P_LN2G, P_LN2B, P_W1, P_B1, P_W2, P_B2 };

#define TRY(expr)          \
  do {                     \
    const int rc_ = (expr); \
    if (rc_) return rc_;   \
  } while (0)

// y[T][N] = x[T][K] W[K][N] (+ epilogue)
int linear_fwd(const Shape& sh, const void* x, const void* W, const void* bias, void* y, int K, int N, k::Epilogue epi,
               const void* aux, void* aux_out, hipStream_t st) {
  k::GemmArgs g{};
  g.A = x; g.B = W; g.C = y; g.bias = bias; g.aux = aux; g.aux_out = aux_out;
  g.M = sh.T; g.N = N; g.K = K; g.lda = K; g.ldb = N; g.ldc = N;
  g.a_t = false; g.b_t = true; g.epi = epi;
  return k::gemm(sh.dtype, g, st);
}

// dx[T][K] = dy[T][N] W[K][N]^T (+ epilogue)
int linear_bwd_input(const Shape& sh, const void* dy, const void* W, void* dx, int K, int N, k::Epilogue epi,
                     const void* aux, hipStream_t st) {
  k::GemmArgs g{};
  g.A = dy; g.B = W; g.C = dx; g.aux = aux;
  g.M = sh.T; g.N = K; g.K = N; g.lda = N; g.ldb = N; g.ldc = K;
  g.a_t = false; g.b_t = false; g.epi = epi;
  return k::gemm(sh.dtype, g, st);
}

// dW[K][N] += x[T][K]^T dy[T][N];  db[N] += column sums of dy
k::GemmArgs bwd_params_gemm(const Shape& sh, const void* x, const void* dy, float* dW, float* db, int K, int N,
                            float* partial) {
  k::GemmArgs g{};
  g.A = x; g.B = dy; g.C = dW;
  g.M = K; g.N = N; g.K = sh.T; g.lda = K; g.ldb = N; g.ldc = N;
  g.a_t = true; g.b_t = true; g.epi = k::EPI_ACCUM_F32;
  g.colsum = db; g.colsum_scratch = partial;  // bias gradient rides along with the weight gradient
  return g;
}

}  // namespace

namespace k {

int raise_lds(const void* kernel, size_t lds, uint64_t& devices) {
  if (lds <= 64 * 1024) return HANAYO_OK;
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess) return set_error(HANAYO_EHIP, "hipGetDevice failed");
  const uint64_t bit = dev < 64 ? uint64_t(1) << dev : 0;
  if (devices & bit) return HANAYO_OK;
  const hipError_t e = hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
  if (e != hipSuccess) return set_error(HANAYO_EHIP, "cannot raise a kernel's LDS limit to %zu bytes: %s", lds, hipGetErrorString(e));
  devices |= bit;
  return HANAYO_OK;
}

namespace {
thread_local int g_gemm_config = -1;  // measurement knob: of the calling thread only
thread_local bool g_in_lanes = false;
thread_local double g_gemm_sharing = 0.0;
}
void set_gemm_config(int config) { g_gemm_config = config; }
bool in_lanes() { return g_in_lanes; }
double gemm_sharing() { return g_gemm_sharing; }
void set_lanes(bool executor, double busy) {
  // Measured: next to one other busy lane the shortest GEMM launch still wins, next to three the one with the least CU time.
  const double share = (busy - 2.0) * 0.5;
  g_in_lanes = executor;
  g_gemm_sharing = !executor || share < 0.0 ? 0.0 : (share > 1.0 ? 1.0 : share);
}

// Rounds of 256 CUs that a launch of `tiles` workgroups pays for: whole ones alone on the chip (share 0); next to kernels of
// other lanes the CUs that its last round leaves idle are not lost, so the count moves towards tiles / 256 (share 1).
double rounds_of(long tiles, double share) {
  return share * (double)tiles / 256.0 + (1.0 - share) * (double)((tiles + 255) / 256);
}

// Tile choice for the direct-to-LDS kernels by a cost model fitted to timings on MI355X: a launch
// runs ceil(tiles / 256 CUs) rounds; a round costs one K tile's time per 64 columns of K (1.60 us for
// 256 x 256, 0.90 us for 256 x 128, 0.54 us for 128 x 128 with two workgroups sharing a CU, measured on a chip in
// its sustained clock state with operands that do not stay in the Infinity Cache) plus an epilogue, and the launch a
// fixed start-up (pipeline fill grows with the tile).  Large tiles reuse operands better; small ones waste less of the last round, which matters
// less the more the chip is shared with other streams' kernels (`share`), and less of ragged edges.
// Returns -1 if no configuration takes every problem.  *cost_us is the time to expect of the chosen one, for the
// comparison with other kernels: the times above are those of a chip whose every CU multiplies and whose clock is down;
// a launch that leaves CUs idle runs at a higher clock (2048 x 2560 x 2560 in 160 tiles of 256 x 128: 0.75 us per K tile).
int choose_dma_config(const GemmArgs* gs, int count, double share, double* cost_us) {
  *cost_us = 0.0;
  if (gemm_dma_config_exists(g_gemm_config)) {
    for (int i = 0; i < count; ++i)
      if (!gemm_dma_supported(gs[i], g_gemm_config)) return -1;
    return g_gemm_config;
  }
  static const struct { int config; double per_ktile, per_ktile_idle, epilogue, start; } kTiles[] = {
      {7, 1.60, 1.04, 3.0, 7.0}, {10, 0.90, 0.63, 2.0, 4.5}, {9, 0.54, 0.38, 2.3, 3.3}};
  int best = -1;
  double best_cost = 0.0;
  long best_tiles = 0;
  for (const auto& t : kTiles) {
    int bm, bn;
    gemm_dma_tile(t.config, bm, bn);
    long tiles = 0;
    double ktiles = 0.0;  // summed over all tiles
    bool ok = true;
    for (int i = 0; i < count && ok; ++i) {
      ok = gemm_dma_supported(gs[i], t.config);
      const long ti = (long)((gs[i].M + bm - 1) / bm) * ((gs[i].N + bn - 1) / bn);
      tiles += ti;
      ktiles += (double)ti * ((gs[i].K + 63) / 64);
    }
    if (!ok || tiles == 0) continue;
    const double cost = t.start + rounds_of(tiles, share) * ((ktiles / tiles) * t.per_ktile + t.epilogue);
    if (best >= 0 && cost >= best_cost) continue;
    best = t.config, best_cost = cost, best_tiles = tiles;
    const double used = tiles / (256.0 * (double)((tiles + 255) / 256));  // share of the CUs over the launch's rounds
    double per_ktile = t.per_ktile_idle + (t.per_ktile - t.per_ktile_idle) * used * used;
    if (t.config == 9 && tiles > 256) per_ktile *= 0.75;  // two tiles in one CU overlap (1536 x 3072 x 768: 14.8 us)
    if (share > 0.0) per_ktile = t.per_ktile;
    *cost_us = t.start + rounds_of(tiles, share) * ((ktiles / tiles) * per_ktile + t.epilogue);
  }
  // For a launch of at most one tile per CU alone on the chip the 128 x 128 tile takes a ring of three stages: with one
  // wavefront per SIMD nothing else covers a load that is late (4096 x 1024 x 4096: 37.0 us, 45.4 with two stages).  Two
  // stages only where a CU holds two workgroups at a time (more than 256 tiles, or a chip shared with other lanes):
  // 2048 x 2560 x 2560 in 320 tiles takes 37.9 us instead of 43.2.
  if (best == 9 && best_tiles <= 256 && share <= 0.0) best = 11;
  return best;
}

// The same cost model for the wavefront-split kernel: the better tile of the first `kinds` and, in us, what it costs.  A round
// costs the K tiles of its tiles plus an epilogue.  bf16: 0.178 us per 64 of K for 64 x 64 (four rounds of 4096 x 1024: 19 us
// at K = 1024, 54 at 4096), 0.075 for 32 x 32.  fp32 is bound by its matrix instructions (256 flop per clock and CU): a 32 x 32
// tile costs a quarter of a 64 x 64 one and 15 % (more loads per flop).
//
// In bf16 what a workgroup loads sets its pace, 44 bytes per clock and CU (16 KiB per 64 of K in 0.178 us): 96 x 64 tiles cost
// 20 KiB, 32 x 64 tiles 12.  They fill the gaps where the square tiles need one round more.  us by the square tiles
// and with all four, 1527 x 768 x 3072 19.3 and 15.3 (288 tiles of 64 x 64, 192 of 96 x 64), 700 x 1536 x 6144 35.3 and 25.1 (264 and
// 192), 777 x 640 x 2560 11.4 and 7.8 (500 of 32 x 32, 250 of 32 x 64), 400 x 1024 x 4096 15.6 and 11.2, 1024 x 512 x 512 3.85 and
// 3.64; at K = 256 two rounds of 32 x 32 are as fast (512 x 1024: 3.3 and 3.5 us).  A 96 x 64 workgroup parks 104 KiB of partial
// tiles and so has a CU to itself: more than 256 of them, with nothing to cover a tile's start and end, are slower than the
// square ones (1025 x 3632 x 1360, 627 tiles: 31.4 against 27.0).  Of 32 x 64 a CU holds three (32 x 30592 x 512, 478 tiles: 6.98
// against 7.36).
WaveTile wave_choice(int dtype, const GemmArgs* gs, int count, double share, int kinds, double* cost_us) {
  struct Kind { WaveTile tile; double per_k, epilogue, start; };
  static const Kind kBf16[] = {{WAVE_64x64, 0.178 / 64, 1.0, 3.0}, {WAVE_32x32, 0.075 / 64, 0.6, 2.5}, {WAVE_96x64, 0.2225 / 64, 1.3, 3.0},
                               {WAVE_32x64, 0.13 / 64, 1.1, 2.7}};
  static const Kind kFp32[] = {{WAVE_64x64, 0.0154, 1.0, 3.0}, {WAVE_32x32, 0.0044, 0.6, 2.5}};
  const Kind* all = dtype == HANAYO_BF16 ? kBf16 : kFp32;
  if (dtype != HANAYO_BF16 || gs[0].epi == EPI_ACCUM_F32 || count > 1) kinds = 2;  // groups and weight gradients: square tiles
  WaveTile best = WAVE_NONE;
  for (int n = 0; n < kinds; ++n) {
    const Kind& t = all[n];
    int bm, bn;
    wave_tile(t.tile, bm, bn);
    long tiles = 0;
    double k = 0.0;
    bool ok = true;
    for (int i = 0; i < count; ++i) {
      ok = ok && gemm_wave_tile_fits(t.tile, dtype, gs[i]);
      const long ti = (long)((gs[i].M + bm - 1) / bm) * ((gs[i].N + bn - 1) / bn);
      tiles += ti;
      k += (double)ti * gs[i].K;
    }
    if (!ok || (t.tile == WAVE_96x64 && tiles > 256)) continue;
    const double cost = t.start + rounds_of(tiles, share) * (k / tiles * t.per_k + t.epilogue);
    if (best == WAVE_NONE || cost < *cost_us) best = t.tile, *cost_us = cost;
  }
  return best;
}

// Tile of the wavefront-split kernel for these problems, WAVE_NONE if it does not take them or a direct-to-LDS kernel is better.
// That kernel adds a contraction in another order than the direct-to-LDS ones, which among themselves (and its tiles
// among themselves) give the same bits.  An executor's results do not depend on its lanes, nor on what its plan
// expects of the other lanes, so between the two kinds the choice is made at one share for all of them.  Alone the split
// kernel's many small tiles win up to K in the thousands; next to other lanes large tiles use the chip better.  us per
// 16 x (forward, backward) of a block, share 0 / share 0.7, with 1 and 2 lanes: H = 2048, T = 1024 8460 / 9248, 7996 / 7507;
// H = 1280, T = 1527 6445 / 6713, 5722 / 5373; H = 512, T = 4096 4210 / 4202, 3274 / 3112.  Up to K = 1024 the time goes into start
// and epilogue, and nothing is won with lanes (H = 256, T = 2048: 1597 / 1685, 1189 / 1201).
WaveTile choose_wave(int dtype, const GemmArgs* gs, int count) {
  if (dtype == HANAYO_BF16 && gemm_dma_config_exists(g_gemm_config)) {
    bool forced = true;  // a kernel that does not take these problems (or fp32) forces nothing
    for (int i = 0; i < count; ++i) forced = forced && gemm_dma_supported(gs[i], g_gemm_config);
    if (forced) return WAVE_NONE;
  }
  for (int i = 0; i < count; ++i)
    if (!gemm_wave_supported(dtype, gs[i])) return WAVE_NONE;
  if (g_gemm_config == 0 || g_gemm_config == 1) return g_gemm_config == 0 ? WAVE_64x64 : WAVE_32x32;
  double wave_cost, dma_cost;
  if (dtype == HANAYO_BF16) {
    double k = 0.0, outputs = 0.0;
    for (int i = 0; i < count; ++i) {
      const double n = (double)gs[i].M * gs[i].N;
      outputs += n;
      k += n * gs[i].K;
    }
    const double share = g_in_lanes && k > 1024.0 * outputs ? 0.7 : 0.0;
    wave_choice(dtype, gs, count, share, 2, &wave_cost);  // by the square tiles, so that the line stays where it was
    if (choose_dma_config(gs, count, share, &dma_cost) >= 0 && dma_cost <= wave_cost) return WAVE_NONE;
  }
  return wave_choice(dtype, gs, count, g_gemm_sharing, 4, &wave_cost);
}

int gemm_kernel(int dtype, const GemmArgs& g) {
  switch (choose_wave(dtype, &g, 1)) {
    case WAVE_64x64: return 0;
    case WAVE_32x32: return 1;
    case WAVE_96x64: return 12;
    case WAVE_32x64: return 13;
    case WAVE_NONE: break;
  }
  double cost;
  const int config = dtype == HANAYO_BF16 ? choose_dma_config(&g, 1, g_gemm_sharing, &cost) : -1;
  return config >= 0 ? config : 14;
}

int gemm(int dtype, const GemmArgs& g, hipStream_t stream) {
  if (g.M < 1 || g.N < 1 || g.K < 1) return set_error(HANAYO_EINVAL, "gemm: empty problem");
  if (g.colsum && (!g.b_t || !g.colsum_scratch)) return set_error(HANAYO_EINVAL, "gemm: colsum needs b_t and scratch");
  if (g.colsum && g.epi != EPI_ACCUM_F32) {  // only the weight-gradient kernels fold column sums in
    GemmArgs plain = g;
    plain.colsum = nullptr;
    const int rc = gemm(dtype, plain, stream);
    return rc ? rc : colsum_add(dtype, g.B, g.K, g.N, g.colsum, g.colsum_scratch, stream);
  }
  if (const WaveTile tile = choose_wave(dtype, &g, 1)) return gemm_wave_group(dtype, &g, 1, tile, stream);
  if (dtype == HANAYO_BF16) {
    // the direct-to-LDS kernels fold the column sums into the GEMM
    double cost;
    const int config = choose_dma_config(&g, 1, g_gemm_sharing, &cost);
    if (config >= 0) return gemm_dma(g, config, stream);
  }
  const int rc = gemm_alu(dtype, g, stream);
  if (rc || !g.colsum) return rc;
  return colsum_add(dtype, g.B, g.K, g.N, g.colsum, g.colsum_scratch, stream);  // B is stored [K][ldb = N]
}

// A launch of few or small tiles takes jobs along: it leaves CUs idle, and one launch less is 2 to 3 us (a backward pass of one
// block, T = 512, H = 256: 36.8 -> 34.6 us, two blocks, T = 777, H = 640: 183.9 -> 180.6).  Beside 256 x 256 tiles the jobs'
// workgroups, which ask for the tiles' 128 KiB of LDS, hold up other lanes' kernels (four lanes, H = 4096: 0.6 % of a step).
int gemm_group(int dtype, const GemmArgs* gs, int count, hipStream_t stream, const FinalizeJob* jobs, int n_jobs, bool* taken) {
  if (taken) *taken = false;
  if (count < 1 || count > 4) return set_error(HANAYO_EINVAL, "gemm_group: %d problems", count);
  bool alike = true;
  for (int i = 0; i < count; ++i) {
    const GemmArgs& g = gs[i];
    if (g.M < 1 || g.N < 1 || g.K < 1) return set_error(HANAYO_EINVAL, "gemm: empty problem");
    if (g.colsum && (!g.b_t || !g.colsum_scratch)) return set_error(HANAYO_EINVAL, "gemm: colsum needs b_t and scratch");
    alike = alike && g.a_t == gs[0].a_t && g.b_t == gs[0].b_t && g.epi == gs[0].epi;
  }
  if (alike) {
    if (const WaveTile tile = choose_wave(dtype, gs, count)) {
      if (taken) *taken = true;
      return gemm_wave_group(dtype, gs, count, tile, stream, jobs, taken ? n_jobs : 0);
    }
  }
  if (alike && dtype == HANAYO_BF16) {
    double cost;
    const int config = choose_dma_config(gs, count, g_gemm_sharing, &cost);
    if (config >= 0) {
      if (taken) *taken = config != 7;
      return gemm_dma_group(gs, count, config, stream, jobs, taken && *taken ? n_jobs : 0);
    }
  }
  for (int i = 0; i < count; ++i) {
    const int rc = gemm(dtype, gs[i], stream);
    if (rc) return rc;
  }
  return HANAYO_OK;
}

int attn_forward(int dtype, const AttnArgs& a, hipStream_t stream) {
  return dtype == HANAYO_BF16 ? attn_forward_mfma(a, stream) : attn_forward_f32(a, stream);
}

int attn_backward(int dtype, const AttnArgs& a, hipStream_t stream) {
  return dtype == HANAYO_BF16 ? attn_backward_mfma(a, stream) : attn_backward_f32(a, stream);
}

}  // namespace k

int chunk_forward(const Shape& sh, const void* weights, const void* x, const int32_t* valid_len, void* y, void* stash,
                  hipStream_t st) {
  const ParamOffsets po = param_offsets(sh);
  const StashLayout L = stash_layout(sh);
  const int T = sh.T, H = sh.H, F = sh.F;
  const size_t act_bytes = (size_t)T * H * sh.esz;
  for (int blk = 0; blk < sh.nb; ++blk) {
    char* sb = static_cast<char*>(stash) + (size_t)blk * L.block_bytes;
    const BlockPtrs p = block_ptrs(sh, po, weights, nullptr, blk);
    // block input: the caller's x for the first block (copied into the stash), else what the block before wrote
    const void* xin = blk == 0 ? x : sb + L.x;
    void* yout = blk == sh.nb - 1 ? y : sb + L.block_bytes + L.x;
    k::AttnArgs at{};
    at.qkv = sb + L.qkv; at.valid_len = valid_len; at.ctx = sb + L.ctx; at.lse = reinterpret_cast<float*>(sb + L.lse);
    at.b = sh.b; at.s = sh.s; at.heads = sh.heads; at.d = sh.d; at.causal = sh.mask == HANAYO_MASK_CAUSAL;
    if (sh.norm == HANAYO_PRE_LN) {
      TRY(k::ln_forward(sh.dtype, xin, p.w[P_LN1G], p.w[P_LN1B], sb + L.ln_a, reinterpret_cast<float2*>(sb + L.stats1),
                        blk == 0 ? sb + L.x : nullptr, T, H, sh.eps, st));
      TRY(linear_fwd(sh, sb + L.ln_a, p.w[P_WQKV], p.w[P_BQKV], sb + L.qkv, H, 3 * H, k::EPI_BIAS, nullptr, nullptr, st));
      TRY(k::attn_forward(sh.dtype, at, st));
      TRY(linear_fwd(sh, sb + L.ctx, p.w[P_WO], p.w[P_BO], sb + L.x1, H, H, k::EPI_BIAS_RES, xin, nullptr, st));
      TRY(k::ln_forward(sh.dtype, sb + L.x1, p.w[P_LN2G], p.w[P_LN2B], sb + L.ln_b, reinterpret_cast<float2*>(sb + L.stats2),
                        nullptr, T, H, sh.eps, st));
      TRY(linear_fwd(sh, sb + L.ln_b, p.w[P_W1], p.w[P_B1], sb + L.act, H, F, k::EPI_BIAS_GELU, nullptr, sb + L.hpre, st));
      TRY(linear_fwd(sh, sb + L.act, p.w[P_W2], p.w[P_B2], yout, F, H, k::EPI_BIAS_RES, sb + L.x1, nullptr, st));
    } else {
      if (blk == 0) TRY(k::copy_bytes(sb + L.x, x, act_bytes, st));
      TRY(linear_fwd(sh, xin, p.w[P_WQKV], p.w[P_BQKV], sb + L.qkv, H, 3 * H, k::EPI_BIAS, nullptr, nullptr, st));
      TRY(k::attn_forward(sh.dtype, at, st));
      TRY(linear_fwd(sh, sb + L.ctx, p.w[P_WO], p.w[P_BO], sb + L.ln_a, H, H, k::EPI_BIAS_RES, xin, nullptr, st));
      TRY(k::ln_forward(sh.dtype, sb + L.ln_a, p.w[P_LN1G], p.w[P_LN1B], sb + L.x1, reinterpret_cast<float2*>(sb + L.stats1),
                        nullptr, T, H, sh.eps, st));
      TRY(linear_fwd(sh, sb + L.x1, p.w[P_W1], p.w[P_B1], sb + L.act, H, F, k::EPI_BIAS_GELU, nullptr, sb + L.hpre, st));
      TRY(linear_fwd(sh, sb + L.act, p.w[P_W2], p.w[P_B2], sb + L.ln_b, F, H, k::EPI_BIAS_RES, sb + L.x1, nullptr, st));
      TRY(k::ln_forward(sh.dtype, sb + L.ln_b, p.w[P_LN2G], p.w[P_LN2B], yout, reinterpret_cast<float2*>(sb + L.stats2),
                        nullptr, T, H, sh.eps, st));
    }
  }
  return HANAYO_OK;
}

int chunk_backward(const Shape& sh, const void* weights, float* grads, const void* dy, const int32_t* valid_len,
                   const void* stash, void* dx, void* workspace, hipStream_t st) {
  const ParamOffsets po = param_offsets(sh);
  const StashLayout L = stash_layout(sh);
  const WorkLayout WL = work_layout(sh);
  char* ws = static_cast<char*>(workspace);
  const int T = sh.T, H = sh.H, F = sh.F;
  float* partial = reinterpret_cast<float*>(ws + WL.partial);
  // Every LayerNorm backward leaves its partial gamma/beta sums in a slot of its own; a block's weight-gradient launch
  // adds its two LayerNorms' to the gradients, or one launch after the last block does it for all of them.
  std::vector<k::FinalizeJob> ln_jobs;
  ln_jobs.reserve(2 * (size_t)sh.nb);
  size_t slot = 0;
  auto ln_slot = [&]() { return reinterpret_cast<float*>(ws + WL.ln_partial + slot * WL.ln_slot_bytes); };
  auto ln_bwd = [&](const void* dout, const void* x, const void* gamma, const void* stats, const void* addend, void* dz,
                    float* dgamma, float* dbeta) {
    k::FinalizeJob job;
    const int rc = k::ln_backward_deferred(sh.dtype, dout, x, gamma, reinterpret_cast<const float2*>(stats), addend, dz,
                                           dgamma, dbeta, ln_slot(), T, H, st, &job);
    if (rc == HANAYO_OK) ln_jobs.push_back(job), ++slot;
    return rc;
  };
  const void* dy_blk = dy;
  for (int blk = sh.nb - 1; blk >= 0; --blk) {
    // The four weight-gradient GEMMs of a block wait until its end and go out as one group: every
    // activation and gradient they read stays untouched until then.
    k::GemmArgs dw[4];
    const char* sb = static_cast<const char*>(stash) + (size_t)blk * L.block_bytes;
    const BlockPtrs p = block_ptrs(sh, po, weights, grads, blk);
    // gradient w.r.t. this block's input: the caller's dx for block 0, else a ping-pong buffer
    void* dx_blk = blk == 0 ? dx : ws + ((blk & 1) ? WL.d_ping : WL.d_pong);
    k::AttnArgs at{};
    at.qkv = sb + L.qkv; at.valid_len = valid_len; at.ctx = const_cast<char*>(sb + L.ctx);
    at.lse = reinterpret_cast<float*>(const_cast<char*>(sb + L.lse));
    at.dqkv = ws + WL.d_qkv; at.delta = reinterpret_cast<float*>(ws + WL.delta);
    at.b = sh.b; at.s = sh.s; at.heads = sh.heads; at.d = sh.d; at.causal = sh.mask == HANAYO_MASK_CAUSAL;
    if (sh.norm == HANAYO_PRE_LN) {
      // y = x1 + W2 GELU(W1 LN2(x1))
      dw[0] = bwd_params_gemm(sh, sb + L.act, dy_blk, p.g[P_W2], p.g[P_B2], F, H, partial);
      TRY(linear_bwd_input(sh, dy_blk, p.w[P_W2], ws + WL.d_act, F, H, k::EPI_MUL_DGELU, sb + L.hpre, st));
      dw[1] = bwd_params_gemm(sh, sb + L.ln_b, ws + WL.d_act, p.g[P_W1], p.g[P_B1], H, F, partial);
      TRY(linear_bwd_input(sh, ws + WL.d_act, p.w[P_W1], ws + WL.d_h0, H, F, k::EPI_NONE, nullptr, st));
      // dx1 = dy + LN2'(d_h0)
      TRY(ln_bwd(ws + WL.d_h0, sb + L.x1, p.w[P_LN2G], sb + L.stats2,
                 dy_blk, ws + WL.d_h1, p.g[P_LN2G], p.g[P_LN2B]));
      // x1 = x + Wo ctx
      dw[2] = bwd_params_gemm(sh, sb + L.ctx, ws + WL.d_h1, p.g[P_WO], p.g[P_BO], H, H, partial);
      TRY(linear_bwd_input(sh, ws + WL.d_h1, p.w[P_WO], ws + WL.d_h0, H, H, k::EPI_NONE, nullptr, st));
      at.dctx = ws + WL.d_h0;
      TRY(k::attn_backward(sh.dtype, at, st));
      dw[3] = bwd_params_gemm(sh, sb + L.ln_a, ws + WL.d_qkv, p.g[P_WQKV], p.g[P_BQKV], H, 3 * H, partial);
      TRY(linear_bwd_input(sh, ws + WL.d_qkv, p.w[P_WQKV], ws + WL.d_h2, H, 3 * H, k::EPI_NONE, nullptr, st));
      // dx = dx1 + LN1'(d_h2)
      TRY(ln_bwd(ws + WL.d_h2, sb + L.x, p.w[P_LN1G], sb + L.stats1,
                 ws + WL.d_h1, dx_blk, p.g[P_LN1G], p.g[P_LN1B]));
    } else {
      // y = LN2(f), f = x1 + W2 GELU(W1 x1)
      TRY(ln_bwd(dy_blk, sb + L.ln_b, p.w[P_LN2G], sb + L.stats2,
                 nullptr, ws + WL.d_h0, p.g[P_LN2G], p.g[P_LN2B]));
      dw[0] = bwd_params_gemm(sh, sb + L.act, ws + WL.d_h0, p.g[P_W2], p.g[P_B2], F, H, partial);
      TRY(linear_bwd_input(sh, ws + WL.d_h0, p.w[P_W2], ws + WL.d_act, F, H, k::EPI_MUL_DGELU, sb + L.hpre, st));
      dw[1] = bwd_params_gemm(sh, sb + L.x1, ws + WL.d_act, p.g[P_W1], p.g[P_B1], H, F, partial);
      // dx1 = df + d_act W1^T
      TRY(linear_bwd_input(sh, ws + WL.d_act, p.w[P_W1], ws + WL.d_h1, H, F, k::EPI_ADD, ws + WL.d_h0, st));
      // x1 = LN1(a), a = x + Wo ctx
      TRY(ln_bwd(ws + WL.d_h1, sb + L.ln_a, p.w[P_LN1G], sb + L.stats1,
                 nullptr, ws + WL.d_h2, p.g[P_LN1G], p.g[P_LN1B]));
      dw[2] = bwd_params_gemm(sh, sb + L.ctx, ws + WL.d_h2, p.g[P_WO], p.g[P_BO], H, H, partial);
      TRY(linear_bwd_input(sh, ws + WL.d_h2, p.w[P_WO], ws + WL.d_h3, H, H, k::EPI_NONE, nullptr, st));
      at.dctx = ws + WL.d_h3;  // d_h0 still feeds the W2 gradient
      TRY(k::attn_backward(sh.dtype, at, st));
      dw[3] = bwd_params_gemm(sh, sb + L.x, ws + WL.d_qkv, p.g[P_WQKV], p.g[P_BQKV], H, 3 * H, partial);
      // dx = da + dqkv Wqkv^T
      TRY(linear_bwd_input(sh, ws + WL.d_qkv, p.w[P_WQKV], dx_blk, H, 3 * H, k::EPI_ADD, ws + WL.d_h2, st));
    }
    bool taken;
    TRY(k::gemm_group(sh.dtype, dw, 4, st, ln_jobs.data() + ln_jobs.size() - 2, 2, &taken));
    if (taken) ln_jobs.resize(ln_jobs.size() - 2);
    dy_blk = dx_blk;
  }
  return k::finalize_group(ln_jobs.data(), (int)ln_jobs.size(), st);
}

int device_ok() { return check_device(); }

int prepare_call(const hanayo_chunk_desc* d, Shape& sh) {
  TRY(make_shape(d, sh));
  return check_device();
}

}  // namespace hanayo

using namespace hanayo;

extern "C" {

int hanayo_chunk_forward(const hanayo_chunk_desc* d, const void* weights, const void* x, const int32_t* valid_len,
                         void* y, void* stash_entry, void* workspace, void* hip_stream) {
  Shape sh;
  TRY(prepare_call(d, sh));
  (void)workspace;
  if (!weights || !x || !y || !stash_entry) return set_error(HANAYO_EINVAL, "chunk_forward: NULL pointer");
  if (misaligned(weights) || misaligned(x) || misaligned(y) || misaligned(stash_entry))
    return set_error(HANAYO_EINVAL, "chunk_forward: device pointers must be 256-byte aligned");
  if (x == y) return set_error(HANAYO_EINVAL, "chunk_forward: y aliases x");
  return chunk_forward(sh, weights, x, valid_len, y, stash_entry, static_cast<hipStream_t>(hip_stream));
}

int hanayo_chunk_backward(const hanayo_chunk_desc* d, const void* weights, float* grads, const void* dy,
                          const int32_t* valid_len, const void* stash_entry, void* dx, void* workspace,
                          void* hip_stream) {
  Shape sh;
  TRY(prepare_call(d, sh));
  if (!weights || !grads || !dy || !dx || !stash_entry || !workspace)
    return set_error(HANAYO_EINVAL, "chunk_backward: NULL pointer");
  if (misaligned(weights) || misaligned(grads) || misaligned(dy) || misaligned(dx) || misaligned(stash_entry) ||
      misaligned(workspace))
    return set_error(HANAYO_EINVAL, "chunk_backward: device pointers must be 256-byte aligned");
  if (dx == dy) return set_error(HANAYO_EINVAL, "chunk_backward: dx aliases dy");
  return chunk_backward(sh, weights, grads, dy, valid_len, stash_entry, dx, workspace,
                        static_cast<hipStream_t>(hip_stream));
}

int hanayo_device_info(char* buf, size_t cap) {
  if (!buf || !cap) return set_error(HANAYO_EINVAL, "device_info: no buffer");
  int dev = 0;
  hipDeviceProp_t prop;
  if (hipGetDevice(&dev) != hipSuccess || hipGetDeviceProperties(&prop, dev) != hipSuccess) {
    (void)hipGetLastError();
    return set_error(HANAYO_EHIP, "device_info: no HIP device");
  }
  std::snprintf(buf, cap, "%s %s CUs=%d clock_khz=%d", prop.name, prop.gcnArchName, prop.multiProcessorCount,
                prop.clockRate);
  return HANAYO_OK;
}

}  // extern "C"
