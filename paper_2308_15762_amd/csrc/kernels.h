// Host-side launchers of the HIP kernels.  Every launcher validates what the
// kernel and its grid assume, enqueues on `stream`, and returns HANAYO_OK or an
// error code (nothing is enqueued on error).
#pragma once

#include <hip/hip_runtime.h>

#include <tuple>

#include "internal.h"

namespace hanayo {
namespace k {

// Raises a kernel's limit of dynamic LDS for a launch of `lds` bytes.  The limit belongs to the device: `devices` (a
// thread_local of the launcher, one bit per device) says where the calling thread has raised it already.
int raise_lds(const void* kernel, size_t lds, uint64_t& devices);

// Enqueues a kernel.  Straight to hipLaunchKernel: the <<<>>> form first pushes the launch configuration onto a stack of the
// runtime's and takes it off again (2.6 -> 2.45 us of host time for 13 arguments).  Errors stay with the runtime until
// check_launch.
template <typename... P, typename... A>
inline void launch_kernel(void (*kernel)(P...), dim3 grid, dim3 block, size_t lds, hipStream_t stream, A... args) {
  static_assert(sizeof...(P) == sizeof...(A), "one argument per parameter");
  std::tuple<P...> values(static_cast<P>(args)...);
  std::apply(
      [&](P&... v) {
        void* at[] = {const_cast<void*>(static_cast<const void*>(&v))...};
        (void)hipLaunchKernel(reinterpret_cast<const void*>(kernel), grid, block, at, lds, stream);
      },
      values);
}

// ---- LayerNorm (row-wise over H; wavefront reductions) ----------------------
// out = LN(x) * gamma + beta; stats[t] = (mean, rstd); copy_out (optional) = x.
int ln_forward(int dtype, const void* x, const void* gamma, const void* beta, void* out, float2* stats, void* copy_out,
               int T, int H, float eps, hipStream_t stream);
// dz = LN'(dout) (+ addend, optional); dgamma += sum_t dout*xhat; dbeta += sum_t dout.
// `partial` is scratch of at least kMaxPartialRows * 2H floats.
int ln_backward(int dtype, const void* dout, const void* x, const void* gamma, const float2* stats, const void* addend,
                void* dz, float* dgamma, float* dbeta, float* partial, int T, int H, hipStream_t stream);
// The same with the last step left to the caller: dz is written, the gamma/beta sums stay as partial rows in
// `partial` (kLnPartialRows * 2H floats, untouched until the job has run) and *job says how to add them up.
// gemm_group takes such jobs along in a launch of weight gradients; finalize_group runs any number of them, eight to a
// launch.
constexpr int kMaxFinalizeJobs = 8;
struct FinalizeJob {
  const float* partial;  // [rows][ld]
  int rows, ld, n;       // columns c < n: (c < split ? out0[c] : out1[c - split]) += sum over rows of partial[r][c]
  float* out0;
  float* out1;
  int split;
};
int ln_backward_deferred(int dtype, const void* dout, const void* x, const void* gamma, const float2* stats,
                         const void* addend, void* dz, float* dgamma, float* dbeta, float* partial, int T, int H,
                         hipStream_t stream, FinalizeJob* job);
int finalize_group(const FinalizeJob* jobs, int count, hipStream_t stream);
// out[n] += sum_t in[t][n]
int colsum_add(int dtype, const void* in, int T, int N, float* out, float* partial, hipStream_t stream);

// ---- GEMM ---------------------------------------------------------------------
enum Epilogue {
  EPI_NONE = 0,       // C = acc
  EPI_BIAS,           // C = acc + bias[n]
  EPI_BIAS_GELU,      // aux_out = acc + bias[n];  C = GELU(aux_out)
  EPI_BIAS_RES,       // C = acc + bias[n] + aux[m][n]
  EPI_MUL_DGELU,      // C = acc * GELU'(aux[m][n])
  EPI_ADD,            // C = acc + aux[m][n]
  EPI_ACCUM_F32,      // C (fp32) += acc
  EPI_STORE_F32       // C (fp32) = acc   (partial products of a K split; !a_t && b_t only)
};

// C[M][N] = A[M][K] * B[K][N] with fp32 accumulation.
//   a_t = false: A stored [M][lda] (K contiguous);  true: stored [K][lda] (M contiguous)
//   b_t = false: B stored [N][ldb] (K contiguous);  true: stored [K][ldb] (N contiguous)
// C, aux, aux_out are row-major [M][ldc]; bias is the storage type, [N].
struct GemmArgs {
  const void* A;
  const void* B;
  void* C;
  const void* bias;
  const void* aux;
  void* aux_out;
  int M, N, K;
  int lda, ldb, ldc;
  bool a_t, b_t;
  Epilogue epi;
  // Optional, only with b_t: colsum[n] (fp32) += sum over k of B[k][n] (the bias gradient that
  // goes with a weight-gradient GEMM).  colsum_scratch: at least 64 * N floats, used by the
  // kernels that cannot fold the sums into the GEMM itself.
  float* colsum;
  float* colsum_scratch;
  // Optional: *live (device) is the number of rows of C (LIVE_M) or of contraction elements (LIVE_K) that count, at most
  // M or K; workgroups past it leave at once.  LIVE_M_SPLIT (EPI_STORE_F32, gemm_dma_group only, one problem): as LIVE_M, with
  // the contraction cut into slices, one partial product each, by split_plan.
  const int* live;
  int live_dim;
};
enum { LIVE_NONE = 0, LIVE_M, LIVE_K, LIVE_M_SPLIT };
// How a grid of `grid` workgroups covers `live` rows x tiles_n 256-column tiles with K cut into slices of `per` elements
// (whole K tiles, at least 8 each): as many slices as the grid holds.  Evaluated on the device, by the GEMM and by the
// kernel that adds the slices.
constexpr int kMaxSlices = 16, kSplitGrid = 256;  // workgroups of a LIVE_M_SPLIT launch: this many, or one per 256 x 256 tile
__host__ __device__ inline int split_plan(int live, int tiles_n, int K, int grid, int& per) {
  const int tiles = (live + 255) / 256 * tiles_n, ktiles = (K + 63) / 64;
  int slices = tiles > 0 ? grid / tiles : 1;
  if (slices > kMaxSlices) slices = kMaxSlices;
  if (slices > ktiles / 8) slices = ktiles / 8;
  if (slices < 1) slices = 1;
  per = (ktiles + slices - 1) / slices * 64;
  return (K + per - 1) / per;
}
int gemm(int dtype, const GemmArgs& g, hipStream_t stream);
// The kernel that gemm would run this problem on, by the numbers of hanayo_op_gemm_kernel.
int gemm_kernel(int dtype, const GemmArgs& g);
// Up to 4 independent problems of one layout and epilogue; one launch where the tiled kernels allow
// it (small problems then fill the chip together), otherwise one after the other.
// `jobs` (at most kMaxJobs): partial rows that the launch may add up besides, in workgroups of their own; *taken says whether
// it has, else finalize_group is left to the caller.  The sums are the same bits either way.
constexpr int kMaxJobs = 2;
int gemm_group(int dtype, const GemmArgs* gs, int count, hipStream_t stream, const FinalizeJob* jobs = nullptr, int n_jobs = 0,
               bool* taken = nullptr);

// ---- attention ------------------------------------------------------------------
// qkv is [b*s][3H] (Q | K | V, head j in columns j*d..), ctx [b*s][H], lse [b][heads][s].
struct AttnArgs {
  const void* qkv;
  const int32_t* valid_len;  // device [b] or nullptr
  void* ctx;                 // forward: out; backward: in
  float* lse;                // forward: out; backward: in
  const void* dctx;          // backward in
  void* dqkv;                // backward out [b*s][3H]
  float* delta;              // backward scratch [b][heads][s]
  int b, s, heads, d;
  bool causal;
};
int attn_forward(int dtype, const AttnArgs& a, hipStream_t stream);
int attn_backward(int dtype, const AttnArgs& a, hipStream_t stream);

// Implementations behind the dispatchers above.
int gemm_alu(int dtype, const GemmArgs& g, hipStream_t stream);
int attn_forward_f32(const AttnArgs& a, hipStream_t stream);  // fp32 storage
int attn_backward_f32(const AttnArgs& a, hipStream_t stream);
int attn_delta(const AttnArgs& a, hipStream_t stream);  // bf16: delta = rowsum(dctx * ctx)
// Direct-to-LDS kernels in large tiles, bf16: config 7 = 256 x 256 (8 wavefronts), 9 / 11 = 128 x 128 with two / three
// stages, 10 = 256 x 128.  Any extents made of whole 16-byte vectors.
bool gemm_dma_config_exists(int config);
bool gemm_dma_supported(const GemmArgs& g, int config);
void gemm_dma_tile(int config, int& bm, int& bn);
int gemm_dma(const GemmArgs& g, int config, hipStream_t stream);
int gemm_dma_group(const GemmArgs* gs, int count, int config, hipStream_t stream, const FinalizeJob* jobs = nullptr,
                   int n_jobs = 0);
// Tiles whose contraction is split over the wavefronts of a workgroup: few tiles, ragged extents, fp32.  Up to 4 problems
// per launch; column sums are folded in.  The tiles among themselves give the same bits; WAVE_96x64 and WAVE_32x64
// exist in bf16, for single problems that are no weight gradients.
enum WaveTile { WAVE_NONE = 0, WAVE_64x64, WAVE_32x32, WAVE_96x64, WAVE_32x64 };
inline void wave_tile(WaveTile t, int& bm, int& bn) {
  bm = t == WAVE_64x64 ? 64 : t == WAVE_96x64 ? 96 : 32;
  bn = t == WAVE_32x32 ? 32 : 64;
}
bool gemm_wave_supported(int dtype, const GemmArgs& g);
bool gemm_wave_tile_fits(WaveTile t, int dtype, const GemmArgs& g);  // of a supported problem: lane offsets within 31 bits
int gemm_wave_group(int dtype, const GemmArgs* gs, int count, WaveTile tile, hipStream_t stream, const FinalizeJob* jobs = nullptr,
                    int n_jobs = 0);
// 7, 9, 10, 11 = force that direct-to-LDS configuration where it applies; 0 / 1 = the wavefront-split kernel with
// 64 x 64 / 32 x 32 tiles where it applies; anything else = automatic choice
void set_gemm_config(int config);
// Whose launches the calling thread enqueues.  executor: a task of the executor, next to which its plan expects `busy` lanes
// to run (itself among them); otherwise a caller's own, alone on the chip.  in_lanes() decides between kernels that add in
// different orders (one choice whatever the lanes do, so that results do not depend on them); gemm_sharing() between tiles
// that give the same bits: 0 = choose for the shortest launch, 1 = idle CUs are always taken by other work.
void set_lanes(bool executor, double busy);
bool in_lanes();
double gemm_sharing();
bool attn_mfma_supported(const AttnArgs& a);
int attn_forward_mfma(const AttnArgs& a, hipStream_t stream);
int attn_forward_split(const AttnArgs& a, hipStream_t stream);   // few rows; head dims 32, 64, 80, 96, 128 (called by attn_*_mfma)
int attn_backward_split(const AttnArgs& a, hipStream_t stream);
int attn_backward_mfma(const AttnArgs& a, hipStream_t stream);

// ---- the model's ends and the optimizer --------------------------------------------
// x[n][i][:] = wte[tokens[n][i]][:] + wpe[i][:]; tokens outside [0, vocab) contribute nothing.
int embed_forward(int dtype, const void* wte, const void* wpe, const int32_t* tokens, void* x, int b, int s, int H,
                  int vocab, hipStream_t stream);
// d_wte[tokens[n][i]][:] += dx[n][i][:] (fixed order, no atomics); d_wpe[i][:] += sum_n dx[n][i][:].
int embed_backward(int dtype, const int32_t* tokens, const void* dx, float* d_wte, float* d_wpe, int b, int s, int H,
                   int vocab, hipStream_t stream);
// The rows whose label lies inside [0, vocab), in order: live[0] = their number n, list[0..n) = the rows, slot[row] = the row's
// place in the list or -1; out[i][:] = in[list[i]][:].
int gather_labelled(int dtype, const int32_t* labels, const void* in, int rows, int vocab, int H, void* out, int* live, int32_t* list,
                    int32_t* slot, hipStream_t stream);
// In place on logits [live][V], whose row i belongs to label labels[list[i]]: the gradient of loss_scale * (mean of the
// rows' negative log-likelihoods); nll[i] = the row's negative log-likelihood.
int softmax_xent(int dtype, void* logits, const int32_t* labels, const int* live, const int32_t* list, float loss_scale,
                 float* nll, int rows, int V, hipStream_t stream);
struct AdamArgs {
  void* params;   // storage type, updated
  float* master;  // bf16 storage: fp32 copy of the parameters, updated; ignored for fp32 storage
  float* grads;
  float* m;
  float* v;
  size_t count;   // multiple of 4
  float lr, beta1, beta2, eps, weight_decay;
  int step;       // t >= 1
  int zero_grads;
  // weight decay applies everywhere (block_elems = 0) or only where (index mod block_elems) falls in one of
  // the four ranges [lo, hi)
  size_t block_elems;
  size_t lo[4], hi[4];
};
int adam(int dtype, const AdamArgs& a, hipStream_t stream);

// out[row][:] = row slot[row] of the [live][H] product (zeros where slot is -1).  grid > 0: the product is the sum of the
// fp32 slices of split_plan(live, tiles_n, K, grid), else it is stored whole in the storage type.
// Also loss[0] = sum(nll[0..live)) / live (0 if live is 0).
int scatter_rows(int dtype, const void* product, const int* live, const int32_t* slot, int grid, int K, void* out, int rows, int H,
                 const float* nll, float* loss, hipStream_t stream);

// ---- misc ------------------------------------------------------------------------
// max_workgroups > 0 caps the grid: a copy that uses only a few CUs and so runs at a chosen fraction of the
// memory bandwidth (the emulated link of the pipeline runs).
int copy_bytes(void* dst, const void* src, size_t bytes, hipStream_t stream, int max_workgroups = 0);

// Checks the last launch; returns HANAYO_EHIP with the HIP message on failure.
int check_launch(const char* what);

}  // namespace k
}  // namespace hanayo
