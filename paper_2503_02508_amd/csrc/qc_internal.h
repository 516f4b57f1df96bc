// Internal declarations shared by the host layer and the kernel launchers.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>
#include <stddef.h>
#include <atomic>
#include <vector>
#include "qc.h"

namespace qc {

// Activation quantiser parameters as the kernels use them: zero point already
// shifted to the signed code range (paper's z minus 128).
struct QParam {
  float s;
  int z;
};

// One quantised weight matrix in the arena.
struct LinearQ {
  void *q = nullptr;         // int8 [N, K] or packed nibbles [N, K/2]
  void *qt = nullptr;        // the same codes in MFMA fragment order for the large-M kernel, or null
  float *scale = nullptr;    // [N]
  int32_t *wsum = nullptr;   // [N]
  float *bias = nullptr;     // [N]
  int N = 0, K = 0;
};

void set_error(const char *fmt, ...);

// Lets a kernel use `bytes` of dynamic LDS on the current device (the attribute is a device's own).  done: one per kernel, a bit
// per device that was asked already.
inline hipError_t allow_lds(const void *kern, int bytes, std::atomic<unsigned long long> &done) {
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  const unsigned long long bit = dev < 64 ? 1ull << dev : 0ull;
  if (done.load(std::memory_order_acquire) & bit) return hipSuccess;
  e = hipFuncSetAttribute(kern, hipFuncAttributeMaxDynamicSharedMemorySize, bytes);
  if (e == hipSuccess) done.fetch_or(bit, std::memory_order_release);
  return e;
}

// ---- epilogues of the int8 GEMM
enum Epi { EPI_F32 = 0, EPI_GELU_Q = 1, EPI_RESID = 2, EPI_QKV = 3 };

struct GemmArgs {
  const int8_t *A;           // [M, lda] signed codes
  const void *W;             // [N, K] int8 or [N, K/2] packed
  const void *Wt;            // the same codes in MFMA fragment order (launch_tile_weight), or null
  const float *w_scale;
  const int32_t *wsum;
  const float *bias;         // may be null
  int M, N, K, lda;
  int w4;                    // weights are packed nibbles
  // activation parameters of the input: either by value or from device memory
  float a_scale;
  int a_zp;                  // signed
  const QParam *a_qp;        // if non-null overrides a_scale / a_zp
  // batching over blockIdx.z (element strides; 0 = shared)
  long long zs_A, zs_W, zs_vecN, zs_out;   // zs_W in bytes, the others in elements
  int zs_qp;
  // subset of output rows: when sel_D > 0 the launch covers 2*sel_D outputs,
  // logical column j maps to j + 2*sel_D for j < sel_D and j + 4*sel_D otherwise
  // (the two gate chunks of an adaLN projection).
  int sel_D;
  int xcd_m;                 // XCD grid rows (set by the launcher)
  int group_m;               // large-M kernel: tile rows per group of its tile order (set by the launcher)
  int beside;                // launches of this kind that run at the same time, this one included (0: this one)
  int stream_out;            // large-M kernel: streaming stores for float32 rows (set by the launcher)
  // EPI_F32
  float *y;
  int ldy;
  int32_t *acc_out;          // optional raw accumulators [M, N]
  // EPI_GELU_Q
  int8_t *q_out;
  int ldq;
  const QParam *o_qp;        // output quantiser
  // EPI_RESID
  void *cache_out;           // [M, N] fp32, or bfloat16 when cache_bf16 is set
  int cache_bf16;
  void *x;                   // [M, N] residual stream (fp32, or bfloat16 when x_bf16 is set), updated in place
  int x_bf16;
  const float *gate;         // [B, ld_gate]
  int ld_gate;
  int rows_per_batch;        // T
  // EPI_QKV: the float32 Q | K | V columns go out in the attention kernel's head-major layouts: Q and K
  // [B, H, T, hd]; V transposed and key-permuted [B, H, DP, Tp] (DP = hd rounded up to 16, Tp = T rounded up to 64);
  // y, when set, also receives them row-major
  float *q32, *k32, *vt32;
  int heads, hd, DP, Tp;
};

// position of key t inside V^T rows: within each group of 32 keys the units of 4 keys are interleaved so that
// the 8 keys a lane of the P^T operand owns (4g..4g+3 and 16+4g..16+4g+3) are contiguous
__host__ __device__ inline int vt_pos(int t) {
  const int u = (t >> 2) & 7;
  return (t & ~31) | ((((u & 3) << 1) | (u >> 2)) << 2) | (t & 3);
}

// ---- storage formats.  The cached tensors and, in the reduced-precision variant, the residual stream are stored as
// fp32 or as bfloat16 (round to nearest even of the fp32 value); element i of a tensor sits at index i of either format.
__host__ __device__ inline unsigned short bf16_bits(float v) {
  unsigned u = __builtin_bit_cast(unsigned, v);
  u += 0x7FFFu + ((u >> 16) & 1u);
  return (unsigned short)(u >> 16);
}
__host__ __device__ inline float bf16_value(unsigned short h) { return __builtin_bit_cast(float, (unsigned)h << 16); }
// element / four elements of the residual stream (bf != 0: bfloat16); i4 counts groups of four elements
__device__ __forceinline__ float stream_load(const void *x, size_t i, int bf) {
  return bf ? bf16_value(((const unsigned short *)x)[i]) : ((const float *)x)[i];
}
__device__ __forceinline__ void stream_store(void *x, size_t i, float v, int bf) {
  if (bf) ((unsigned short *)x)[i] = bf16_bits(v);
  else ((float *)x)[i] = v;
}
__device__ __forceinline__ float4 stream_load4(const void *x, size_t i4, int bf) {
  if (bf) {
    const uint2 r = ((const uint2 *)x)[i4];
    return make_float4(__builtin_bit_cast(float, r.x << 16), __builtin_bit_cast(float, r.x & 0xFFFF0000u),
                       __builtin_bit_cast(float, r.y << 16), __builtin_bit_cast(float, r.y & 0xFFFF0000u));
  }
  return ((const float4 *)x)[i4];
}
__device__ __forceinline__ void stream_store4(void *x, size_t i4, float4 v, int bf) {
  if (bf) {
    uint2 r;
    r.x = (unsigned)bf16_bits(v.x) | ((unsigned)bf16_bits(v.y) << 16);
    r.y = (unsigned)bf16_bits(v.z) | ((unsigned)bf16_bits(v.w) << 16);
    ((uint2 *)x)[i4] = r;
  } else {
    ((float4 *)x)[i4] = v;
  }
}

// ---- cross-lane moves of a double on the data-parallel-primitive paths (no LDS)
template <int CTRL>
__device__ __forceinline__ double dpp_move_d(double v) {
  const unsigned long long b = __builtin_bit_cast(unsigned long long, v);
  const int lo = __builtin_amdgcn_update_dpp(0, (int)(unsigned)b, CTRL, 0xF, 0xF, false);
  const int hi = __builtin_amdgcn_update_dpp(0, (int)(unsigned)(b >> 32), CTRL, 0xF, 0xF, false);
  return __builtin_bit_cast(double, ((unsigned long long)(unsigned)hi << 32) | (unsigned long long)(unsigned)lo);
}
__device__ __forceinline__ double readlane_d(double v, int l) {
  const unsigned long long b = __builtin_bit_cast(unsigned long long, v);
  const unsigned lo = (unsigned)__builtin_amdgcn_readlane((int)(unsigned)b, l);
  const unsigned hi = (unsigned)__builtin_amdgcn_readlane((int)(unsigned)(b >> 32), l);
  return __builtin_bit_cast(double, ((unsigned long long)hi << 32) | (unsigned long long)lo);
}
// the same value in every lane (every lane adds the same pairs in the same order)
__device__ __forceinline__ double wave_sum_dpp(double v) {
  v += dpp_move_d<0xB1>(v);     // quad_perm [1, 0, 3, 2]
  v += dpp_move_d<0x4E>(v);     // quad_perm [2, 3, 0, 1]
  v += dpp_move_d<0x141>(v);    // row_half_mirror: the other quad of the half row
  v += dpp_move_d<0x140>(v);    // row_mirror: the other half of the row of 16
  return (readlane_d(v, 0) + readlane_d(v, 16)) + (readlane_d(v, 32) + readlane_d(v, 48));
}

hipError_t launch_gemm(const GemmArgs &a, int epi, int nz, hipStream_t st, int site);
// the large-M kernel (gemm_i8_big.hip): whether a launch is one of its, and the launch
bool gemm_big_pays(const GemmArgs &a, int epi, int nz);
hipError_t launch_gemm_big(const GemmArgs &a, int epi, hipStream_t st, int site);
// the same with float32 results (rows of N, nothing between them) and row-major weights: whether it pays, and the launches
bool gemm_big_rows_pays(const GemmArgs &a);
hipError_t launch_gemm_big_rows(const GemmArgs &a, hipStream_t st);
// the split-K kernel of small launches (gemm_i8_split.hip): whether a launch is one of them, and the launch
bool gemm_split_pays(const GemmArgs &a, int epi, int nz);
hipError_t launch_gemm_split(const GemmArgs &a, int epi, hipStream_t st);
// row-major codes [N, K] (or packed [N, K/2], K % 16 == 0) -> fragment order, zeros up to the next 32 rows and to Kp (% 32 == 0)
hipError_t launch_tile_weight(const void *q, void *qt, int N, int K, int bits, int Kp, hipStream_t st);

// ---- elementwise / row kernels
hipError_t launch_quantize_act(const float *x, int8_t *q, size_t n, float s, int z_signed, hipStream_t st);
hipError_t launch_quantize_weight(const float *w, int N, int K, int bits, void *qw, float *scale, int32_t *wsum,
                                  hipStream_t st);
// x_bf16 / tok_bf16 below: the residual stream argument is bfloat16 instead of fp32
hipError_t launch_ln_mod_quant(const void *x, int x_bf16, const float *shift, const float *scale, int ld_mod, int M, int D, int T,
                               const QParam *qp, int8_t *q, float *f32_out, hipStream_t st);
// x == nullptr: the inputs are the sinusoidal embeddings (K wide) of the timesteps t_first + row * t_step
hipError_t launch_small_linear(const float *x, int ldx, int t_first, int t_step, const float *W, const float *b, float *y, int ldy, int B, int N,
                               int K, int act_in, int act_out, hipStream_t st);
// te == nullptr: c is given; qp == nullptr: no codes
hipError_t launch_cond_silu(const float *te, const float *table, const int32_t *labels, int n_labels, int null_label, int rows, int B,
                            int D, float *c, int *flags, int L, const QParam *qp, int qp_stride, int8_t *q, size_t l_stride,
                            hipStream_t st);
hipError_t launch_embed(const float *x, const float *pw, const float *pb, const float *pos, void *tok, int tok_bf16, int B,
                        int n_src, int C, int H, int W, int p, int D, int b_off, hipStream_t st);
// The latents that tokens are embedded from: batch element b reads latent b % n_src of x, [C, H, W] each, in patches of p x p
struct EmbedSrc {
  const float *x, *pw, *pb, *pos;
  int n_src, C, H, W, p;
};
// Conditioning of one timestep and a few rows in three launches: whether they cover a call of B rows and M tokens; the hidden layer of
// the timestep MLP beside the patch embedding; its output, c and the codes of SiLU(c); the adaLN projections of nz blocks (a: as for
// launch_gemm) beside the final layer's modulation
bool step_cond_covers(int B, int freq_dim, int C, int p, int D, int M);
hipError_t launch_step_time(int t, const float *w1, const float *b1, float *h1, int freq_dim, const EmbedSrc &e, void *tok, int tok_bf16, int B,
                            int D, hipStream_t st);
hipError_t launch_step_cond(const float *h1, const float *w2, const float *b2, const float *table, const int32_t *labels, int n_labels,
                            int null_label, int B, int D, float *c, int *flags, int L, const QParam *qp, int qp_stride, int8_t *q,
                            size_t l_stride, hipStream_t st);
hipError_t launch_step_mod(const float *cond, const float *fw, const float *fb, float *fmod, int B, int D, const GemmArgs &a, int nz,
                           hipStream_t st);
hipError_t launch_final(const void *tok, int tok_bf16, const float *fmod, const float *fw, const float *fb, float *eps, int B,
                        int C, int H, int W, int p, int D, hipStream_t st);
hipError_t launch_cache_store(const float *src, void *dst, size_t n, bool bf16, hipStream_t st);
hipError_t launch_cache_reuse(void *x, int x_bf16, const void *cached, const float *gate, int ld_gate, int B, int T, int D,
                              bool bf16, hipStream_t st);
hipError_t launch_cached_blocks(void *x, int x_bf16, const void *cache, size_t cache_block_stride, size_t cache_which_stride,
                                const float *mod, size_t mod_block_stride, int ld_mod, int L, int B, int T, int D, bool bf16,
                                hipStream_t st);
hipError_t launch_ddim_vc(float *x, const float *eps, int B, int C, int HW, double cx, double ce, float cfg_scale,
                          const float *K_t, hipStream_t st);
hipError_t launch_vc(float *x, const float *K_t, const float *mu, int B, int C, int HW, hipStream_t st);
hipError_t launch_vc_fit(const float *x_hat, const float *x_ref, int B, int C, int HW, float eps, double *work, float *K_t,
                         hipStream_t st);
hipError_t launch_attention(const float *qkv, int B, int T, int H, int hd, const QParam *qp, int8_t *q_out, float *f32_out,
                            hipStream_t st);
// `beside`: launches of its kind that run at the same time (sub-batches of a denoiser call), this one included
hipError_t launch_attention_f16(const float *q32, const float *k32, const float *vt32, int B, int T, int Tp, int H, int hd,
                                int DPv, const QParam *qp, int8_t *q_out, int beside, hipStream_t st);
// calibration helpers
// gate != null: y[m, :] += gate[m / T, :] * (x W^T + b)[m, :]
hipError_t launch_linear_f32(const float *x, const float *W, const float *b, float *y, int M, int N, int K, int gelu, const float *gate,
                             int ld_gate, int T, hipStream_t st);
// one few-rows linear layer per block: y[l, b, :] = W_l silu(x[b, :]) + b_l, l < n <= BLOCK_LINEARS
constexpr int BLOCK_LINEARS = 32;
struct BlockLinears {
  const float *W[BLOCK_LINEARS], *b[BLOCK_LINEARS];
};
hipError_t launch_block_linears(const BlockLinears &w, int n, const float *x, float *y, size_t block_stride, int B, int N, int K,
                                hipStream_t st);
hipError_t launch_minmax(const float *x, size_t n, int *slot, hipStream_t st);
hipError_t launch_minmax_silu(const float *x, size_t n, int *slot, hipStream_t st);
hipError_t launch_fill_i32(int *p, size_t n, int v, hipStream_t st);

}  // namespace qc
