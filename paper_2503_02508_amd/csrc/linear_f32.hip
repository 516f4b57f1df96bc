// float32 linear layers of the un-quantised reference network (calibration, variance-compensation fit):
// y = act(x W^T + b), every output one chain of float32 fused multiply-adds in ascending k.
//
// The chain runs on the matrix cores: v_mfma_f32_16x16x4_f32 adds its four products one after the other, each with the
// rounding of a fused multiply-add, in ascending k (checked bit by bit against fmaf; the same holds for 32x32x2), so the
// result is that of a plain loop over k, whatever the tile.  That also means that K is never split: the activation ranges
// of the calibration, and with them every quantised code downstream, do not depend on how a product is launched.
//
// A workgroup of four wavefronts (2 x 2) owns a tile of 32 TB x 32 TB outputs, a wavefront TB x TB blocks of 16 x 16.  K is
// walked in slabs of 32 through two LDS buffers (rows of 32 floats padded to 36: the fragment reads, 16 rows x 4
// consecutive floats, fall into 64 different banks), the next slab's loads in flight in registers.  What bounds it: the
// float32 matrix rate (157 TFLOP/s) when the launch fills the chip; otherwise the chain of one output, K / 4 dependent
// instructions of 32 cycles (K = 4608: 18 us).  TB = 2 reads half the bytes per product and is taken when it leaves no
// compute unit idle; TB = 1 makes four times as many workgroups.
#include <math.h>

#include "qc_internal.h"

namespace qc {

typedef float v4f __attribute__((ext_vector_type(4)));

__device__ __forceinline__ float gelu_f(float v) {
  const float k0 = 0.7978845608028654f, k1 = 0.044715f;
  return 0.5f * v * (1.0f + tanhf(k0 * (v + k1 * v * v * v)));
}

template <int TB>
__global__ __launch_bounds__(256) void linear_f32_kernel(const float *__restrict__ x, const float *__restrict__ W,
                                                         const float *__restrict__ bias, float *__restrict__ y, int M, int N, int K,
                                                         int gelu) {
  constexpr int R = 32 * TB, BK = 32, S = BK + 4;
  __shared__ __align__(16) float xs[2][R * S];
  __shared__ __align__(16) float ws[2][R * S];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int m0 = blockIdx.y * R, n0 = blockIdx.x * R;
  const int lr = tid >> 3, lc = (tid & 7) * 4;         // slab row (per pass of 32 rows) and first float of this thread's loads
  const float *px[TB], *pw[TB];
#pragma unroll
  for (int i = 0; i < TB; ++i) {                       // rows beyond the matrix re-read its last row (never stored)
    px[i] = x + (size_t)min(m0 + lr + 32 * i, M - 1) * K;
    pw[i] = W + (size_t)min(n0 + lr + 32 * i, N - 1) * K;
  }
  v4f rx[TB], rw[TB];
  auto load = [&](int k0) {
    const int k = min(k0 + lc, K - 4);                 // a last half slab re-reads its end (never multiplied)
#pragma unroll
    for (int i = 0; i < TB; ++i) {
      rx[i] = *(const v4f *)(px[i] + k);
      rw[i] = *(const v4f *)(pw[i] + k);
    }
  };
  auto store = [&](int b) {
#pragma unroll
    for (int i = 0; i < TB; ++i) {
      *(v4f *)(xs[b] + (lr + 32 * i) * S + lc) = rx[i];
      *(v4f *)(ws[b] + (lr + 32 * i) * S + lc) = rw[i];
    }
  };
  v4f acc[TB][TB];
#pragma unroll
  for (int i = 0; i < TB; ++i)
#pragma unroll
    for (int j = 0; j < TB; ++j) acc[i][j] = (v4f){0.f, 0.f, 0.f, 0.f};
  const int wm = (wave >> 1) * 16 * TB, wn = (wave & 1) * 16 * TB;
  const int fo = (lane & 15) * S + (lane >> 4);        // lane l supplies row l % 16, k = l / 16 of either operand
  load(0);
  store(0);
  if (BK < K) load(BK);
  __syncthreads();
  int b = 0;
  for (int k0 = 0; k0 < K; k0 += BK, b ^= 1) {
    if (k0 + BK < K) store(b ^ 1);
    if (k0 + 2 * BK < K) load(k0 + 2 * BK);
    const float *ax = xs[b] + wm * S + fo, *aw = ws[b] + wn * S + fo;
    const int nq = min(BK, K - k0) / 4;
    auto step = [&](int q) {
      float fx[TB], fw[TB];
#pragma unroll
      for (int i = 0; i < TB; ++i) {
        fx[i] = ax[i * 16 * S + 4 * q];
        fw[i] = aw[i * 16 * S + 4 * q];
      }
#pragma unroll
      for (int i = 0; i < TB; ++i)
#pragma unroll
        for (int j = 0; j < TB; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(fx[i], fw[j], acc[i][j], 0, 0, 0);
    };
    if (nq == BK / 4) {
#pragma unroll
      for (int q = 0; q < BK / 4; ++q) step(q);
    } else {
      for (int q = 0; q < nq; ++q) step(q);
    }
    // one barrier per slab: buffer b is overwritten two slabs on, behind the barrier that everyone passes after reading it
    __syncthreads();
  }
#pragma unroll
  for (int j = 0; j < TB; ++j) {
    const int n = n0 + wn + 16 * j + (lane & 15);
    const float bs = (bias && n < N) ? bias[n] : 0.0f;
#pragma unroll
    for (int i = 0; i < TB; ++i)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int m = m0 + wm + 16 * i + 4 * (lane >> 4) + r;
        if (m < M && n < N) {
          float v = acc[i][j][r] + bs;
          if (gelu) v = gelu_f(v);
          y[(size_t)m * N + n] = v;
        }
      }
  }
}

hipError_t launch_linear_f32(const float *x, const float *W, const float *b, float *y, int M, int N, int K, int gelu, hipStream_t st) {
  if (K % 4 || K < 4) return hipErrorInvalidValue;
  const long long big = (long long)((M + 63) / 64) * ((N + 63) / 64);
  if (big >= 400)
    hipLaunchKernelGGL(linear_f32_kernel<2>, dim3((N + 63) / 64, (M + 63) / 64), dim3(256), 0, st, x, W, b, y, M, N, K, gelu);
  else
    hipLaunchKernelGGL(linear_f32_kernel<1>, dim3((N + 31) / 32, (M + 31) / 32), dim3(256), 0, st, x, W, b, y, M, N, K, gelu);
  return hipGetLastError();
}

}  // namespace qc
