// Bandwidth-bound kernels of the sampler step: activation / weight quantisers,
// LayerNorm + adaLN modulation + quantise, conditioning, patch embedding, final
// layer, cache store / reuse, DDIM update + variance compensation.
// One wavefront is 64 lanes; row reductions use cross-lane shuffles only.
#include "gemm_i8_epilogue.h"

namespace qc {

__device__ __forceinline__ float wave_sum(float v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  return v;
}
__device__ __forceinline__ float wave_max(float v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v = fmaxf(v, __shfl_xor(v, o, 64));
  return v;
}
__device__ __forceinline__ int wave_sum_i(int v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  return v;
}
__device__ __forceinline__ float silu_f(float x) { return x / (1.0f + expf(-x)); }
// Eq. 1 on signed codes: clip(round(v / s) + z, -128, 127), z already shifted.
__device__ __forceinline__ int quant_code(float v, float s, int z) {
  float r = rintf(v / s) + (float)z;
  return (int)fminf(fmaxf(r, -128.0f), 127.0f);
}
__device__ __forceinline__ unsigned pack4(int a, int b, int c, int d) {
  return (unsigned)(a & 0xFF) | ((unsigned)(b & 0xFF) << 8) | ((unsigned)(c & 0xFF) << 16) | ((unsigned)(d & 0xFF) << 24);
}

// ------------------------------------------------------------ quantize_act
__global__ __launch_bounds__(256) void quantize_act_kernel(const float *__restrict__ x, int8_t *__restrict__ q, size_t n,
                                                           float s, int z) {
  const size_t n4 = n >> 2;
  const size_t stride = (size_t)gridDim.x * blockDim.x;
  for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n4; i += stride) {
    float4 v = ((const float4 *)x)[i];
    ((unsigned *)q)[i] = pack4(quant_code(v.x, s, z), quant_code(v.y, s, z), quant_code(v.z, s, z), quant_code(v.w, s, z));
  }
  if (blockIdx.x == 0) {
    size_t i = (n4 << 2) + threadIdx.x;
    if (i < n) q[i] = (int8_t)quant_code(x[i], s, z);
  }
}

hipError_t launch_quantize_act(const float *x, int8_t *q, size_t n, float s, int z, hipStream_t st) {
  if (n == 0) return hipSuccess;
  size_t blocks = ((n >> 2) + 255) / 256;
  if (blocks < 1) blocks = 1;
  if (blocks > 65536) blocks = 65536;
  hipLaunchKernelGGL(quantize_act_kernel, dim3((unsigned)blocks), dim3(256), 0, st, x, q, n, s, z);
  return hipGetLastError();
}

// ---------------------------------------------------------- quantize_weight
// One wavefront per output row: max |w|, scale, codes, row sum.
__global__ __launch_bounds__(256) void quantize_weight_kernel(const float *__restrict__ w, int N, int K, int bits,
                                                              unsigned char *__restrict__ qw, float *__restrict__ scale,
                                                              int32_t *__restrict__ wsum) {
  const int lane = threadIdx.x & 63;
  const int n = blockIdx.x * 4 + (threadIdx.x >> 6);
  if (n >= N) return;
  const float *row = w + (size_t)n * K;
  float amax = 0.0f;
  for (int k = lane; k < K; k += 64) amax = fmaxf(amax, fabsf(row[k]));
  amax = wave_max(amax);
  const float qmax = (float)((1 << (bits - 1)) - 1);
  const float s = amax > 0.0f ? amax / qmax : 1.0f;
  int sum = 0;
  for (int k = 2 * lane; k < K; k += 128) {
    float2 v = *(const float2 *)(row + k);
    int q0 = (int)fminf(fmaxf(rintf(v.x / s), -qmax), qmax);
    int q1 = (int)fminf(fmaxf(rintf(v.y / s), -qmax), qmax);
    sum += q0 + q1;
    if (bits == 4) {
      qw[(size_t)n * (K >> 1) + (k >> 1)] = (unsigned char)((q0 & 0xF) | ((q1 & 0xF) << 4));
    } else {
      *(unsigned short *)(qw + (size_t)n * K + k) = (unsigned short)((q0 & 0xFF) | ((q1 & 0xFF) << 8));
    }
  }
  sum = wave_sum_i(sum);
  if (lane == 0) {
    scale[n] = s;
    wsum[n] = sum;
  }
}

hipError_t launch_quantize_weight(const float *w, int N, int K, int bits, void *qw, float *scale, int32_t *wsum,
                                  hipStream_t st) {
  hipLaunchKernelGGL(quantize_weight_kernel, dim3((N + 3) / 4), dim3(256), 0, st, w, N, K, bits, (unsigned char *)qw, scale,
                     wsum);
  return hipGetLastError();
}

// ------------------------------------------------ weights in fragment order
// Copies the codes of a quantised weight matrix into the order the large-M GEMM streams them in: fragment
// (n / 32, k / 32) is 64 lanes x 16 bytes (8 bytes for packed nibbles), lane l holds row n % 32 = l % 32, k values
// 16 (l / 32) .. 16 (l / 32) + 15 of the group.  One thread per (fragment, lane).
__global__ __launch_bounds__(256) void tile_weight_kernel(const unsigned char *__restrict__ q, unsigned char *__restrict__ qt, int N,
                                                          int K, int Kp, int w4) {
  const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int ng = Kp / 32;
  if (i >= (size_t)((N + 31) / 32) * ng * 64) return;
  const int l = (int)(i & 63), kg = (int)((i >> 6) % ng), nb = (int)((i >> 6) / ng);
  const size_t n = (size_t)nb * 32 + (l & 31);
  const int k = kg * 32 + (l >> 5) * 16;
  const bool in = n < (size_t)N && k < K;         // K is a multiple of 16
  if (w4) *(uint2 *)(qt + i * 8) = in ? *(const uint2 *)(q + n * (K >> 1) + (k >> 1)) : make_uint2(0, 0);
  else *(uint4 *)(qt + i * 16) = in ? *(const uint4 *)(q + n * K + k) : make_uint4(0, 0, 0, 0);
}

hipError_t launch_tile_weight(const void *q, void *qt, int N, int K, int bits, int Kp, hipStream_t st) {
  if (K % 16 || Kp % 32 || Kp < K) return hipErrorInvalidValue;
  const size_t n = (size_t)((N + 31) / 32) * (Kp / 32) * 64;
  hipLaunchKernelGGL(tile_weight_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, (const unsigned char *)q,
                     (unsigned char *)qt, N, K, Kp, bits == 4 ? 1 : 0);
  return hipGetLastError();
}

// ------------------------------------------- LayerNorm + modulate + quantise
// One wavefront per token row; the row lives in registers (D <= 2048).
constexpr int LN_MAX_IT = 8;

__device__ __forceinline__ double wave_sum_d(double v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  return v;
}

// v_permlane32_swap / v_permlane16_swap: the upper half (the odd rows of 16) of a changes places with the lower half (the even rows) of b
template <int W>
__device__ __forceinline__ void swap_rows(double a, double b, double &a2, double &b2) {
  typedef unsigned u2 __attribute__((ext_vector_type(2)));
  const unsigned long long x = __builtin_bit_cast(unsigned long long, a), y = __builtin_bit_cast(unsigned long long, b);
  u2 lo, hi;
  if constexpr (W == 32) {
    lo = __builtin_amdgcn_permlane32_swap((unsigned)x, (unsigned)y, false, false);
    hi = __builtin_amdgcn_permlane32_swap((unsigned)(x >> 32), (unsigned)(y >> 32), false, false);
  } else {
    lo = __builtin_amdgcn_permlane16_swap((unsigned)x, (unsigned)y, false, false);
    hi = __builtin_amdgcn_permlane16_swap((unsigned)(x >> 32), (unsigned)(y >> 32), false, false);
  }
  a2 = __builtin_bit_cast(double, ((unsigned long long)hi[0] << 32) | lo[0]);
  b2 = __builtin_bit_cast(double, ((unsigned long long)hi[1] << 32) | lo[1]);
}

// Both sums of a wavefront at once: the first in lanes 0 .. 31, the second in 32 .. 63 ...
__device__ __forceinline__ double wave_sum_halves(double a, double b) {
  double v, w;
  swap_rows<32>(a, b, v, w);
  v += w;
  v += dpp_move_d<0xB1>(v);     // as in wave_sum_dpp
  v += dpp_move_d<0x4E>(v);
  v += dpp_move_d<0x141>(v);
  v += dpp_move_d<0x140>(v);
  swap_rows<16>(v, v, v, w);
  return v + w;
}
// ... and both in every lane.
__device__ __forceinline__ void wave_sum_pair(double &a, double &b) {
  const double v = wave_sum_halves(a, b);
  swap_rows<32>(v, v, a, b);
}

// The value that gets quantised is formed in fp64 and rounded to fp32 once: the codes then differ from
// exact arithmetic only where the fp32 residual stream itself does, which keeps code flips (and the
// error they seed in every later layer) at the floor.
// One workgroup per R consecutive token rows, one float4 of every row per thread (the launch sizes the workgroup to
// D / 4 rounded up to whole wavefronts, D <= 2048): every load of the rows and of their modulation vectors is issued
// at once, one memory round trip.  R = 1 gives the most workgroups (small M); R = 4 puts four times the bytes in
// flight per compute unit, which is what the memory system needs to run near its peak at large M.  The arithmetic of a
// row, and with it every code, is the same for both.  What bounds a small launch is its chain of round trips: the parameters come with the
// rows, the sums of a wavefront meet in lane moves and, ALL, every thread finishes the statistics, behind one barrier (256 rows of
// 1152 3.10 -> 2.86 us, 425 3.53 -> 3.08).  A large launch has the double-precision division and square root of all its wavefronts to issue
// instead (8192 rows of 2048 25 -> 32 us): there one thread a row finishes them and a second barrier hands them on.
template <int R, bool ALL>
__global__ __launch_bounds__(512) void ln_mod_quant_kernel(const void *__restrict__ x, int x_bf16, const float *__restrict__ shift,
                                                           const float *__restrict__ scale, int ld_mod, int M, int D, int T,
                                                           const QParam *qp, int8_t *__restrict__ q,
                                                           float *__restrict__ f32_out) {
  __shared__ double red[R][16];
  const int m0 = blockIdx.x * R;
  const int k = threadIdx.x * 4;
  const bool live = k < D;
  const int kc = live ? k : 0;
  float4 v[R], s4[R], c4[R];
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const int m = min(m0 + r, M - 1);             // rows beyond M re-read the last row (never stored)
    const int b = m / T;
    v[r] = stream_load4(x, ((size_t)m * D + kc) >> 2, x_bf16);
    s4[r] = *(const float4 *)(shift + (size_t)b * ld_mod + kc);
    c4[r] = *(const float4 *)(scale + (size_t)b * ld_mod + kc);
  }
  float qs = 1.0f;                                // requested with the rows
  int qz = 0;
  if (qp) {
    const QParam t = *qp;
    qs = t.s;
    qz = t.z;
  }
  // mean and variance from one reduction of (sum, sum of squares): in fp64 the cancellation in
  // E[x^2] - mean^2 costs ~1e-13 relative for rows of O(1) values, far below the fp32 rounding of the result
  const int nw = blockDim.x >> 6;
#pragma unroll
  for (int r = 0; r < R; ++r) {
    double sum = 0.0, sq = 0.0;
    if (live) {
      const double a = v[r].x, bq = v[r].y, c = v[r].z, d = v[r].w;
      sum = (a + bq) + (c + d);
      sq = (a * a + bq * bq) + (c * c + d * d);
    }
    wave_sum_pair(sum, sq);
    if ((threadIdx.x & 63) == 0) {
      red[r][threadIdx.x >> 6] = sum;
      red[r][8 + (threadIdx.x >> 6)] = sq;
    }
  }
  __syncthreads();
  const auto finish = [&](int r, double &mean, double &rstd) {
    double tot = 0.0, tot2 = 0.0;
    for (int w = 0; w < nw; ++w) {
      tot += red[r][w];
      tot2 += red[r][8 + w];
    }
    mean = tot / (double)D;
    const double var = tot2 / (double)D - mean * mean;
    rstd = 1.0 / sqrt(fmax(var, 0.0) + 1e-6);
  };
  double stat[R][2];
  if constexpr (ALL) {
#pragma unroll
    for (int r = 0; r < R; ++r) finish(r, stat[r][0], stat[r][1]);
  } else {
    __shared__ double stat_s[R][2];
    if (threadIdx.x < R) finish(threadIdx.x, stat_s[threadIdx.x][0], stat_s[threadIdx.x][1]);
    __syncthreads();
#pragma unroll
    for (int r = 0; r < R; ++r) {
      stat[r][0] = stat_s[r][0];
      stat[r][1] = stat_s[r][1];
    }
  }
  if (!live) return;
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const int m = m0 + r;
    if (m >= M) break;
    const double mean = stat[r][0], rstd = stat[r][1];
    const float h0 = (float)((v[r].x - mean) * rstd * (1.0 + (double)c4[r].x) + (double)s4[r].x);
    const float h1 = (float)((v[r].y - mean) * rstd * (1.0 + (double)c4[r].y) + (double)s4[r].y);
    const float h2 = (float)((v[r].z - mean) * rstd * (1.0 + (double)c4[r].z) + (double)s4[r].z);
    const float h3 = (float)((v[r].w - mean) * rstd * (1.0 + (double)c4[r].w) + (double)s4[r].w);
    if (q)
      *(unsigned *)(q + (size_t)m * D + k) =
          pack4(quant_code(h0, qs, qz), quant_code(h1, qs, qz), quant_code(h2, qs, qz), quant_code(h3, qs, qz));
    if (f32_out) *(float4 *)(f32_out + (size_t)m * D + k) = make_float4(h0, h1, h2, h3);
  }
}

// ---- one wavefront per token row
// The wavefront-per-row form of the same operation, for launches of many rows (launch_ln_mod_quant): a lane holds NV float4 of
// the row (float4 index lane + 64 it), the sums of values and squares stay inside the wavefront (no LDS, no barrier), a wavefront walks
// `rows_per_wave` consecutive rows with the next row's loads in flight while it works on the current one, and keeps the modulation
// vectors of the batch element in registers from row to row.
//
// Mean and variance are float64 sums; the code of an element is decided in float32 where that is certain to be the code of the float64
// value.  With c' = (1 + scale) / s and s' = shift / s + zero point (formed once a batch element),
//   v = ((x - mean) rstd) c',   q = v + s',   code = q rounded to nearest even, clamped to 0 .. 255 (the paper's unsigned code)
// is off the value that Eq. 1 rounds by at most, in units of 2^-24: of |v| 1 (x - mean) + 3 (reciprocal square root, its argument) + 2
// (two products) + 3.5 (c': 1 + scale, 1 / s, their product) + 1 (the sum) + 2 (on the other side, the value's rounding to float32 and
// the quotient's) = 12.5, and of |shift| / s 1.5 + 1 (s') + 1 (the sum) + 2; the zero point in s' and in the sum, 2^-17 each below 256 (beyond,
// every value clamps to the same code); and the mean's rounding, |mean| rstd |c'|.  So an element is in doubt when q lies closer than
// 8e-7 |v| + near to a half, near = 1.6e-5 + 3.4e-7 |shift| / s + 6.2e-8 |mean| rstd |c'| (maxima and sums of the lane's columns): about
// 8e-5 of the elements; the wavefront's values around them take the float64 expression and the IEEE quotient (ln_codes_exact).  A row
// or a column whose window is not finite is in doubt throughout.
//
// What bounds it: at thousands of rows the memory system (32768 rows of 1152, 189 MB, in 31 us, the input in the memory-side cache in
// part); else vector issue, some 13 instructions an element and 50 a row for the sums (in pairs: the sum of the values in the lower half
// of the wavefront, that of the squares in the upper).  With every value in float64 it was 34 an element: 8192 rows 13.6 -> 11.1 us, 32768
// 38 -> 31, bfloat16 rows, whose conversion also waited for the loads, 46 -> 26.  In the sampler, beside the other half's attention, whose two
// wavefronts leave a SIMD no registers for another, it gained 1 - 2 % of a run of 16 x 1024 tokens.
__device__ __forceinline__ unsigned ln_codes_exact(float4 x, float4 c, float4 sh, double mean, double var, float s, float zu) {
  const double rstd = 1.0 / sqrt(fmax(var, 0.0) + 1e-6);
  const float xs[4] = {x.x, x.y, x.z, x.w}, cs[4] = {c.x, c.y, c.z, c.w}, ss[4] = {sh.x, sh.y, sh.z, sh.w};
  unsigned w = 0;
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    const float h = (float)((xs[e] - mean) * rstd * (1.0 + (double)cs[e]) + (double)ss[e]);
    w = __builtin_amdgcn_cvt_pk_u8_f32(__builtin_amdgcn_fmed3f(__builtin_rintf(h / s) + zu, 0.0f, 255.0f), e, w);
  }
  return w;
}

// ONE: a wavefront has one row, no next one to request (1024 rows 5.8 -> 5.5 us beside the other half's kernels).
template <int NV, bool BF16, bool ONE>
__global__ __launch_bounds__(256) void ln_mod_quant_wave_kernel(const void *__restrict__ x, const float *__restrict__ shift,
                                                                const float *__restrict__ scale, int ld_mod, int M, int D, int T,
                                                                const QParam *qp, int8_t *__restrict__ q, int rows_per_wave) {
  typedef typename std::conditional<BF16, uint2, float4>::type raw4;      // four elements as they lie in memory
  const auto value4 = [](const raw4 &r) {
    if constexpr (BF16)
      return make_float4(__builtin_bit_cast(float, r.x << 16), __builtin_bit_cast(float, r.x & 0xFFFF0000u),
                         __builtin_bit_cast(float, r.y << 16), __builtin_bit_cast(float, r.y & 0xFFFF0000u));
    else
      return r;
  };
  const int lane = threadIdx.x & 63;
  const int wv = __builtin_amdgcn_readfirstlane(blockIdx.x * 4 + (threadIdx.x >> 6));
  const int m_begin = wv * rows_per_wave;
  if (m_begin >= M) return;                        // whole wavefronts leave; the kernel has no barrier
  const int m_end = min(m_begin + rows_per_wave, M);
  const int nv4 = D >> 2;                          // 64 (NV - 1) < nv4 <= 64 NV: only the last float4 of a lane may lie beyond the row
  const bool in_last = lane + 64 * (NV - 1) < nv4;
  int kc[NV];
#pragma unroll
  for (int it = 0; it < NV; ++it) kc[it] = it < NV - 1 || in_last ? lane + 64 * it : 0;
  const QParam t = *qp;
  const float qs = t.s, zu = (float)(t.z + 128), inv_s = 1.0f / t.s;
  const double inv_d = 1.0 / (double)D;
  float4 xa[NV], cq[NV], sq4[NV];
  raw4 xn[NV];
#pragma unroll
  for (int it = 0; it < NV; ++it) xa[it] = value4(((const raw4 *)x)[(((size_t)m_begin * D) >> 2) + kc[it]]);
  float near_s = 0.f, near_c = 0.f;
  int b = m_begin / T, left = 0;                   // batch element; rows that its vectors in registers still serve
  for (int m = m_begin; m < m_end; ++m) {
    const int mn = min(m + 1, m_end - 1);          // the last row is requested once more (never used)
#pragma unroll
    for (int it = 0; it < NV && !ONE; ++it) xn[it] = ((const raw4 *)x)[(((size_t)mn * D) >> 2) + kc[it]];
    if (left == 0) {
      if (m > m_begin) ++b;
      left = (b + 1) * T - m;
      near_c = near_s = 0.f;
#pragma unroll
      for (int it = 0; it < NV; ++it) {
        const float4 sv = *(const float4 *)(shift + (size_t)b * ld_mod + 4 * kc[it]), cv = *(const float4 *)(scale + (size_t)b * ld_mod + 4 * kc[it]);
        cq[it] = make_float4((1.f + cv.x) * inv_s, (1.f + cv.y) * inv_s, (1.f + cv.z) * inv_s, (1.f + cv.w) * inv_s);
        sq4[it] = make_float4(fmaf(sv.x, inv_s, zu), fmaf(sv.y, inv_s, zu), fmaf(sv.z, inv_s, zu), fmaf(sv.w, inv_s, zu));
        near_c += (fabsf(cq[it].x) + fabsf(cq[it].y)) + (fabsf(cq[it].z) + fabsf(cq[it].w));      // (a NaN stays)
        near_s = fmaxf(near_s, fmaxf(fmaxf(fabsf(sv.x), fabsf(sv.y)), fmaxf(fabsf(sv.z), fabsf(sv.w))));
      }
      near_c *= 6.2e-8f;
      near_s = fmaf(3.4e-7f * near_s, inv_s, 1.6e-5f);
    }
    --left;
    if (!in_last) xa[NV - 1] = make_float4(0.f, 0.f, 0.f, 0.f);
    double sum = 0.0, sq = 0.0;
#pragma unroll
    for (int it = 0; it < NV; ++it) {
      const double a0 = xa[it].x, a1 = xa[it].y, a2 = xa[it].z, a3 = xa[it].w;
      sum += (a0 + a1) + (a2 + a3);
      sq = fma(a0, a0, fma(a1, a1, fma(a2, a2, fma(a3, a3, sq))));
    }
    double v = wave_sum_halves(sum, sq);
    const double est = v * inv_d;                  // v / D: the quotient's estimate with its remainder divided once more
    v = fabs(est) < 1e300 ? fma(fma(-est, (double)D, v), inv_d, est) : est;
    double mean, var;
    swap_rows<32>(v, v, mean, var);
    var = var - mean * mean;
    const float mh = (float)mean, vf = (float)fmax(var, 0.0) + 1e-6f;
    const float rstd = __builtin_amdgcn_rsqf(vf);
    // a variance beyond float32's range: every element in doubt
    const float near = vf < 1e37f ? fmaf(near_c * fabsf(mh), rstd, near_s) : INFINITY;
    unsigned w[NV];
    float least[NV];
    bool doubt = false;
#pragma unroll
    for (int it = 0; it < NV; ++it) {
      const float xs[4] = {xa[it].x, xa[it].y, xa[it].z, xa[it].w}, cs[4] = {cq[it].x, cq[it].y, cq[it].z, cq[it].w};
      const float ss[4] = {sq4[it].x, sq4[it].y, sq4[it].z, sq4[it].w};
      float clear[4];
      w[it] = 0;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const float u = ((xs[e] - mh) * rstd) * cs[e];
        const float qv = u + ss[e];
        w[it] = __builtin_amdgcn_cvt_pk_u8_f32(qv, e, w[it]);
        clear[e] = fmaf(-8e-7f, fabsf(u), fabsf(__builtin_amdgcn_fractf(qv) - 0.5f));
      }
      least[it] = fminf(fminf(clear[0], clear[1]), fminf(clear[2], clear[3]));
      doubt = doubt || !(least[it] >= near);
    }
    if (__builtin_amdgcn_ballot_w64(doubt) != 0ull) {
#pragma unroll
      for (int it = 0; it < NV; ++it)
        if (__builtin_amdgcn_ballot_w64(!(least[it] >= near)) != 0ull)
          w[it] = ln_codes_exact(xa[it], *(const float4 *)(scale + (size_t)b * ld_mod + 4 * kc[it]), *(const float4 *)(shift + (size_t)b * ld_mod + 4 * kc[it]),
                                 mean, var, qs, zu);
    }
#pragma unroll
    for (int it = 0; it < NV; ++it)
      if (it < NV - 1 || in_last) *(unsigned *)(q + (size_t)m * D + 4 * kc[it]) = w[it] ^ 0x80808080u;
#pragma unroll
    for (int it = 0; it < NV && !ONE; ++it) xa[it] = value4(xn[it]);
  }
}

hipError_t launch_ln_mod_quant(const void *x, int x_bf16, const float *shift, const float *scale, int ld_mod, int M, int D, int T,
                               const QParam *qp, int8_t *q, float *f32_out, hipStream_t st) {
  const int threads = ((D / 4 + 63) / 64) * 64;
  if (D % 4 || threads > 512) return hipErrorInvalidValue;
  const int nv = (D / 4 + 63) / 64;
  if (q && !f32_out && M >= 640 && nv <= 5) {
    // wavefront per row; with thousands of rows several consecutive ones (they share the batch element's modulation vectors and its
    // float32 constants).  1 / 2 / 4 / 8 rows, us (width 1152): 2048 rows 4.2 / 4.9 / 6.6 / 9.8, 4096: 6.7 / 6.2 / 7.0 / 10.0, 8192: 11.9 / 12.2 /
    // 11.0 / 12.5, 32768: 33.8 / 32.7 / 31.8 / 34.7; narrower rows 1 / 2 / 4: 4096 of 384 3.9 / 4.2 / 4.8, of 768 4.8 / 4.8 / 5.5, 8192 of 384 5.7 / 5.5 /
    // 5.8, of 1024 10.3 / 9.4 / 9.8.  (bfloat16 rows alone would rather have one up to 6144, 4096 of 1152 8.8 / 9.5 / 10.5; beside the other half's
    // kernels one row costs networks of width 768 and 1152 1 %.)
    // From where, a workgroup a row | a wavefront a row, networks in two halves, width 1152: 768 rows a half 4709 | 4657 us, 960 5953 | 5871, 1000 7943 |
    // 7801; in one part, and with widths of 128 to 768, the sides differ by less than runs of one do (1 - 3 %).  1024 rows alone: 3.7 | 3.5
    const int rpw = M >= 8192 ? 4 : M >= 4096 ? 2 : 1;
    const int waves = (M + rpw - 1) / rpw;
    const dim3 grid((waves + 3) / 4);
#define QC_LN_AS(NV, BF16, ONE) \
  hipLaunchKernelGGL((ln_mod_quant_wave_kernel<NV, BF16, ONE>), grid, dim3(256), 0, st, x, shift, scale, ld_mod, M, D, T, qp, q, rpw)
#define QC_LN(NV)                                  \
  do {                                             \
    if (x_bf16 && rpw == 1) QC_LN_AS(NV, true, true); \
    else if (x_bf16) QC_LN_AS(NV, true, false);    \
    else if (rpw == 1) QC_LN_AS(NV, false, true);  \
    else QC_LN_AS(NV, false, false);               \
  } while (0)
    switch (nv) {
      case 1: QC_LN(1); break;
      case 2: QC_LN(2); break;
      case 3: QC_LN(3); break;
      case 4: QC_LN(4); break;
      default: QC_LN(5); break;
    }
#undef QC_LN
#undef QC_LN_AS
  } else if (M >= 8192)
    hipLaunchKernelGGL((ln_mod_quant_kernel<4, false>), dim3((M + 3) / 4), dim3(threads), 0, st, x, x_bf16, shift, scale, ld_mod, M, D, T,
                       qp, q, f32_out);
  else if (M * nv <= 2400 && nv < 8)
    // every thread finishes the statistics while the launch has fewer wavefronts than the chip finishes side by side.  Every thread | one,
    // us: 256 rows of 384 2.36 | 2.48, 512 of 768 2.75 | 2.78, 512 of 1152 3.12 | 3.09, 800 of 768 3.20 | 3.13, 800 of 1152 4.28 | 3.46; 16 rows
    // of 1536 2.73 | 2.76, of 2048 2.63 | 2.53
    hipLaunchKernelGGL((ln_mod_quant_kernel<1, true>), dim3(M), dim3(threads), 0, st, x, x_bf16, shift, scale, ld_mod, M, D, T, qp, q,
                       f32_out);
  else
    hipLaunchKernelGGL((ln_mod_quant_kernel<1, false>), dim3(M), dim3(threads), 0, st, x, x_bf16, shift, scale, ld_mod, M, D, T, qp, q,
                       f32_out);
  return hipGetLastError();
}

// ------------------------------------------------- small linear (few rows)
// y[b, n] = act_out(W[n, :] . act_in(x[b, :]) + bias[n]); one wavefront per n.  Inputs and outputs are float32 tensors;
// the arithmetic in between is float64 and the result is rounded once, so that what is stored does not depend on the
// summation order (conditioning vectors feed quantisers, where a last-bit difference can move a code).
__device__ __forceinline__ double silu_d(double x) { return x / (1.0 + exp(-x)); }

// Widths that the kernel below does not cover (a timestep embedding whose width is not a multiple of 4 or beyond 2048): one
// wavefront per output.
__device__ __forceinline__ float time_embed_value(int t, int k, int dim);
__global__ __launch_bounds__(256) void small_linear_any_kernel(const float *__restrict__ x, int ldx, int t_first, int t_step,
                                                               const float *__restrict__ W, const float *__restrict__ bias,
                                                               float *__restrict__ y, int ldy, int N, int K, int act_in, int act_out) {
  const int lane = threadIdx.x & 63, n = blockIdx.x * 4 + (threadIdx.x >> 6), b = blockIdx.y;
  if (n >= N) return;
  double t = 0.0;
  for (int k = lane; k < K; k += 64) {
    double v = x ? (double)x[(size_t)b * ldx + k] : (double)time_embed_value(t_first + b * t_step, k, K);
    if (act_in == 1) v = silu_d(v);
    t = fma((double)W[(size_t)n * K + k], v, t);
  }
  t = wave_sum_d(t);
  if (lane == 0) {
    t += bias ? (double)bias[n] : 0.0;
    if (act_out == 1) t = silu_d(t);
    y[(size_t)b * ldy + n] = (float)t;
  }
}
static hipError_t launch_small_linear_any(const float *x, int ldx, int t_first, int t_step, const float *W, const float *b, float *y, int ldy,
                                          int B, int N, int K, int act_in, int act_out, hipStream_t st) {
  hipLaunchKernelGGL(small_linear_any_kernel, dim3((N + 3) / 4, B), dim3(256), 0, st, x, ldx, t_first, t_step, W, b, y, ldy, N, K, act_in,
                     act_out);
  return hipGetLastError();
}

// One workgroup = R rows x 16 outputs: the (activated) inputs of the R rows are formed once, in float64, and kept in LDS (the
// activation is an exponential per value: it must not be repeated per output); a wavefront takes four outputs, so that
// every input value read from LDS and every weight read from memory feeds 4 and R multiply-adds.  A lane owns four
// consecutive k of every 256 and requests its whole share of the four weight rows at once (NIT x 4 16-byte loads); the 4 R
// sums are then reduced together, each exchange between lanes halving the number of sums a lane still carries.
// x == nullptr: the inputs are the sinusoidal embeddings of the timesteps t_first + row * t_step (rounded to float32, as the
// stored embedding would be).
// Bound: the weights' bytes for a few rows (float32, read once per R rows), the float64 rate for many.  Rows are taken R =
// 1, 2, 4 or 8 at a time, whichever covers them: absent rows used to cost as much as real ones (one row of 256 inputs and
// 384 outputs 15 us, now 4.5; 6912 x 1152 weights, two rows: 41 us, now 13).
__device__ __forceinline__ float time_embed_value(int t, int k, int dim) {
  // [cos | sin], frequencies exp(-ln(1e4) j / half), evaluated in double so that the float32 result is correctly rounded
  const int half = dim / 2, f = k < half ? k : k - half;
  const double a = (double)t * exp(-log(10000.0) * (double)f / (double)half);
  return (float)(k < half ? cos(a) : sin(a));
}

// The parts of it, 256 threads each; xs: [R][K] of LDS.  The weights of a workgroup's outputs n0 .. n0 + 15 ...
template <int NIT>
__device__ __forceinline__ void small_linear_weights(float4 (&w4)[NIT][4], int n0, const float *__restrict__ W, int N, int K) {
  const int lane = threadIdx.x & 63, nw = n0 + (threadIdx.x >> 6) * 4;
#pragma unroll
  for (int it = 0; it < NIT; ++it)
#pragma unroll
    for (int j = 0; j < 4; ++j)                   // outputs beyond N repeat the last, k beyond K the row's end (multiplied by zero)
      w4[it][j] = *(const float4 *)(W + (size_t)min(nw + j, N - 1) * K + min(4 * (lane + 64 * it), K - 4));
}
// ... the inputs of rows b0 .. b0 + R - 1 ...
template <int R>
__device__ __forceinline__ void small_linear_inputs(double *xs, int b0, const float *__restrict__ x, int ldx, int t_first, int t_step, int B,
                                                    int K, int act_in) {
  for (int i = threadIdx.x; i < R * K; i += 256) {
    const int r = i / K, k = i - r * K;
    double v = 0.0;
    if (b0 + r < B) {
      v = x ? (double)x[(size_t)(b0 + r) * ldx + k] : (double)time_embed_value(t_first + (b0 + r) * t_step, k, K);
      if (act_in == 1) v = silu_d(v);
    }
    xs[i] = v;
  }
  __syncthreads();
}
// ... and the results: out(row, n, value) takes one (in one lane)
template <int R, int NIT, typename Out>
__device__ __forceinline__ void small_linear_dot(const double *xs, const float4 (&w4)[NIT][4], int b0, int n0, const float *__restrict__ bias,
                                                 int B, int N, int K, int act_out, const Out &out) {
  const int lane = threadIdx.x & 63;
  n0 += (threadIdx.x >> 6) * 4;
  double part[4 * R];                             // sum of (row r, output j) at r * 4 + j
#pragma unroll
  for (int i = 0; i < 4 * R; ++i) part[i] = 0.0;
#pragma unroll
  for (int it = 0; it < NIT; ++it) {
    const int k = 4 * (lane + 64 * it);
    if (k < K) {
#pragma unroll
      for (int r = 0; r < R; ++r) {
        const double x0 = xs[r * K + k], x1 = xs[r * K + k + 1], x2 = xs[r * K + k + 2], x3 = xs[r * K + k + 3];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          part[r * 4 + j] = fma((double)w4[it][j].x, x0, part[r * 4 + j]);
          part[r * 4 + j] = fma((double)w4[it][j].y, x1, part[r * 4 + j]);
          part[r * 4 + j] = fma((double)w4[it][j].z, x2, part[r * 4 + j]);
          part[r * 4 + j] = fma((double)w4[it][j].w, x3, part[r * 4 + j]);
        }
      }
    }
  }
  // exchange over distance 32, 16, ...: a lane keeps the upper or lower half of its sums, as its own lane bit says
  int mine = 0;
  constexpr int V = 4 * R;
#pragma unroll
  for (int s2 = 0, half = V / 2; half > 0; ++s2, half >>= 1) {
    const int dist = 32 >> s2;
    const bool upper = (lane & dist) != 0;
    mine += upper ? half : 0;
#pragma unroll
    for (int u = 0; u < half; ++u) {
      const double keep = upper ? part[u + half] : part[u];
      const double send = upper ? part[u] : part[u + half];
      part[u] = keep + __shfl_xor(send, dist, 64);
    }
  }
  double t = part[0];
#pragma unroll
  for (int dist = 32 / V; dist > 0; dist >>= 1) t += __shfl_xor(t, dist, 64);
  const int r = mine >> 2, n = n0 + (mine & 3);
  if ((lane & (64 / V - 1)) == 0 && b0 + r < B && n < N) {
    t += bias ? (double)bias[n] : 0.0;
    if (act_out == 1) t = silu_d(t);
    out(b0 + r, n, (float)t);
  }
}

template <int R, int NIT, typename Out>
__device__ __forceinline__ void small_linear_tile(double *xs, int bx, int by, const float *__restrict__ x, int ldx, int t_first, int t_step,
                                                  const float *__restrict__ W, const float *__restrict__ bias, int B, int N, int K,
                                                  int act_in, int act_out, const Out &out) {
  float4 w4[NIT][4];                              // first: they do not depend on the inputs
  small_linear_weights<NIT>(w4, bx * 16, W, N, K);
  small_linear_inputs<R>(xs, by * R, x, ldx, t_first, t_step, B, K, act_in);
  small_linear_dot<R, NIT>(xs, w4, by * R, bx * 16, bias, B, N, K, act_out, out);
}

template <int R, int NIT>
__global__ __launch_bounds__(256) void small_linear_kernel(const float *__restrict__ x, int ldx, int t_first, int t_step,
                                                           const float *__restrict__ W, const float *__restrict__ bias,
                                                           float *__restrict__ y, int ldy, int B, int N, int K, int act_in, int act_out) {
  extern __shared__ double xs[];                  // [R][K]
  small_linear_tile<R, NIT>(xs, blockIdx.x, blockIdx.y, x, ldx, t_first, t_step, W, bias, B, N, K, act_in, act_out,
                            [&](int b, int n, float v) { y[(size_t)b * ldy + n] = v; });
}

template <int R, int NIT>
static hipError_t launch_small_linear_as(const float *x, int ldx, int t_first, int t_step, const float *W, const float *b, float *y, int ldy,
                                         int B, int N, int K, int act_in, int act_out, hipStream_t st) {
  const size_t smem = (size_t)R * K * sizeof(double);
  if (smem > 64 * 1024) {                         // more than a kernel may use without asking: ask once, for the widest input
    static std::atomic<unsigned long long> lds{0};
    if (const hipError_t e = allow_lds((const void *)small_linear_kernel<R, NIT>, R * 256 * NIT * (int)sizeof(double), lds)) return e;
  }
  hipLaunchKernelGGL((small_linear_kernel<R, NIT>), dim3((N + 15) / 16, (B + R - 1) / R), dim3(256), smem, st, x, ldx, t_first, t_step, W, b,
                     y, ldy, B, N, K, act_in, act_out);
  return hipGetLastError();
}

template <int R>
static hipError_t launch_small_linear_rows(const float *x, int ldx, int t_first, int t_step, const float *W, const float *b, float *y, int ldy,
                                           int B, int N, int K, int act_in, int act_out, hipStream_t st) {
  if (K <= 256) return launch_small_linear_as<R, 1>(x, ldx, t_first, t_step, W, b, y, ldy, B, N, K, act_in, act_out, st);
  if (K <= 512) return launch_small_linear_as<R, 2>(x, ldx, t_first, t_step, W, b, y, ldy, B, N, K, act_in, act_out, st);
  if (K <= 1280) return launch_small_linear_as<R, 5>(x, ldx, t_first, t_step, W, b, y, ldy, B, N, K, act_in, act_out, st);
  return launch_small_linear_as<R, 8>(x, ldx, t_first, t_step, W, b, y, ldy, B, N, K, act_in, act_out, st);
}

// x == nullptr: rows are the embeddings of timesteps t_first, t_first + t_step, ... (K wide)
hipError_t launch_small_linear(const float *x, int ldx, int t_first, int t_step, const float *W, const float *b, float *y, int ldy, int B, int N,
                               int K, int act_in, int act_out, hipStream_t st) {
  if (K % 4 || K > 2048) return launch_small_linear_any(x, ldx, t_first, t_step, W, b, y, ldy, B, N, K, act_in, act_out, st);
  if (B <= 1) return launch_small_linear_rows<1>(x, ldx, t_first, t_step, W, b, y, ldy, B, N, K, act_in, act_out, st);
  if (B <= 2) return launch_small_linear_rows<2>(x, ldx, t_first, t_step, W, b, y, ldy, B, N, K, act_in, act_out, st);
  if (B <= 4) return launch_small_linear_rows<4>(x, ldx, t_first, t_step, W, b, y, ldy, B, N, K, act_in, act_out, st);
  return launch_small_linear_rows<8>(x, ldx, t_first, t_step, W, b, y, ldy, B, N, K, act_in, act_out, st);
}

// The same for one linear layer per block in one launch (grid z): the weights of all blocks stream from memory once for up to eight rows,
// where a launch per block and half of the samples stood in the chain of the un-quantised network (18 us each, DiT-XL/2, two samples).
// Four rows at a time | eight, us, 28 blocks of width 1152: 4 rows 274 | 292, 8 rows 524 | 328, 64 rows 3654 | 2175 (a launch a block 4671); 12
// of 384: 64 rows 343 | 127 (239).  A workgroup takes 4 x 16 outputs, which share the activated inputs.  With the gated additions in the products' epilogues (4.6 us
// each), a factor fit of 3 steps and 2 latents takes 19.3 -> 18.4 ms.
constexpr int BL_TILES = 4;
template <int R, int NIT>
__global__ __launch_bounds__(256) void block_linears_kernel(BlockLinears w, const float *__restrict__ x, float *__restrict__ y, size_t block_stride,
                                                            int B, int N, int K) {
  extern __shared__ double xs[];                  // [R][K]
  const int b0 = blockIdx.y * R;
  const float *const W = w.W[blockIdx.z], *const bias = w.b[blockIdx.z];
  float *const yz = y + blockIdx.z * block_stride;
  float4 w4[NIT][4];
  small_linear_weights<NIT>(w4, blockIdx.x * BL_TILES * 16, W, N, K);
  small_linear_inputs<R>(xs, b0, x, K, 0, 0, B, K, 1);
  for (int i = 0; i < BL_TILES; ++i) {
    const int n0 = (blockIdx.x * BL_TILES + i) * 16;
    if (n0 >= N) return;
    if (i) small_linear_weights<NIT>(w4, n0, W, N, K);
    small_linear_dot<R, NIT>(xs, w4, b0, n0, bias, B, N, K, 0, [&](int b, int n, float v) { yz[(size_t)b * N + n] = v; });
  }
}

template <int R, int NIT>
static hipError_t launch_block_linears_as(const BlockLinears &w, int n, const float *x, float *y, size_t block_stride, int B, int N, int K,
                                          hipStream_t st) {
  const size_t smem = (size_t)R * K * sizeof(double);
  if (smem > 64 * 1024) {                         // as for one linear
    static std::atomic<unsigned long long> lds{0};
    if (const hipError_t e = allow_lds((const void *)block_linears_kernel<R, NIT>, R * 256 * NIT * (int)sizeof(double), lds)) return e;
  }
  hipLaunchKernelGGL((block_linears_kernel<R, NIT>), dim3((N + 16 * BL_TILES - 1) / (16 * BL_TILES), (B + R - 1) / R, n), dim3(256), smem, st, w, x,
                     y, block_stride, B, N, K);
  return hipGetLastError();
}

template <int R>
static hipError_t launch_block_linears_rows(const BlockLinears &w, int n, const float *x, float *y, size_t block_stride, int B, int N, int K,
                                            hipStream_t st) {
  if (K <= 256) return launch_block_linears_as<R, 1>(w, n, x, y, block_stride, B, N, K, st);
  if (K <= 512) return launch_block_linears_as<R, 2>(w, n, x, y, block_stride, B, N, K, st);
  if (K <= 1280) return launch_block_linears_as<R, 5>(w, n, x, y, block_stride, B, N, K, st);
  return launch_block_linears_as<R, 8>(w, n, x, y, block_stride, B, N, K, st);
}

hipError_t launch_block_linears(const BlockLinears &w, int n, const float *x, float *y, size_t block_stride, int B, int N, int K,
                                hipStream_t st) {
  if (K % 4 || K > 2048 || n > BLOCK_LINEARS) return hipErrorInvalidValue;
  if (B <= 1) return launch_block_linears_rows<1>(w, n, x, y, block_stride, B, N, K, st);
  if (B <= 2) return launch_block_linears_rows<2>(w, n, x, y, block_stride, B, N, K, st);
  if (B <= 4) return launch_block_linears_rows<4>(w, n, x, y, block_stride, B, N, K, st);
  return launch_block_linears_rows<8>(w, n, x, y, block_stride, B, N, K, st);
}

// ----------------------------------------------------------- conditioning
// c[r, :] = te[r / B, :] + table[label of batch element r % B] (rows are (timestep slot, batch element)), and the codes of
// SiLU(c) for the adaLN site of L blocks: q[l, r, n].  te == nullptr: c is given and only the codes are formed; qp ==
// nullptr: no codes.
__global__ void cond_silu_kernel(const float *__restrict__ te, const float *__restrict__ table, const int32_t *__restrict__ labels,
                                 int n_labels, int null_label, int rows, int B, int D, float *__restrict__ c, int *__restrict__ flags,
                                 int L, const QParam *qp, int qp_stride, int8_t *__restrict__ q, size_t l_stride) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= rows * D) return;
  float cv;
  if (te) {
    const int r = i / D, n = i % D, w = r / B, b = r % B;
    int y = b < n_labels ? labels[b] : null_label;
    if (y < 0 || y > null_label) {                // the table has null_label + 1 rows: clamp, and tell the host
      if (n == 0) atomicOr(flags, 1);
      y = min(max(y, 0), null_label);
    }
    cv = te[(size_t)w * D + n] + table[(size_t)y * D + n];
    c[i] = cv;
  } else {
    cv = c[i];
  }
  if (!qp) return;
  const float v = (float)silu_d((double)cv);      // float64 value rounded once, then Eq. 1
  for (int l = 0; l < L; ++l) {
    QParam t = qp[(size_t)l * qp_stride];
    q[(size_t)l * l_stride + i] = (int8_t)quant_code(v, t.s, t.z);
  }
}

hipError_t launch_cond_silu(const float *te, const float *table, const int32_t *labels, int n_labels, int null_label, int rows, int B,
                            int D, float *c, int *flags, int L, const QParam *qp, int qp_stride, int8_t *q, size_t l_stride,
                            hipStream_t st) {
  hipLaunchKernelGGL(cond_silu_kernel, dim3((rows * D + 255) / 256), dim3(256), 0, st, te, table, labels, n_labels, null_label, rows, B,
                     D, c, flags, L, qp, qp_stride, q, l_stride);
  return hipGetLastError();
}

// --------------------------------------------------------- patch embedding
// tok[b, t, n] = sum_f pw[n, f] * patch(b, t)[f] + pb[n] + pos[t, n], features f = (c, ph, pw).
// A thread owns four adjacent outputs n and keeps their F = 16 weights each in registers (as float64) over TPW consecutive
// tokens, so a workgroup writes whole token rows (16 bytes per thread) and reads the weights once per TPW tokens; one token
// per workgroup re-read 74 KB of weights for every 4.6 KB written (177 us at 32768 tokens of 1152, now 90).
// Float64 dot products in ascending f, rounded once when the token is stored.
template <int TPW>
__device__ __forceinline__ void embed16_tile(double (*patch)[16], int block, const float *__restrict__ x, const float *__restrict__ pw,
                                             const float *__restrict__ pb, const float *__restrict__ pos, void *__restrict__ tok, int tok_bf16,
                                             int n_src, int C, int H, int W, int p, int D, int b_off, int M) {
  constexpr int F = 16;
  const int gw = W / p, T = (H / p) * gw, m0 = block * TPW;
  for (int i = threadIdx.x; i < TPW * F; i += blockDim.x) {
    const int m = min(m0 + i / F, M - 1), f = i % F, b = m / T, t = m % T;
    const int c = f / (p * p), ph = (f / p) % p, pq = f % p;
    patch[i / F][f] = (double)x[(((size_t)((b + b_off) % n_src) * C + c) * H + (t / gw) * p + ph) * W + (t % gw) * p + pq];
  }
  const int n = threadIdx.x * 4;
  const bool live = n < D;
  const int nc = live ? n : 0;
  double w[4][F], bn[4];
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    bn[j] = (double)pb[nc + j];
#pragma unroll
    for (int f = 0; f < F; f += 4) {
      const float4 t4 = *(const float4 *)(pw + (size_t)(nc + j) * F + f);
      w[j][f] = t4.x; w[j][f + 1] = t4.y; w[j][f + 2] = t4.z; w[j][f + 3] = t4.w;
    }
  }
  __syncthreads();
  if (!live) return;
  float4 ps = *(const float4 *)(pos + (size_t)(m0 % T) * D + n);
#pragma unroll 1
  for (int k = 0; k < TPW; ++k) {
    const int m = m0 + k;
    if (m >= M) break;
    const float4 ps_next = *(const float4 *)(pos + (size_t)((m + 1) % T) * D + n);       // arrives behind this token's products
    double acc[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int f = 0; f < F; ++f) {
      const double pv = patch[k][f];
#pragma unroll
      for (int j = 0; j < 4; ++j) acc[j] = fma(w[j][f], pv, acc[j]);
    }
    stream_store4(tok, ((size_t)m * D + n) >> 2,
                  make_float4((float)((acc[0] + bn[0]) + (double)ps.x), (float)((acc[1] + bn[1]) + (double)ps.y),
                              (float)((acc[2] + bn[2]) + (double)ps.z), (float)((acc[3] + bn[3]) + (double)ps.w)), tok_bf16);
    ps = ps_next;
  }
}

template <int TPW>
__global__ __launch_bounds__(512) void embed16_kernel(const float *__restrict__ x, const float *__restrict__ pw, const float *__restrict__ pb,
                                                      const float *__restrict__ pos, void *__restrict__ tok, int tok_bf16, int n_src, int C,
                                                      int H, int W, int p, int D, int b_off, int M) {
  __shared__ double patch[TPW][16];
  embed16_tile<TPW>(patch, blockIdx.x, x, pw, pb, pos, tok, tok_bf16, n_src, C, H, W, p, D, b_off, M);
}

// Any other number of patch features: one token per workgroup.
__global__ __launch_bounds__(256) void embed_kernel(const float *__restrict__ x, const float *__restrict__ pw,
                                                    const float *__restrict__ pb, const float *__restrict__ pos,
                                                    void *__restrict__ tok, int tok_bf16, int n_src, int C, int H, int W, int p,
                                                    int D, int b_off) {
  __shared__ float patch[256];
  const int gw = W / p, T = (H / p) * gw;
  const int bt = blockIdx.x, b = bt / T, t = bt % T;
  const int F = C * p * p;
  const int ty = t / gw, tx = t % gw;
  const float *src = x + (size_t)((b + b_off) % n_src) * C * H * W;
  for (int f = threadIdx.x; f < F; f += blockDim.x) {
    const int c = f / (p * p), ph = (f / p) % p, pq = f % p;
    patch[f] = src[((size_t)c * H + ty * p + ph) * W + tx * p + pq];
  }
  __syncthreads();
  for (int n = threadIdx.x; n < D; n += blockDim.x) {
    // float64 dot product, rounded once when the token is stored
    double acc = 0.0;
    const float *wr = pw + (size_t)n * F;
    if (F % 4 == 0) {
      for (int f0 = 0; f0 < F; f0 += 16) {
        float4 w4[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) w4[u] = *(const float4 *)(wr + min(f0 + 4 * u, F - 4));
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          const int f = f0 + 4 * u;
          if (f < F) {
            acc = fma((double)w4[u].x, (double)patch[f], acc);
            acc = fma((double)w4[u].y, (double)patch[f + 1], acc);
            acc = fma((double)w4[u].z, (double)patch[f + 2], acc);
            acc = fma((double)w4[u].w, (double)patch[f + 3], acc);
          }
        }
      }
    } else {
      for (int f = 0; f < F; ++f) acc = fma((double)wr[f], (double)patch[f], acc);
    }
    stream_store(tok, (size_t)bt * D + n, (float)((acc + (double)pb[n]) + (double)pos[(size_t)t * D + n]), tok_bf16);
  }
}

hipError_t launch_embed(const float *x, const float *pw, const float *pb, const float *pos, void *tok, int tok_bf16, int B,
                        int n_src, int C, int H, int W, int p, int D, int b_off, hipStream_t st) {
  const int T = (H / p) * (W / p), M = B * T;
  if (C * p * p == 16 && D % 4 == 0 && D <= 2048) {
    // tokens per workgroup: as many as leave two workgroups per compute unit
    const int threads = (D / 4 + 63) / 64 * 64;
#define QC_EMBED(TPW) hipLaunchKernelGGL(embed16_kernel<TPW>, dim3((M + TPW - 1) / TPW), dim3(threads), 0, st, x, pw, pb, pos, tok, tok_bf16, n_src, C, H, W, p, D, b_off, M)
    if (M >= 32 * 512) QC_EMBED(32);
    else if (M >= 8 * 512) QC_EMBED(8);
    else if (M >= 4 * 512) QC_EMBED(4);
    else if (M >= 2 * 512) QC_EMBED(2);
    else QC_EMBED(1);
#undef QC_EMBED
    return hipGetLastError();
  }
  hipLaunchKernelGGL(embed_kernel, dim3(B * T), dim3(256), 0, st, x, pw, pb, pos, tok, tok_bf16, n_src, C, H, W, p, D, b_off);
  return hipGetLastError();
}

// ------------------------------------------------- conditioning of one step, few rows
// A caller that drives the sampler step by step has one timestep and a few latents a call, and every launch in front of the
// first block is as short as launches get (4.4 us, one after the other).  So what does not depend on each other shares a launch:
//   step_time_kernel   hidden layer of the timestep MLP | patch embedding of all tokens
//   step_cond_kernel   its output layer, with the label's row added, and the codes of SiLU(c) for every block
//   step_mod_kernel    adaLN projections of all blocks | modulation of the final layer
// instead of six.  DiT-S/2 block, 1 latent, a refreshed and a cached step: 24 launches, 104 us -> 18, 86 us.  Each part's
// arithmetic is that of its kernel of many rows.
constexpr int STEP_ROWS = 8;                      // rows of conditioning at most

template <int TPW>
__global__ __launch_bounds__(512) void step_time_kernel(int nb_time, int t, const float *__restrict__ w1, const float *__restrict__ b1, float *__restrict__ h1,
                                                        int K, const float *__restrict__ x, const float *__restrict__ pw,
                                                        const float *__restrict__ pb, const float *__restrict__ pos, void *__restrict__ tok,
                                                        int tok_bf16, int n_src, int C, int H, int W, int p, int D, int M) {
  __shared__ double xs[256];
  __shared__ double patch[TPW][16];
  if ((int)blockIdx.x < nb_time) {
    if (threadIdx.x >= 256) return;               // whole wavefronts
    small_linear_tile<1, 1>(xs, blockIdx.x, 0, nullptr, 0, t, 0, w1, b1, 1, D, K, 0, 1, [&](int, int n, float v) { h1[n] = v; });
  } else {
    embed16_tile<TPW>(patch, blockIdx.x - nb_time, x, pw, pb, pos, tok, tok_bf16, n_src, C, H, W, p, D, 0, M);
  }
}

// one workgroup = 16 features of every row
template <int NIT>
__global__ __launch_bounds__(256) void step_cond_kernel(const float *__restrict__ h1, const float *__restrict__ w2, const float *__restrict__ b2,
                                                        const float *__restrict__ table, const int32_t *__restrict__ labels, int n_labels,
                                                        int null_label, int B, int D, float *__restrict__ c, int *__restrict__ flags, int L,
                                                        const QParam *qp, int qp_stride, int8_t *__restrict__ q, size_t l_stride) {
  extern __shared__ double xs[];                  // [D]
  __shared__ float te[16], vs[STEP_ROWS][16];
  const int n0 = blockIdx.x * 16;
  small_linear_tile<1, NIT>(xs, blockIdx.x, 0, h1, D, 0, 0, w2, b2, 1, D, D, 0, 0, [&](int, int n, float v) { te[n - n0] = v; });
  __syncthreads();
  if ((int)threadIdx.x < 16 * B) {
    const int b = threadIdx.x >> 4, j = threadIdx.x & 15;
    int y = b < n_labels ? labels[b] : null_label;
    if (y < 0 || y > null_label) {                // as in cond_silu_kernel
      if (n0 + j == 0) atomicOr(flags, 1);
      y = min(max(y, 0), null_label);
    }
    const float cv = te[j] + table[(size_t)y * D + n0 + j];
    c[(size_t)b * D + n0 + j] = cv;
    vs[b][j] = (float)silu_d((double)cv);
  }
  __syncthreads();
  // four codes at a time: thread = (block and row, quarter of the 16 features)
  const int f = (threadIdx.x & 3) * 4;
  for (int i = threadIdx.x >> 2; i < L * B; i += 64) {
    const int l = i / B, b = i - l * B;
    const QParam t = qp[(size_t)l * qp_stride];
    const float *v = vs[b] + f;
    *(unsigned *)(q + (size_t)l * l_stride + (size_t)b * D + n0 + f) =
        pack4(quant_code(v[0], t.s, t.z), quant_code(v[1], t.s, t.z), quant_code(v[2], t.s, t.z), quant_code(v[3], t.s, t.z));
  }
}

// The adaLN part: a wavefront takes eight output columns at a time, eight lanes each, 16 bytes of codes per lane and load (whole
// cache lines of a weight row), four-product integer dot instructions, and the eight lanes' sums meet in DPP moves.  One pass over
// the weights whatever the number of rows, bound by their bytes (223 MB for the 28 blocks of DiT-XL/2, a third of that in a cached step):
// with all three kernels a refreshed step of 1 latent of 256 tokens takes 1643 -> 1620 us, a cached one 79 -> 59; 8 latents of 16
// tokens cached 91 -> 72.  R rows at once there, RF at once in the final layer's part (whose inputs lie in LDS as
// float64); NI: loads of 128 bytes a weight row.
template <int R, int RF, int NIT, int NI, bool W4>
__global__ __launch_bounds__(256) void step_mod_kernel(int nb_final, const float *__restrict__ cond, const float *__restrict__ fw,
                                                       const float *__restrict__ fb, float *__restrict__ fmod, int B, int D, int nb_ada, GemmArgs p) {
  extern __shared__ double xs[];                  // [RF][D]
  if ((int)blockIdx.x < nb_final) {
    const int tiles = (2 * D + 15) / 16, by = blockIdx.x / tiles;
    small_linear_tile<RF, NIT>(xs, blockIdx.x - by * tiles, by, cond, D, 0, 0, fw, fb, B, 2 * D, D, 1, 0,
                              [&](int b, int n, float v) { fmod[(size_t)b * 2 * D + n] = v; });
    return;
  }
  const int bi = blockIdx.x - nb_final, z = bi / nb_ada, lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int ncover = p.sel_D ? 2 * p.sel_D : p.N;
  const int j = (bi - z * nb_ada) * 32 + wave * 8 + (lane >> 3), c = lane & 7;
  const int n = map_col(min(j, ncover - 1), p.sel_D);
  const unsigned char *w = (const unsigned char *)p.W + (size_t)z * p.zs_W + (size_t)n * (W4 ? p.K >> 1 : p.K);
  const int8_t *act = p.A + (size_t)z * p.zs_A;
  typedef typename std::conditional<W4, v2i, v4i>::type wload_t;
  wload_t wv[NI];
#pragma unroll
  for (int i = 0; i < NI; ++i) {
    const int k = min((8 * i + c) * 16, p.K - 16);
    wv[i] = *(const wload_t *)(w + (W4 ? k >> 1 : k));
  }
  int acc[R];
#pragma unroll
  for (int r = 0; r < R; ++r) acc[r] = 0;
#pragma unroll
  for (int i = 0; i < NI; ++i) {
    v4i v;
    if constexpr (W4) v = unpack_w4(wv[i]);
    else v = wv[i];
    const int k = (8 * i + c) * 16;
    if (k >= p.K) v = (v4i){0, 0, 0, 0};
#pragma unroll
    for (int r = 0; r < R; ++r) {
      const v4i x = *(const v4i *)(act + (size_t)min(r, B - 1) * p.lda + min(k, p.K - 16));
#pragma unroll
      for (int e = 0; e < 4; ++e) acc[r] = __builtin_amdgcn_sdot4(x[e], v[e], acc[r], false);
    }
  }
  // the eight lanes of a column: neighbours, the other pair, the other quad of the half row
  int sum = 0;
#pragma unroll
  for (int r = 0; r < R; ++r) {
    int a = acc[r];
    a += __builtin_amdgcn_update_dpp(0, a, 0xB1, 0xF, 0xF, false);
    a += __builtin_amdgcn_update_dpp(0, a, 0x4E, 0xF, 0xF, false);
    a += __builtin_amdgcn_update_dpp(0, a, 0x141, 0xF, 0xF, false);
    if (c == r) sum = a;
  }
  if (c >= B || j >= ncover) return;              // lane c finishes row c
  const QParam q = p.a_qp[(size_t)z * p.zs_qp];
  const size_t at = (size_t)z * p.zs_vecN + n;
  const double sc = (double)q.s * (double)p.w_scale[at];
  p.y[(size_t)z * p.zs_out + (size_t)c * p.ldy + n] = dequant_f32(sc, sum - q.z * p.wsum[at], p.bias ? (double)p.bias[at] : 0.0);
}

// Whether the three kernels cover a call: one timestep, a few rows, and few enough tokens that embedding them takes no longer than the
// linear beside it: the gain ends there (two blocks, a refreshed | a cached step in six launches -> three: 1 latent of 1024 tokens, width 384
// 150 -> 140 | 34 -> 25 us, 1152 266 -> 256 | 53 -> 43; of 2048 tokens, width 384 274 -> 265 | 37 -> 28, 1152 503 -> 498 | 58 -> 54, 2048 775 -> 777 | 82 -> 78).
bool step_cond_covers(int B, int freq_dim, int C, int p, int D, int M) {
  return B <= STEP_ROWS && freq_dim <= 256 && freq_dim % 4 == 0 && C * p * p == 16 && D <= 2048 && M <= 2048;
}

hipError_t launch_step_time(int t, const float *w1, const float *b1, float *h1, int freq_dim, const EmbedSrc &e, void *tok, int tok_bf16, int B,
                            int D, hipStream_t st) {
  const int M = B * (e.H / e.p) * (e.W / e.p), nb_time = (D + 15) / 16;
  const int threads = std::max(256, (D / 4 + 63) / 64 * 64);
#define QC_STEP_TIME(TPW)                                                                                                                  \
  hipLaunchKernelGGL(step_time_kernel<TPW>, dim3(nb_time + (M + TPW - 1) / TPW), dim3(threads), 0, st, nb_time, t, w1, b1, h1, freq_dim, e.x, \
                     e.pw, e.pb, e.pos, tok, tok_bf16, e.n_src, e.C, e.H, e.W, e.p, D, M)
  if (M >= 2 * 512) QC_STEP_TIME(2);
  else QC_STEP_TIME(1);
#undef QC_STEP_TIME
  return hipGetLastError();
}

hipError_t launch_step_cond(const float *h1, const float *w2, const float *b2, const float *table, const int32_t *labels, int n_labels,
                            int null_label, int B, int D, float *c, int *flags, int L, const QParam *qp, int qp_stride, int8_t *q,
                            size_t l_stride, hipStream_t st) {
#define QC_STEP_COND(NIT)                                                                                                               \
  hipLaunchKernelGGL(step_cond_kernel<NIT>, dim3(D / 16), dim3(256), (size_t)D * sizeof(double), st, h1, w2, b2, table, labels, n_labels, \
                     null_label, B, D, c, flags, L, qp, qp_stride, q, l_stride)
  if (D <= 256) QC_STEP_COND(1);
  else if (D <= 512) QC_STEP_COND(2);
  else if (D <= 1280) QC_STEP_COND(5);
  else QC_STEP_COND(8);
#undef QC_STEP_COND
  return hipGetLastError();
}

template <int R, int RF, int NIT, int NI>
static hipError_t launch_step_mod_as(const float *cond, const float *fw, const float *fb, float *fmod, int B, int D, const GemmArgs &a, int nz,
                                     hipStream_t st) {
  const int nb_final = (2 * D + 15) / 16 * ((B + RF - 1) / RF), nb_ada = ((a.sel_D ? 2 * a.sel_D : a.N) + 31) / 32;
  const dim3 grid(nb_final + nb_ada * nz);
  const size_t smem = (size_t)RF * D * sizeof(double);           // 64 KB at most
  if (a.w4) hipLaunchKernelGGL((step_mod_kernel<R, RF, NIT, NI, true>), grid, dim3(256), smem, st, nb_final, cond, fw, fb, fmod, B, D, nb_ada, a);
  else hipLaunchKernelGGL((step_mod_kernel<R, RF, NIT, NI, false>), grid, dim3(256), smem, st, nb_final, cond, fw, fb, fmod, B, D, nb_ada, a);
  return hipGetLastError();
}

template <int R, int RF>
static hipError_t launch_step_mod_rows(const float *cond, const float *fw, const float *fb, float *fmod, int B, int D, const GemmArgs &a, int nz,
                                       hipStream_t st) {
  if (D <= 256) return launch_step_mod_as<R, RF, 1, 2>(cond, fw, fb, fmod, B, D, a, nz, st);
  if (D <= 512) return launch_step_mod_as<R, RF, 2, 4>(cond, fw, fb, fmod, B, D, a, nz, st);
  if (D <= 1280) return launch_step_mod_as<R, RF, 5, 10>(cond, fw, fb, fmod, B, D, a, nz, st);
  return launch_step_mod_as<R, RF, 8, 16>(cond, fw, fb, fmod, B, D, a, nz, st);
}

hipError_t launch_step_mod(const float *cond, const float *fw, const float *fb, float *fmod, int B, int D, const GemmArgs &a, int nz,
                           hipStream_t st) {
  if (B <= 1) return launch_step_mod_rows<1, 1>(cond, fw, fb, fmod, B, D, a, nz, st);
  if (B <= 2) return launch_step_mod_rows<2, 2>(cond, fw, fb, fmod, B, D, a, nz, st);
  if (B <= 4) return launch_step_mod_rows<4, 4>(cond, fw, fb, fmod, B, D, a, nz, st);
  return launch_step_mod_rows<8, 4>(cond, fw, fb, fmod, B, D, a, nz, st);
}

// ---------------------------------------------------------------- final layer
// Per token: LayerNorm, modulate with (shift, scale) = fmod[b, 0:D], fmod[b, D:2D],
// dot with the rows of the output linear that belong to the first C of the 2C
// channels, and scatter to eps[b, c, ty*p+ph, tx*p+pw] (output features (ph, pw, c)).
// Float64 throughout, rounded once when the noise estimate is stored; the dot products run on the float64 matrix cores.
// One workgroup = 16 tokens, its eight wavefronts share the features: 16-feature chunk c belongs to wavefront c % 8, lane l
// holds features 4 (l / 16) .. + 3 of it for token l % 16 (and, as the other operand, for output l % 16), so a chunk is four
// 16x16x4 products and a row is read from memory once, into registers.  The row sums and the partial products of the
// wavefronts meet in LDS.  Bound: the token tensor's bytes (32768 tokens of 1152: 151 MB) and the load instructions; with one
// wavefront per token, which fetched all 74 KB of weights for its 4.6 KB, 247 us; now 92.
typedef double d4v __attribute__((ext_vector_type(4)));

constexpr int FW = 8;  // wavefronts
template <int NJ>      // chunks a wavefront holds (D <= 16 FW NJ)
__global__ __launch_bounds__(64 * FW, NJ < 9 ? 4 : 2) void final_kernel(const void *__restrict__ tok, int tok_bf16, const float *__restrict__ fmod,
                                                       const float *__restrict__ fw, const float *__restrict__ fb,
                                                       float *__restrict__ eps, int M, int C, int H, int W, int p, int D) {
  __shared__ double red[2][FW][16];
  __shared__ double prod[FW][16][17];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, row = lane & 15, g = lane >> 4;
  const int gw = W / p, T = (H / p) * gw, m0 = blockIdx.x * 16;
  const int m = min(m0 + row, M - 1);             // rows beyond M repeat the last (not stored)
  const float *sh = fmod + (size_t)(m / T) * 2 * D, *sc = sh + D;
  // loads never branch: features beyond D re-read the row's end and are zeroed
  float4 v[NJ];
#pragma unroll
  for (int j = 0; j < NJ; ++j) v[j] = stream_load4(tok, ((size_t)m * D + min((j * FW + wave) * 16 + 4 * g, D - 4)) >> 2, tok_bf16);
  double sum = 0.0;
#pragma unroll
  for (int j = 0; j < NJ; ++j)
    if ((j * FW + wave) * 16 + 4 * g < D) sum += ((double)v[j].x + (double)v[j].y) + ((double)v[j].z + (double)v[j].w);
  sum += __shfl_xor(sum, 16, 64);
  sum += __shfl_xor(sum, 32, 64);
  if (g == 0) red[0][wave][row] = sum;
  __syncthreads();
  double mu = 0.0, var = 0.0;
#pragma unroll
  for (int w = 0; w < FW; ++w) mu += red[0][w][row];
  mu /= (double)D;
  double sq = 0.0;
#pragma unroll
  for (int j = 0; j < NJ; ++j)
    if ((j * FW + wave) * 16 + 4 * g < D) {
      const double a = v[j].x - mu, b = v[j].y - mu, c = v[j].z - mu, d = v[j].w - mu;
      sq += (a * a + b * b) + (c * c + d * d);
    }
  sq += __shfl_xor(sq, 16, 64);
  sq += __shfl_xor(sq, 32, 64);
  if (g == 0) red[1][wave][row] = sq;
  __syncthreads();
#pragma unroll
  for (int w = 0; w < FW; ++w) var += red[1][w][row];
  double rstd = 1.0 / sqrt(var / (double)D + 1e-6);
  const int n_out = p * p * C;
  int zero = 0;
  for (int o0 = 0; o0 < n_out; o0 += 16) {
    const int oi = min(o0 + row, n_out - 1);      // outputs beyond the last repeat it (not stored)
    const float *wr = fw + (size_t)((oi / C) * 2 * C + oi % C) * D;
    d4v acc = {0.0, 0.0, 0.0, 0.0};
    asm volatile("" : "+v"(mu), "+v"(rstd), "+v"(zero));      // keeps the row's float64 values out of registers between passes
#pragma unroll
    for (int j = 0; j < NJ; ++j) {
      const int k = (j * FW + wave) * 16 + 4 * g, kc = min(k, D - 4) + zero;
      const float4 s4 = *(const float4 *)(sh + kc), c4 = *(const float4 *)(sc + kc), w4 = *(const float4 *)(wr + kc);
      const bool in = k < D;
      const double h0 = in ? (v[j].x - mu) * rstd * (1.0 + (double)c4.x) + (double)s4.x : 0.0;
      const double h1 = in ? (v[j].y - mu) * rstd * (1.0 + (double)c4.y) + (double)s4.y : 0.0;
      const double h2 = in ? (v[j].z - mu) * rstd * (1.0 + (double)c4.z) + (double)s4.z : 0.0;
      const double h3 = in ? (v[j].w - mu) * rstd * (1.0 + (double)c4.w) + (double)s4.w : 0.0;
      acc = __builtin_amdgcn_mfma_f64_16x16x4f64(h0, (double)w4.x, acc, 0, 0, 0);
      acc = __builtin_amdgcn_mfma_f64_16x16x4f64(h1, (double)w4.y, acc, 0, 0, 0);
      acc = __builtin_amdgcn_mfma_f64_16x16x4f64(h2, (double)w4.z, acc, 0, 0, 0);
      acc = __builtin_amdgcn_mfma_f64_16x16x4f64(h3, (double)w4.w, acc, 0, 0, 0);
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) prod[wave][g + 4 * i][row] = acc[i];      // lane l: tokens l / 16 + 4 i, output l % 16
    __syncthreads();
    const int tk = threadIdx.x & 15, u = threadIdx.x >> 4, o = o0 + u, mt = m0 + tk;
    if (u < 16 && mt < M && o < n_out) {
      const int pp = o / C, c = o % C, b = mt / T, t = mt % T, ty = t / gw, tx = t % gw;
      double r = 0.0;
#pragma unroll
      for (int w = 0; w < FW; ++w) r += prod[w][tk][u];
      eps[(((size_t)b * C + c) * H + ty * p + pp / p) * W + tx * p + pp % p] = (float)(r + (double)fb[pp * 2 * C + c]);
    }
    __syncthreads();
  }
}

hipError_t launch_final(const void *tok, int tok_bf16, const float *fmod, const float *fw, const float *fb, float *eps, int B,
                        int C, int H, int W, int p, int D, hipStream_t st) {
  const int M = B * (H / p) * (W / p);
  const dim3 grid((M + 15) / 16);
#define QC_FINAL(NJ) hipLaunchKernelGGL(final_kernel<NJ>, grid, dim3(64 * FW), 0, st, tok, tok_bf16, fmod, fw, fb, eps, M, C, H, W, p, D)
  if (D <= 16 * FW * 3) QC_FINAL(3);
  else if (D <= 16 * FW * 6) QC_FINAL(6);
  else if (D <= 16 * FW * 9) QC_FINAL(9);
  else QC_FINAL(16);
#undef QC_FINAL
  return hipGetLastError();
}

// ---------------------------------------------------------------- cache ops
// The cached tensors are stored as fp32 or, in the reduced-precision variant, as bfloat16; so is the residual stream.

template <bool BF16>
__device__ __forceinline__ float4 load_cached4(const void *base, size_t i4) {
  if (BF16) {
    const uint2 r = ((const uint2 *)base)[i4];       // four bfloat16
    return make_float4(__builtin_bit_cast(float, r.x << 16), __builtin_bit_cast(float, r.x & 0xFFFF0000u),
                       __builtin_bit_cast(float, r.y << 16), __builtin_bit_cast(float, r.y & 0xFFFF0000u));
  }
  return ((const float4 *)base)[i4];
}

template <bool BF16>
__global__ __launch_bounds__(256) void cache_store_kernel(const float4 *__restrict__ s, void *__restrict__ d, size_t n4) {
  const size_t stride = (size_t)gridDim.x * blockDim.x;
  for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n4; i += stride) {
    const float4 v = s[i];
    if (BF16) {
      uint2 r;
      r.x = (unsigned)bf16_bits(v.x) | ((unsigned)bf16_bits(v.y) << 16);
      r.y = (unsigned)bf16_bits(v.z) | ((unsigned)bf16_bits(v.w) << 16);
      ((uint2 *)d)[i] = r;
    } else {
      ((float4 *)d)[i] = v;
    }
  }
}

hipError_t launch_cache_store(const float *src, void *dst, size_t n, bool bf16, hipStream_t st) {
  size_t n4 = n / 4, blocks = (n4 + 255) / 256;
  if (blocks > 16384) blocks = 16384;
  if (blocks == 0) return hipSuccess;
  if (bf16) hipLaunchKernelGGL(cache_store_kernel<true>, dim3((unsigned)blocks), dim3(256), 0, st, (const float4 *)src, dst, n4);
  else hipLaunchKernelGGL(cache_store_kernel<false>, dim3((unsigned)blocks), dim3(256), 0, st, (const float4 *)src, dst, n4);
  return hipGetLastError();
}

// x[b, t, :] += gate[b, :] * cached[b, t, :]
template <bool BF16>
__global__ __launch_bounds__(256) void cache_reuse_kernel(void *__restrict__ x, int x_bf16, const void *__restrict__ cached,
                                                          const float *__restrict__ gate, int ld_gate, size_t n4, int TD4,
                                                          int D4) {
  const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n4) return;
  const int b = (int)(i / TD4), n = (int)(i % D4) * 4;
  float4 xv = stream_load4(x, i, x_bf16);
  const float4 cv = load_cached4<BF16>(cached, i);
  float4 g = *(const float4 *)(gate + (size_t)b * ld_gate + n);
  xv.x = xv.x + g.x * cv.x;
  xv.y = xv.y + g.y * cv.y;
  xv.z = xv.z + g.z * cv.z;
  xv.w = xv.w + g.w * cv.w;
  stream_store4(x, i, xv, x_bf16);
}

hipError_t launch_cache_reuse(void *x, int x_bf16, const void *cached, const float *gate, int ld_gate, int B, int T, int D,
                              bool bf16, hipStream_t st) {
  const size_t n4 = (size_t)B * T * D / 4;
  const dim3 grid((unsigned)((n4 + 255) / 256));
  if (bf16) hipLaunchKernelGGL(cache_reuse_kernel<true>, grid, dim3(256), 0, st, x, x_bf16, cached, gate, ld_gate, n4, T * D / 4, D / 4);
  else hipLaunchKernelGGL(cache_reuse_kernel<false>, grid, dim3(256), 0, st, x, x_bf16, cached, gate, ld_gate, n4, T * D / 4, D / 4);
  return hipGetLastError();
}

// All blocks of a cached step in one pass over x: for every block in order,
// x += gate_msa * attn_cached; x += gate_mlp * mlp_cached (same association
// as block after block; a bfloat16 stream is rounded to its storage format after every addition, as it would be if
// it went through memory).  mod[l, b, 6D] holds the gates in chunks 2 and 5.  Cache strides are in elements.
__device__ __forceinline__ float as_stored(float v, int bf) { return bf ? bf16_value(bf16_bits(v)) : v; }

template <bool BF16>
__global__ __launch_bounds__(256) void cached_blocks_kernel(void *__restrict__ x, int x_bf16, const void *__restrict__ cache,
                                                            size_t cache_block_stride, size_t cache_which_stride,
                                                            const float *__restrict__ mod, size_t mod_block_stride,
                                                            int ld_mod, int L, size_t n4, int TD4, int D4, int D) {
  const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n4) return;
  const int b = (int)(i / TD4), n = (int)(i % D4) * 4;
  constexpr size_t ES = BF16 ? 2 : 4;               // bytes per cached element
  const char *cbase = (const char *)cache;
  float4 xv = stream_load4(x, i, x_bf16);
  auto apply = [&](const float4 &g1, const float4 &a, const float4 &g2, const float4 &mo) {
    xv.x = as_stored(xv.x + g1.x * a.x, x_bf16); xv.y = as_stored(xv.y + g1.y * a.y, x_bf16);
    xv.z = as_stored(xv.z + g1.z * a.z, x_bf16); xv.w = as_stored(xv.w + g1.w * a.w, x_bf16);
    xv.x = as_stored(xv.x + g2.x * mo.x, x_bf16); xv.y = as_stored(xv.y + g2.y * mo.y, x_bf16);
    xv.z = as_stored(xv.z + g2.z * mo.z, x_bf16); xv.w = as_stored(xv.w + g2.w * mo.w, x_bf16);
  };
  // the loads of four blocks are in flight together; the additions keep the block order
  constexpr int U = 4;
  int l = 0;
  for (; l + U <= L; l += U) {
    float4 g1[U], g2[U], a[U], mo[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const float *mrow = mod + (size_t)(l + u) * mod_block_stride + (size_t)b * ld_mod + n;
      g1[u] = *(const float4 *)(mrow + 2 * D);
      g2[u] = *(const float4 *)(mrow + 5 * D);
      a[u] = load_cached4<BF16>(cbase + (size_t)(l + u) * cache_block_stride * ES, i);
      mo[u] = load_cached4<BF16>(cbase + ((size_t)(l + u) * cache_block_stride + cache_which_stride) * ES, i);
    }
#pragma unroll
    for (int u = 0; u < U; ++u) apply(g1[u], a[u], g2[u], mo[u]);
  }
  for (; l < L; ++l) {
    const float *mrow = mod + (size_t)l * mod_block_stride + (size_t)b * ld_mod + n;
    const float4 g1 = *(const float4 *)(mrow + 2 * D), g2 = *(const float4 *)(mrow + 5 * D);
    const float4 a = load_cached4<BF16>(cbase + (size_t)l * cache_block_stride * ES, i);
    const float4 mo = load_cached4<BF16>(cbase + ((size_t)l * cache_block_stride + cache_which_stride) * ES, i);
    apply(g1, a, g2, mo);
  }
  stream_store4(x, i, xv, x_bf16);
}

hipError_t launch_cached_blocks(void *x, int x_bf16, const void *cache, size_t cache_block_stride, size_t cache_which_stride,
                                const float *mod, size_t mod_block_stride, int ld_mod, int L, int B, int T, int D, bool bf16,
                                hipStream_t st) {
  const size_t n4 = (size_t)B * T * D / 4;
  const dim3 grid((unsigned)((n4 + 255) / 256));
  if (bf16)
    hipLaunchKernelGGL(cached_blocks_kernel<true>, grid, dim3(256), 0, st, x, x_bf16, cache, cache_block_stride, cache_which_stride, mod,
                       mod_block_stride, ld_mod, L, n4, T * D / 4, D / 4, D);
  else
    hipLaunchKernelGGL(cached_blocks_kernel<false>, grid, dim3(256), 0, st, x, x_bf16, cache, cache_block_stride, cache_which_stride, mod,
                       mod_block_stride, ld_mod, L, n4, T * D / 4, D / 4, D);
  return hipGetLastError();
}

// ------------------------------------------------- DDIM update + guidance + VC
__device__ __forceinline__ float block_sum_256(float v, float *red) {
  v = wave_sum(v);
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  __syncthreads();
  if (lane == 0) red[w] = v;
  __syncthreads();
  return (red[0] + red[1]) + (red[2] + red[3]);
}

// One workgroup per (latent, channel) plane.  xhat = cx*x + ce*eps is DDIM with
// eta = 0 (cx = sqrt(abar_prev/abar_t), ce = sqrt(1-abar_prev) - cx*sqrt(1-abar_t));
// then Eq. 10 with mu = plane mean: x~ = xhat + (K-1)(xhat - mu).  Both the updated sample and the corrected sample are
// stored float32 tensors; guidance + solver update, and VC, are each evaluated in float64 from the stored tensors they
// read and rounded once (the same values the separate DDIM, fit and VC launches of the factor fitting produce).
__device__ __forceinline__ double block_sum_256d(double v, double *red) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  __syncthreads();                       // red may still be read from the previous use
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
  __syncthreads();
  return (red[0] + red[1]) + (red[2] + red[3]);
}

__global__ __launch_bounds__(256) void ddim_vc_kernel(float *__restrict__ x, const float *__restrict__ eps, int B, int C,
                                                      int HW, double cx, double ce, float cfg, const float *__restrict__ K_t) {
  __shared__ double red[4];
  const int plane = blockIdx.x, c = plane % C;
  float *xp = x + (size_t)plane * HW;
  const float *ec = eps + (size_t)plane * HW;
  const float *eu = eps + ((size_t)B * C + plane) * HW;
  const double w = (double)cfg;
  double sum = 0.0;
  for (int i = threadIdx.x; i < HW; i += 256) {
    double e = (double)ec[i];
    if (cfg > 0.0f) {
      const double u = (double)eu[i];
      e = u + w * (e - u);
    }
    const float xh = (float)(cx * (double)xp[i] + ce * e);
    xp[i] = xh;
    sum += (double)xh;
  }
  if (!K_t) return;
  const double mu = block_sum_256d(sum, red) / (double)HW;
  const double km1 = (double)K_t[c] - 1.0;
  for (int i = threadIdx.x; i < HW; i += 256) {          // a thread re-reads only what it wrote itself
    const double xh = (double)xp[i];
    xp[i] = (float)(xh + km1 * (xh - mu));
  }
}

hipError_t launch_ddim_vc(float *x, const float *eps, int B, int C, int HW, double cx, double ce, float cfg_scale,
                          const float *K_t, hipStream_t st) {
  hipLaunchKernelGGL(ddim_vc_kernel, dim3(B * C), dim3(256), 0, st, x, eps, B, C, HW, cx, ce, cfg_scale, K_t);
  return hipGetLastError();
}

__global__ __launch_bounds__(256) void vc_kernel(float *__restrict__ x, const float *__restrict__ K_t,
                                                 const float *__restrict__ mu_in, int C, int HW) {
  __shared__ double red[4];
  const int plane = blockIdx.x, c = plane % C;
  float *xp = x + (size_t)plane * HW;
  double mu;
  if (mu_in) {
    mu = (double)mu_in[c];
  } else {
    double sum = 0.0;
    for (int i = threadIdx.x; i < HW; i += 256) sum += (double)xp[i];
    mu = block_sum_256d(sum, red) / (double)HW;
  }
  const double km1 = (double)K_t[c] - 1.0;
  for (int i = threadIdx.x; i < HW; i += 256) {
    const double v = (double)xp[i];
    xp[i] = (float)(v + km1 * (v - mu));
  }
}

hipError_t launch_vc(float *x, const float *K_t, const float *mu, int B, int C, int HW, hipStream_t st) {
  hipLaunchKernelGGL(vc_kernel, dim3(B * C), dim3(256), 0, st, x, K_t, mu, C, HW);
  return hipGetLastError();
}

// ------------------------------------------------------------------ VC fit
// Factors of one timestep: the exact minimiser, channel by channel, of
//   sum ((x~ - x') / x')^2 + sum (x~ - x')^2,   x~ = mu + K (x^ - mu)     (objective after Eq. 10)
// over the elements of the channel in the whole batch: K = S1 / S2 with S1 = sum d (x' - mu) w,
// S2 = sum d^2 w, d = x^ - mu, w = 1 + 1 / (x'^2 + eps), mu = spatial mean of the x^ plane.
// One workgroup per (sample, channel) plane writes its two partial sums (fp64); a second, tiny kernel adds the
// planes of a channel in a fixed order, so the result does not depend on scheduling.
__global__ __launch_bounds__(256) void vc_fit_sums_kernel(const float *__restrict__ x_hat, const float *__restrict__ x_ref,
                                                          int HW, double eps, double *__restrict__ part) {
  __shared__ double red[4];
  const int plane = blockIdx.x;
  const float *xh = x_hat + (size_t)plane * HW, *xr = x_ref + (size_t)plane * HW;
  double sum = 0.0;
  for (int i = threadIdx.x; i < HW; i += 256) sum += (double)xh[i];
  const double mu = block_sum_256d(sum, red) / (double)HW;
  double s1 = 0.0, s2 = 0.0;
  for (int i = threadIdx.x; i < HW; i += 256) {
    const double d = (double)xh[i] - mu, r = (double)xr[i];
    const double w = 1.0 + 1.0 / (r * r + eps);
    s1 += d * (r - mu) * w;
    s2 += d * d * w;
  }
  s1 = block_sum_256d(s1, red);
  s2 = block_sum_256d(s2, red);
  if (threadIdx.x == 0) {
    part[2 * plane] = s1;
    part[2 * plane + 1] = s2;
  }
}

__global__ void vc_fit_solve_kernel(const double *__restrict__ part, int B, int C, float *__restrict__ K_t) {
  const int c = blockIdx.x * blockDim.x + threadIdx.x;
  if (c >= C) return;
  double s1 = 0.0, s2 = 0.0;
  for (int b = 0; b < B; ++b) {
    s1 += part[2 * ((size_t)b * C + c)];
    s2 += part[2 * ((size_t)b * C + c) + 1];
  }
  K_t[c] = s2 > 0.0 ? (float)(s1 / s2) : 1.0f;
}

hipError_t launch_vc_fit(const float *x_hat, const float *x_ref, int B, int C, int HW, float eps, double *work, float *K_t,
                         hipStream_t st) {
  hipLaunchKernelGGL(vc_fit_sums_kernel, dim3(B * C), dim3(256), 0, st, x_hat, x_ref, HW, (double)eps, work);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(vc_fit_solve_kernel, dim3((C + 63) / 64), dim3(64), 0, st, work, B, C, K_t);
  return hipGetLastError();
}

// ------------------------------------------------------ calibration helpers
// Running min / max of a tensor kept as order-preserving integers:
// slot[0] = min, slot[1] = max; act = 1 takes SiLU of the values first.
__device__ __forceinline__ int f2ord(float f) {
  int i = __float_as_int(f);
  return i ^ ((i >> 31) & 0x7FFFFFFF);
}
// One pair of atomics per workgroup and at most 256 workgroups: atomics on one address are carried out one after the other
// (8192 of them, one pair per wavefront of 1024 workgroups, took 77 us of a call's 77).
__global__ __launch_bounds__(256) void minmax_kernel(const float *__restrict__ x, size_t n, int act, int *slot) {
  __shared__ float red[2][4];
  float lo = INFINITY, hi = -INFINITY;
  const size_t stride = (size_t)gridDim.x * blockDim.x;
  for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride) {
    float v = x[i];
    if (act == 1) v = silu_f(v);
    lo = fminf(lo, v);
    hi = fmaxf(hi, v);
  }
  hi = wave_max(hi);
  lo = -wave_max(-lo);
  if ((threadIdx.x & 63) == 0) {
    red[0][threadIdx.x >> 6] = lo;
    red[1][threadIdx.x >> 6] = hi;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    lo = fminf(fminf(red[0][0], red[0][1]), fminf(red[0][2], red[0][3]));
    hi = fmaxf(fmaxf(red[1][0], red[1][1]), fmaxf(red[1][2], red[1][3]));
    if (lo <= hi) {
      atomicMin(slot, f2ord(lo));
      atomicMax(slot + 1, f2ord(hi));
    }
  }
}

static hipError_t launch_minmax_act(const float *x, size_t n, int act, int *slot, hipStream_t st) {
  size_t blocks = (n + 255) / 256;
  if (blocks > 256) blocks = 256;
  if (blocks == 0) return hipSuccess;
  hipLaunchKernelGGL(minmax_kernel, dim3((unsigned)blocks), dim3(256), 0, st, x, n, act, slot);
  return hipGetLastError();
}
hipError_t launch_minmax(const float *x, size_t n, int *slot, hipStream_t st) { return launch_minmax_act(x, n, 0, slot, st); }
hipError_t launch_minmax_silu(const float *x, size_t n, int *slot, hipStream_t st) { return launch_minmax_act(x, n, 1, slot, st); }

__global__ void fill_i32_kernel(int *p, size_t n, int v) {
  const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) p[i] = v;
}
hipError_t launch_fill_i32(int *p, size_t n, int v, hipStream_t st) {
  if (n == 0) return hipSuccess;
  hipLaunchKernelGGL(fill_i32_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, p, n, v);
  return hipGetLastError();
}

}  // namespace qc
