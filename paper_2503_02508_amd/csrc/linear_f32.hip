// float32 linear layers of the un-quantised reference network (calibration, variance-compensation fit):
// y = act(x W^T + b) or y += gate * (x W^T + b), every output one chain of float32 fused multiply-adds in ascending k.
//
// The chain runs on the matrix cores: v_mfma_f32_16x16x4_f32 adds its four products one after the other, each with the
// rounding of a fused multiply-add, in ascending k (checked bit by bit against fmaf; the same holds for 32x32x2), so the
// result is that of a plain loop over k, whatever the tile.  That also means that K is never split: the activation ranges
// of the calibration, and with them every quantised code downstream, do not depend on how a product is launched.
//
// A workgroup of four wavefronts (2 x 2) owns a tile of 32 TB x 32 TB outputs, a wavefront TB x TB blocks of 16 x 16.  K is
// walked in slabs of BK that go from memory straight to LDS (four buffers, chunks swizzled by the thread that fetches them); the
// fragments of the next slab are read into registers while one is multiplied.  What bounds it: the float32 matrix rate (157
// TFLOP/s), the whole tiles a compute unit gets, and what gets in front of the products of a wavefront.  LDS writes from registers
// run at 32 bytes a clock, 512 clocks of a slab whose products take 1024 (TB = 2) or 512 (TB = 1), and fragment reads ahead of
// the products delayed the first one: with both gone, and an XCD's workgroups on a contiguous range of weight panels,
// 512 x 3456 x 1152 takes 41 instead of 51 us, 512 x 1152 x 1152 21 / 25, 512 x 4608 x 1152 57 / 75, 512 x 1152 x 4608 68 / 95.
#include <math.h>

#include "qc_internal.h"

namespace qc {

// all but the last n loads of this wavefront and all its LDS reads done, then the workgroup barrier
#define QC_SLAB_BARRIER(n) asm volatile("s_waitcnt vmcnt(" #n ") lgkmcnt(0)\n\ts_barrier" ::: "memory")

typedef float v4f __attribute__((ext_vector_type(4)));

__device__ __forceinline__ float gelu_f(float v) {
  const float k0 = 0.7978845608028654f, k1 = 0.044715f;
  return 0.5f * v * (1.0f + tanhf(k0 * (v + k1 * v * v * v)));
}

template <int TB, int BK>
__global__ __launch_bounds__(256, 2) void linear_f32_kernel(const float *__restrict__ x, const float *__restrict__ W,
                                                            const float *__restrict__ bias, float *__restrict__ y, int M, int N, int K,
                                                            int gelu, const float *__restrict__ gate, int ld_gate, int T) {
  constexpr int R = 32 * TB, NQ = BK / 4, NS = 4;            // rows of either operand, steps of a slab, slab buffers
  constexpr int CH = BK / 4, RP = 256 / CH, NL = R / RP;     // 16-byte chunks of a slab row, rows per pass, passes
  __shared__ __align__(16) float slabs[NS][2][R * BK];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int tiles_m = (M + R - 1) / R, tiles_n = (N + R - 1) / R;
  const int t = (blockIdx.x & 7) * (gridDim.x >> 3) + (blockIdx.x >> 3);
  if (t >= tiles_m * tiles_n) return;
  const int m0 = __builtin_amdgcn_readfirstlane((t % tiles_m) * R), n0 = __builtin_amdgcn_readfirstlane((t / tiles_m) * R);
  // Pass i of the loads covers rows RP i .. of a slab, 16 bytes per thread, and goes straight to LDS, thread after thread.  Chunk c
  // of row r lies at chunk c ^ swz(r) (so that the 16 rows of a fragment read cover the 64 banks): the thread of a place fetches
  // the chunk that belongs there.
  const auto swz = [](int r) { return (BK == 32 ? r >> 1 : r) & (CH - 1); };
  const int lr = tid / CH, lc = (tid % CH) ^ swz(lr);
  const int ns = (K + BK - 1) / BK;
  unsigned xo[NL], wo[NL];                             // byte offsets of this thread's chunk in slab 0
#pragma unroll
  for (int i = 0; i < NL; ++i) {                       // rows beyond the matrix re-read its last row (never stored)
    xo[i] = ((unsigned)(min(m0 + lr + RP * i, M - 1) - m0) * (unsigned)K + lc * 4) * 4;
    wo[i] = ((unsigned)(min(n0 + lr + RP * i, N - 1) - n0) * (unsigned)K + lc * 4) * 4;
  }
  const unsigned back = (unsigned)max((ns - 1) * BK + lc * 4 + 4 - K, 0) * 4;      // chunks of the last slab beyond K re-read its end
  const float *xb = x + (size_t)m0 * K, *wb = W + (size_t)n0 * K;
  const unsigned lds0 = (unsigned)(size_t)(__attribute__((address_space(3))) float *)&slabs[0][0][0] + wave * 1024;
  // (m0 is a reserved register, which a clobber list cannot name: nothing else in this kernel uses it, tests/test_codegen_cpu.py)
  auto load = [&](int s, int b, int op, int i) {       // slabs past the end re-read the last one (never used)
    const unsigned off = (op ? wo[i] : xo[i]) - (s >= ns - 1 ? back : 0u);
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" ::"s"(lds0 + ((b * 2 + op) * R + i * RP) * BK * 4), "v"(off),
                 "s"((op ? wb : xb) + (size_t)min(s, ns - 1) * BK)
                 : "memory");
  };
  v4f acc[TB][TB];
#pragma unroll
  for (int i = 0; i < TB; ++i)
#pragma unroll
    for (int j = 0; j < TB; ++j) acc[i][j] = (v4f){0.f, 0.f, 0.f, 0.f};
  const int wm = (wave >> 1) * 16 * TB, wn = (wave & 1) * 16 * TB;
  // lane l supplies row l % 16, k = l / 16 of either operand
  const int fo = (lane & 15) * BK + (swz(lane & 15) << 2) + (lane >> 4);
  const int fox = wm * BK + fo, fow = wn * BK + fo;
  float fx[2][NQ][TB], fw[2][NQ][TB];
  // fragment read n of a slab: operand, block and k in the order of use
  auto read = [&](int f, int b, int n) {
    const int q = n / (2 * TB), i = n % TB;
    if (n % (2 * TB) < TB) fx[f][q][i] = slabs[b][0][(fox ^ (q << 2)) + i * 16 * BK];
    else fw[f][q][i] = slabs[b][1][(fow ^ (q << 2)) + i * 16 * BK];
  };
  auto mul = [&](int f, int n) {
    const int q = n / (TB * TB), i = n / TB % TB, j = n % TB;
    acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(fx[f][q][i], fw[f][q][j], acc[i][j], 0, 0, 0);
  };
  constexpr int NM = NQ * TB * TB, NR = NQ * TB * 2, RM = TB == 2 ? 2 : 3;      // products and fragment reads of a slab, reads behind a product
  static_assert((NM - 1) * RM >= NR && NL == 2, "the barrier stands behind every read");
  // Step s: fragment set s % 2 holds slab s, buffer (s + 1) % NS slab s + 1; slabs s + 2 .. are on their way.  Buffer s % NS was
  // read in step s - 1, before its barrier, and takes slab s + NS.  The wait before the barrier is for slab s + 2: those of steps
  // s - 1 and s (2 NL loads each) may be outstanding.  Every LDS and memory instruction is issued behind a product.
  auto step = [&](int s, int u) {                      // u = s mod NS
    const int f = u & 1;
#pragma unroll
    for (int n = 0; n < NM; ++n) {
      __builtin_amdgcn_sched_barrier(0);
      mul(f, n);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int r = n * RM; r < min(n * RM + RM, NR); ++r) read(f ^ 1, (u + 1) % NS, r);
      if (n < 2 * NL) load(s + NS, u, n & 1, n >> 1);
      if (n == NM - 2) QC_SLAB_BARRIER(8);
    }
  };
#pragma unroll
  for (int b = 0; b < NS; ++b)
#pragma unroll
    for (int i = 0; i < 2 * NL; ++i) load(b, b, i & 1, i >> 1);
  QC_SLAB_BARRIER(8);                                  // slabs 0 and 1
#pragma unroll
  for (int r = 0; r < NR; ++r) read(0, 0, r);
  QC_SLAB_BARRIER(8);
  int s = 0;
  for (; s + NS < ns; s += NS) {
#pragma unroll
    for (int u = 0; u < NS; ++u) step(s + u, u);
  }
#pragma unroll
  for (int u = 0; u < NS; ++u) {
    if (s + u + 1 < ns) {
      step(s + u, u);
    } else if (s + u < ns) {                           // no slab follows
      const int nm = (K - (s + u) * BK) / 4 * TB * TB;
#pragma unroll
      for (int n = 0; n < NM; ++n)
        if (n < nm) mul(u & 1, n);
    }
  }
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");     // nothing lands in LDS after the workgroup's end
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
          float *const at = y + (size_t)m * N + n;
          if (gate) *at = *at + gate[(size_t)(m / T) * ld_gate + n] * v;      // as cache_reuse_kernel adds a stored v
          else *at = v;
        }
      }
  }
}

hipError_t launch_linear_f32(const float *x, const float *W, const float *b, float *y, int M, int N, int K, int gelu, const float *gate,
                             int ld_gate, int T, hipStream_t st) {
  if (K % 4 || K < 4) return hipErrorInvalidValue;           // chunks of 16 bytes; the widths of a model are multiples of 16
  // Whole tiles per compute unit, in blocks of 16 x 16 per SIMD.  TB = 2 moves half the bytes per product, which is worth 16 % of a
  // block's time (K = 1152: 5.2 against 6.2 us); TB = 1 divides the work among the compute units more evenly.
  const long long t2 = (long long)((M + 63) / 64) * ((N + 63) / 64), t1 = (long long)((M + 31) / 32) * ((N + 31) / 32);
  if (0.84 * 4.0 * (double)((t2 + 255) / 256) <= (double)((t1 + 255) / 256))
    hipLaunchKernelGGL((linear_f32_kernel<2, 32>), dim3((unsigned)((t2 + 7) / 8 * 8)), dim3(256), 0, st, x, W, b, y, M, N, K, gelu, gate, ld_gate, T);
  else
    hipLaunchKernelGGL((linear_f32_kernel<1, 64>), dim3((unsigned)((t1 + 7) / 8 * 8)), dim3(256), 0, st, x, W, b, y, M, N, K, gelu, gate, ld_gate, T);
  return hipGetLastError();
}

}  // namespace qc
