// Calibration-set clustering (temporal-aware parallel clustering, TAP; the paper's section of that name and its
// algorithm): similarity matrices on the fp32 matrix cores, degree normalisation, leading singular vectors by block
// power iteration with Cholesky QR and a Jacobi Rayleigh-Ritz step, k-means, aggregation over subsamples.
#include <hip/hip_runtime.h>
#include <stdint.h>
#include <math.h>
#include <algorithm>
#include <utility>
#include <vector>
#include "qc_tap.h"
#include "qc_internal.h"
#include "gemm_f32_tile.h"

namespace {

#define TAP_FAIL(code, ...)     \
  do {                          \
    qc::set_error(__VA_ARGS__); \
    return (code);              \
  } while (0)

#define TAP_HIP(expr)                                                                       \
  do {                                                                                      \
    hipError_t e_ = (expr);                                                                 \
    if (e_ != hipSuccess) TAP_FAIL(QC_ERR_HIP, "%s: %s", #expr, hipGetErrorString(e_));     \
  } while (0)

#define TAP_RC(expr)       \
  do {                     \
    int rc_ = (expr);      \
    if (rc_) return rc_;   \
  } while (0)

inline bool aligned16(const void *p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }

typedef float floatx16 __attribute__((ext_vector_type(16)));

constexpr int NUM_XCD = 8;
constexpr int KB_MAX = 128;
constexpr int M_MAX = 8;

// Every kernel of the chain works on one subsample per grid layer z: the subsamples of a group lie the same number of bytes
// apart in the workspace (0 for what they share), so one launch serves them all.
template <class T>
__device__ __forceinline__ T *in_slot(T *p, long long bytes) {
  return reinterpret_cast<T *>(reinterpret_cast<uintptr_t>(p) + blockIdx.z * (uintptr_t)bytes);
}

__device__ __forceinline__ double wave_sum(double v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  return v;
}

// ------------------------------------------------------------------------------------------------ fp32 GEMM
// C[m, n] = sum_k A(m, k) B(n, k) with A(m, k) = A[m * sam + k * sak], B(n, k) = B[n * sbn + k * sbk]; each operand
// is contiguous either along k (KC) or along its own index.  128 x 128 tile per workgroup of four wavefronts (2 x 2,
// each 64 x 64 = 2 x 2 blocks of v_mfma_f32_32x32x2_f32), K walked in slabs of 32 staged through LDS k-major, so that
// an operand fetch is 32 consecutive floats per half wavefront.  The next slab's global loads are in flight while the
// current one is multiplied.
constexpr int TM = 128, TN = 128, TK = 32;
// LDS row stride (floats) of a k-major tile.  An operand contiguous along k is transposed on the way in: lane l
// writes element (k = 4 (l % 8) + i, o = l / 8); 4 * 130 = 8 (mod 64) spreads the 64 lanes over 64 banks.  An operand
// contiguous along its own index is stored with 16-byte writes and needs a stride that is a multiple of 4.
template <bool KC>
constexpr int ldt() { return KC ? 130 : 132; }

enum SgemmEpi { SE_PLAIN = 0, SE_SIM = 1, SE_COLSCALE = 2 };

struct SgemmArgs {
  const float *A, *B;
  float *C;
  long long sam, sak, sbn, sbk, ldc;
  int M, N, K;
  int a_kc, b_kc;     // operand contiguous along k (else along its own index)
  int a_vec, b_vec;   // 16-byte loads are safe (alignment and extents are multiples of 4)
  // SE_SIM: C = alpha * acc * rs[m] * cs[n] + (1 - alpha) * exp(-|tr[m] - tc[n]|);  SE_COLSCALE: C = acc * cs[n]
  const float *rs, *cs, *tr, *tc;
  float alpha;
  // split K (SE_PLAIN only): workgroup (tile, blockIdx.y = s) multiplies k in [s * kchunk, (s + 1) * kchunk) and writes
  // its partial product to C + s * part_stride; a second kernel adds the partial products in order.  zero_k: that many of the last k
  // are padding, zero in both operands: they don't count for where K is split, so that padding changes no sum
  int zero_k, kchunk;
  long long part_stride;
  // symmetric product (SE_PLAIN, B = A with the same strides, M = N): only the tiles on and below the diagonal are
  // computed; the kernel that adds the partial products also writes the mirror image
  int sym;
  // bytes from one subsample to the next (grid z): the operands, the result, the partial products, the epilogue's factors
  long long za, zb, zc, zpart, zrs, zcs, ztr, ztc;
};

// One operand's share of a slab for this thread: four units of four consecutive elements.
//  KC: unit u -> (o = u / 8, k4 = (u % 8) * 4), elements along k
//  else: unit u -> (k = u / 32, o4 = (u % 32) * 4), elements along o
// Out-of-range elements are loaded from a clamped (valid) address and zeroed only when the slab is written to LDS
// (bit 4 p + i of the returned mask = element i of unit p is in range): nothing touches a loaded register before
// that, so all loads of a slab stay in flight together while the previous slab is multiplied.
template <bool KC, bool vec>
__device__ __forceinline__ unsigned load_units(const float *P, long long so, long long sk, int o0, int O, int k0, int K,
                                               int tid, float4 (&r)[4]) {
  unsigned mask = 0;
#pragma unroll
  for (int p = 0; p < 4; ++p) {
    const int u = tid + 256 * p;
    if (KC) {
      const int o = o0 + (u >> 3), k = k0 + ((u & 7) << 2);
      if (vec) {
        const bool ok = o < O && k < K;
        r[p] = *reinterpret_cast<const float4 *>(P + (ok ? (long long)o * so + k : 0));
        mask |= ok ? 0xFu << (4 * p) : 0u;
      } else {
        float e[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const bool ok = o < O && k + i < K;
          e[i] = P[ok ? (long long)o * so + (long long)(k + i) * sk : 0];
          mask |= ok ? 1u << (4 * p + i) : 0u;
        }
        r[p] = make_float4(e[0], e[1], e[2], e[3]);
      }
    } else {
      const int k = k0 + (u >> 5), o = o0 + ((u & 31) << 2);
      if (vec) {
        const bool ok = o < O && k < K;
        r[p] = *reinterpret_cast<const float4 *>(P + (ok ? (long long)k * sk + o : 0));
        mask |= ok ? 0xFu << (4 * p) : 0u;
      } else {
        // element loads: lane l takes o = l % 32 + 32 i, so that every load covers 32 consecutive floats
        const int ob = o0 + (u & 31);
        float e[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const bool ok = ob + 32 * i < O && k < K;
          e[i] = P[ok ? (long long)k * sk + (long long)(ob + 32 * i) * so : 0];
          mask |= ok ? 1u << (4 * p + i) : 0u;
        }
        r[p] = make_float4(e[0], e[1], e[2], e[3]);
      }
    }
  }
  return mask;
}

template <bool KC, bool vec>
__device__ __forceinline__ void store_units(float *T, int tid, unsigned mask, const float4 (&r)[4]) {
  constexpr int LDT = ldt<KC>();
#pragma unroll
  for (int p = 0; p < 4; ++p) {
    const int u = tid + 256 * p;
    const float x = (mask >> (4 * p)) & 1u ? r[p].x : 0.f, y = (mask >> (4 * p + 1)) & 1u ? r[p].y : 0.f;
    const float z = (mask >> (4 * p + 2)) & 1u ? r[p].z : 0.f, w = (mask >> (4 * p + 3)) & 1u ? r[p].w : 0.f;
    if (KC) {
      const int o = u >> 3, k = (u & 7) << 2;
      T[(k + 0) * LDT + o] = x;
      T[(k + 1) * LDT + o] = y;
      T[(k + 2) * LDT + o] = z;
      T[(k + 3) * LDT + o] = w;
    } else {
      const int k = u >> 5;
      if (vec) {
        *reinterpret_cast<float4 *>(T + k * LDT + ((u & 31) << 2)) = make_float4(x, y, z, w);
      } else {
        float *d = T + k * LDT + (u & 31);
        d[0] = x;
        d[32] = y;
        d[64] = z;
        d[96] = w;
      }
    }
  }
}

// entry t of the lower triangle walked row by row -> (row, column), column <= row
__device__ __forceinline__ void tri_decode(int t, int &row, int &col) {
  int r = (int)((sqrtf(8.f * (float)t + 1.f) - 1.f) * 0.5f);
  while (r * (r + 1) / 2 > t) --r;
  while ((r + 1) * (r + 2) / 2 <= t) ++r;
  row = r;
  col = t - r * (r + 1) / 2;
}

// VEC: both operands take 16-byte loads (a compile-time choice: a run-time branch around the loads would make the
// compiler wait for them at the join and expose their latency)
template <bool AKC, bool BKC, int EPI, bool VEC>
__global__ __launch_bounds__(256, 2) void sgemm_kernel(SgemmArgs p) {
  constexpr int LDA = ldt<AKC>(), LDB = ldt<BKC>();
  p.A = in_slot(p.A, p.za);
  p.B = in_slot(p.B, p.zb);
  p.C = in_slot(p.C, gridDim.y > 1 ? p.zpart : p.zc);
  if (EPI != SE_PLAIN) p.cs = in_slot(p.cs, p.zcs);
  if (EPI == SE_SIM) {
    p.rs = in_slot(p.rs, p.zrs);
    p.tr = in_slot(p.tr, p.ztr);
    p.tc = in_slot(p.tc, p.ztc);
  }
  __shared__ __align__(16) float As[2][TK * LDA];
  __shared__ __align__(16) float Bs[2][TK * LDB];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int tiles_m = (p.M + TM - 1) / TM, tiles_n = (p.N + TN - 1) / TN;
  const int total = p.sym ? tiles_m * (tiles_m + 1) / 2 : tiles_m * tiles_n;
  // workgroups are dealt round-robin to the 8 XCDs: give each XCD a contiguous run of tiles (n fastest) so that the
  // tiles sharing an A panel meet in one L2
  const int per_xcd = (total + NUM_XCD - 1) / NUM_XCD;
  const int tile = (blockIdx.x % NUM_XCD) * per_xcd + blockIdx.x / NUM_XCD;
  if (blockIdx.x / NUM_XCD >= per_xcd || tile >= total) return;
  int tm, tn;
  if (p.sym) {
    tri_decode(tile, tm, tn);
  } else {
    tm = tile / tiles_n;
    tn = tile % tiles_n;
  }
  const int m0 = tm * TM, n0 = tn * TN;
  const int wm0 = (wave >> 1) * 64, wn0 = (wave & 1) * 64;

  floatx16 acc[2][2];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;

  // Two LDS buffers: while slab s is multiplied from one, slab s + 1 (already in registers) is written to the other
  // and slab s + 2 is requested from memory; one barrier per slab.  A buffer is overwritten two slabs after it was
  // read, and the barrier in between is passed only by wavefronts that have finished reading it.
  float4 ra[4], rb[4];
  const int kbeg = blockIdx.y * p.kchunk, kend = min(p.K, kbeg + p.kchunk);
  const int nslab = (kend - kbeg + TK - 1) / TK;
  if (EPI == SE_PLAIN) p.C += (long long)blockIdx.y * p.part_stride;
  unsigned ma = load_units<AKC, VEC>(p.A, p.sam, p.sak, m0, p.M, kbeg, kend, tid, ra);
  unsigned mb = load_units<BKC, VEC>(p.B, p.sbn, p.sbk, n0, p.N, kbeg, kend, tid, rb);
  store_units<AKC, VEC>(As[0], tid, ma, ra);
  store_units<BKC, VEC>(Bs[0], tid, mb, rb);
  ma = load_units<AKC, VEC>(p.A, p.sam, p.sak, m0, p.M, kbeg + TK, kend, tid, ra);
  mb = load_units<BKC, VEC>(p.B, p.sbn, p.sbk, n0, p.N, kbeg + TK, kend, tid, rb);
  __syncthreads();
  for (int s = 0; s < nslab; ++s) {
    const int cur = s & 1;
    if (s + 1 < nslab) {
      store_units<AKC, VEC>(As[cur ^ 1], tid, ma, ra);
      store_units<BKC, VEC>(Bs[cur ^ 1], tid, mb, rb);
    }
    if (s + 2 < nslab) {
      ma = load_units<AKC, VEC>(p.A, p.sam, p.sak, m0, p.M, kbeg + (s + 2) * TK, kend, tid, ra);
      mb = load_units<BKC, VEC>(p.B, p.sbn, p.sbk, n0, p.N, kbeg + (s + 2) * TK, kend, tid, rb);
    }
    const float *ap = As[cur] + (lane >> 5) * LDA + wm0 + (lane & 31);
    const float *bp = Bs[cur] + (lane >> 5) * LDB + wn0 + (lane & 31);
    // the fragments of step kk + 1 are read from LDS before the four products of step kk are issued (the
    // scheduling barriers pin that order), so an LDS round trip hides behind 256 cycles of matrix-core work
    float a0 = ap[0], a1 = ap[32], b0 = bp[0], b1 = bp[32];
    __builtin_amdgcn_sched_group_barrier(0x100, 2, 0);
#pragma unroll
    for (int kk = 0; kk < TK / 2; ++kk) {
      float na0 = 0.f, na1 = 0.f, nb0 = 0.f, nb1 = 0.f;
      if (kk + 1 < TK / 2) {
        na0 = ap[(kk + 1) * 2 * LDA];
        na1 = ap[(kk + 1) * 2 * LDA + 32];
        nb0 = bp[(kk + 1) * 2 * LDB];
        nb1 = bp[(kk + 1) * 2 * LDB + 32];
        __builtin_amdgcn_sched_group_barrier(0x100, 2, 0);      // the LDS reads (two paired loads)
      }
      acc[0][0] = __builtin_amdgcn_mfma_f32_32x32x2f32(a0, b0, acc[0][0], 0, 0, 0);
      acc[0][1] = __builtin_amdgcn_mfma_f32_32x32x2f32(a0, b1, acc[0][1], 0, 0, 0);
      acc[1][0] = __builtin_amdgcn_mfma_f32_32x32x2f32(a1, b0, acc[1][0], 0, 0, 0);
      acc[1][1] = __builtin_amdgcn_mfma_f32_32x32x2f32(a1, b1, acc[1][1], 0, 0, 0);
      __builtin_amdgcn_sched_group_barrier(0x008, 4, 0);        // then the four matrix instructions
      a0 = na0;
      a1 = na1;
      b0 = nb0;
      b1 = nb1;
    }
    __syncthreads();
  }

  // epilogue: register r of a 32 x 32 block is row 8 (r / 4) + 4 (lane / 32) + r % 4, column lane % 32.  The row
  // factors of the similarity epilogue are fetched for all 32 rows of this lane in one batch (clamped, branch-free)
  float rsv[2][16], trv[2][16];
  if (EPI == SE_SIM) {
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int m = m0 + wm0 + i * 32 + (r >> 2) * 8 + (lane >> 5) * 4 + (r & 3);
        const int mm = m < p.M ? m : p.M - 1;
        rsv[i][r] = p.rs[mm];
        trv[i][r] = p.tr[mm];
      }
  }
#pragma unroll
  for (int j = 0; j < 2; ++j) {
    const int n = n0 + wn0 + j * 32 + (lane & 31);
    const bool nok = n < p.N;
    float csn = 1.f, tcn = 0.f;
    if (EPI != SE_PLAIN) csn = p.cs[nok ? n : 0];
    if (EPI == SE_SIM) tcn = p.tc[nok ? n : 0];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int m = m0 + wm0 + i * 32 + (r >> 2) * 8 + (lane >> 5) * 4 + (r & 3);
        float v = acc[i][j][r];
        if (EPI == SE_SIM) v = p.alpha * (v * rsv[i][r] * csn) + (1.f - p.alpha) * expf(-fabsf(trv[i][r] - tcn));
        if (EPI == SE_COLSCALE) v *= csn;
        if (nok && m < p.M) p.C[(long long)m * p.ldc + n] = v;
      }
  }
}

// The same product for operands that are both contiguous along k, K a multiple of 4 (split K: whole slabs), or both along their own
// index, and take 16-byte loads, on tiles of 64 WT x 64 WT whose slabs go straight to LDS (gemm_f32_tile.h).  Same chains, same bits.  What bounds it: the matrix
// rate at the clock the chip holds (2.1 - 2.3 GHz).  32768 x 1638 x 4096: 4.2 ms on sgemm_kernel (105 TFLOP/s, slabs through
// registers, two workgroups a compute unit), 3.2 here with one workgroup of 128 x 128 and six buffers a compute unit (138; four buffers 3.3,
// eight 3.2, ten 3.25, slabs of 32 k 3.3, wavefronts of 128 x 64 3.5, tiles of 128 x 256 3.25); the library's product takes 2.96.  The order of
// the tiles made no difference.  Four buffers leave room for two such workgroups (64 KB of LDS each), so that one multiplies while
// the other starts or stores, which a lone one does with the matrix cores idle: similarity of three subsamples with its epilogue 11.08 ->
// 10.78 ms (119 -> 122 TFLOP/s), L^T L of 32768 x 1640 (three; 3.0 ms on sgemm_kernel) 2.60 -> 2.51, block products 76 -> 67 us.  Tiles of
// 64 x 64 have room for three with six buffers; four buffers made no difference there.
constexpr int NT_BK = 16;
template <int WT, int EPI, bool TN>      // TN: both operands contiguous along their own index (plain products)
__global__ __launch_bounds__(256, 2) void sgemm_slab_kernel(SgemmArgs p) {
  constexpr int NS = WT == 2 ? 4 : 6;      // slab buffers
  using Tile = qc::F32Tile<2, 2, WT, WT, NT_BK, NS>;
  __shared__ __align__(16) float slabs[NS * Tile::SLAB];
  const int tiles_m = (p.M + Tile::RM - 1) / Tile::RM, tiles_n = (p.N + Tile::RN - 1) / Tile::RN;
  const int total = TN && p.sym ? tiles_m * (tiles_m + 1) / 2 : tiles_m * tiles_n, per_xcd = (total + NUM_XCD - 1) / NUM_XCD;
  const int t = (blockIdx.x % NUM_XCD) * per_xcd + blockIdx.x / NUM_XCD;
  if (blockIdx.x / NUM_XCD >= per_xcd || t >= total) return;
  int tm = t / tiles_n, tn = t % tiles_n;
  if (TN && p.sym) tri_decode(t, tm, tn);
  const int m0 = __builtin_amdgcn_readfirstlane(tm * Tile::RM), n0 = __builtin_amdgcn_readfirstlane(tn * Tile::RN);
  const float *A = in_slot(p.A, p.za), *B = in_slot(p.B, p.zb);
  float *C = in_slot(p.C, gridDim.y > 1 ? p.zpart : p.zc) + (EPI == SE_PLAIN ? (long long)blockIdx.y * p.part_stride : 0);
  const int kbeg = EPI == SE_PLAIN ? blockIdx.y * p.kchunk : 0, kend = EPI == SE_PLAIN ? min(p.K, kbeg + p.kchunk) : p.K;
  Tile tile;
  if (TN) tile.run_tn(A + (size_t)kbeg * p.sak, (size_t)p.sak, B + (size_t)kbeg * p.sbk, (size_t)p.sbk, p.M, p.N, kend - kbeg, m0, n0, slabs);
  else tile.run(A + kbeg, (size_t)p.sam, B + kbeg, (size_t)p.sbn, p.M, p.N, kend - kbeg, m0, n0, slabs);
  // register r of a 32 x 32 block is row 8 (r / 4) + 4 (lane / 32) + r % 4, column lane % 32
  const int lane = threadIdx.x & 63;
  const float *rs = nullptr, *tr = nullptr, *tc = nullptr, *cs = nullptr;
  if (EPI != SE_PLAIN) cs = in_slot(p.cs, p.zcs);
  if (EPI == SE_SIM) {
    rs = in_slot(p.rs, p.zrs);
    tr = in_slot(p.tr, p.ztr);
    tc = in_slot(p.tc, p.ztc);
  }
#pragma unroll
  for (int i = 0; i < WT; ++i) {
    float rsv[16], trv[16];
    if (EPI == SE_SIM) {
#pragma unroll
      for (int r = 0; r < 16; ++r) {        // the row factors of this lane in one batch (clamped, branch-free)
        const int m = min(m0 + tile.wm + 32 * i + (r >> 2) * 8 + (lane >> 5) * 4 + (r & 3), p.M - 1);
        rsv[r] = rs[m];
        trv[r] = tr[m];
      }
    }
#pragma unroll
    for (int j = 0; j < WT; ++j) {
      const int n = n0 + tile.wn + 32 * j + (lane & 31);
      const bool nok = n < p.N;
      const float csn = EPI != SE_PLAIN ? cs[nok ? n : 0] : 1.f, tcn = EPI == SE_SIM ? tc[nok ? n : 0] : 0.f;
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int m = m0 + tile.wm + 32 * i + (r >> 2) * 8 + (lane >> 5) * 4 + (r & 3);
        float v = tile.acc[i][j][r];
        if (EPI == SE_SIM) v = p.alpha * (v * rsv[r] * csn) + (1.f - p.alpha) * expf(-fabsf(trv[r] - tcn));
        if (EPI == SE_COLSCALE) v *= csn;
        if (nok && m < p.M) C[(long long)m * p.ldc + n] = v;
      }
    }
  }
}

__global__ __launch_bounds__(256) void splitk_reduce_kernel(const float *part, int splits, long long stride,
                                                            long long count, float *out, long long zpart, long long zout) {
  part = in_slot(part, zpart);
  out = in_slot(out, zout);
  const long long i = (long long)blockIdx.x * 256 + threadIdx.x;
  if (i >= count) return;
  float s = 0.f;
  for (int q = 0; q < splits; ++q) s += part[q * stride + i];
  out[i] = s;
}

// the same for a symmetric n x n product of which only the tiles on and below the diagonal were computed: one
// workgroup per 32 x 32 block on or below the diagonal adds the partial products, writes the block and, through LDS,
// its transpose (`out` may be `part` when there is a single partial product)
__global__ __launch_bounds__(256) void splitk_reduce_sym_kernel(const float *part, int splits, long long stride, int n,
                                                                long long ldc, float *out, long long zpart, long long zout) {
  part = in_slot(part, zpart);
  out = in_slot(out, zout);
  __shared__ float tile[32][33];
  int bm, bn;
  tri_decode(blockIdx.x, bm, bn);
  const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5;
#pragma unroll
  for (int rr = 0; rr < 4; ++rr) {
    const int r = bm * 32 + ty + 8 * rr, c = bn * 32 + tx;
    const bool ok = r < n && c < n;
    float s = 0.f;
    for (int q = 0; q < splits; ++q) s += part[ok ? q * stride + (long long)r * ldc + c : 0];
    if (ok) out[(long long)r * ldc + c] = s;
    tile[ty + 8 * rr][tx] = s;
  }
  __syncthreads();
  if (bm == bn) return;
#pragma unroll
  for (int rr = 0; rr < 4; ++rr) {
    const int r = bn * 32 + ty + 8 * rr, c = bm * 32 + tx;
    if (r < n && c < n) out[(long long)r * ldc + c] = tile[tx][ty + 8 * rr];
  }
}

// `part` (part_elems floats) allows a plain product with few tiles and a long K to be split along K
hipError_t sgemm(SgemmArgs a, int epi, int nz, hipStream_t st, float *part = nullptr, size_t part_elems = 0) {
  if (a.M <= 0 || a.N <= 0) return hipSuccess;
  a.a_kc = a.sak == 1;
  a.b_kc = a.sbk == 1;
  if (!a.a_kc && a.sam != 1) return hipErrorInvalidValue;
  if (!a.b_kc && a.sbn != 1) return hipErrorInvalidValue;
  // 16-byte loads: base aligned, the strided dimension's stride and the contiguous extent multiples of 4
  a.a_vec = aligned16(a.A) && (a.a_kc ? (a.sam % 4 == 0 && a.K % 4 == 0) : (a.sak % 4 == 0 && a.M % 4 == 0));
  a.b_vec = aligned16(a.B) && (a.b_kc ? (a.sbn % 4 == 0 && a.K % 4 == 0) : (a.sbk % 4 == 0 && a.N % 4 == 0));
  if (a.sym && (epi != SE_PLAIN || a.M != a.N || a.A != a.B || a.sam != a.sbn || a.sak != a.sbk)) return hipErrorInvalidValue;
  const int tiles_m = (a.M + TM - 1) / TM;
  const int tiles = a.sym ? tiles_m * (tiles_m + 1) / 2 : tiles_m * ((a.N + TN - 1) / TN);
  const int grid = ((tiles + NUM_XCD - 1) / NUM_XCD) * NUM_XCD;
  int splits = 1;
  a.kchunk = a.K > 0 ? a.K : 1;
  a.part_stride = 0;
  float *out = a.C;
  const long long out_elems = (long long)a.M * a.ldc;
  const int K = a.K - a.zero_k;
  if (epi == SE_PLAIN && part && tiles < 256 && K >= 8 * TK) {
    long long want = 512 / tiles;            // at most the 512 workgroups the chip holds at a time
    if (want > 16) want = 16;
    if (want > K / (4 * TK)) want = K / (4 * TK);
    if (want > (long long)(part_elems / (size_t)out_elems)) want = (long long)(part_elems / (size_t)out_elems);
    if (want > 1) {
      a.kchunk = (int)(((K + want - 1) / want + TK - 1) / TK * TK);
      splits = (a.K + a.kchunk - 1) / a.kchunk;
      a.part_stride = out_elems;
      a.C = part;
    }
  }
  const bool vec = a.a_vec && a.b_vec;
  // Both operands contiguous along k or both along their own index, whole 16-byte chunks: the kernel whose slabs go straight to LDS
  // (its offsets inside a tile are 32-bit bytes: rows shorter than 2^22 floats).  Tiles of 128 x 128 while they fill the chip, of
  // 64 x 64 below (1536 x 160 x 256, three subsamples: 38 us on sgemm_kernel, 21 on 128 x 128, 16 on 64 x 64).
  const bool nt = a.a_kc && a.b_kc && a.sam < (1 << 22) && a.sbn < (1 << 22);
  const bool tn = !a.a_kc && !a.b_kc && epi == SE_PLAIN && a.sak < (1 << 22) && a.sbk < (1 << 22);
  if (vec && a.K >= 4 && a.M >= 4 && a.N >= 4 && (nt || tn)) {
    const int wt = (long long)tiles * splits * nz >= 256 ? 2 : 1;
    const int side = (a.M + 63) / 64;
    const int slab_tiles = wt == 2 ? tiles : a.sym ? side * (side + 1) / 2 : side * ((a.N + 63) / 64);
    const dim3 slab_grid((unsigned)((slab_tiles + NUM_XCD - 1) / NUM_XCD * NUM_XCD), (unsigned)splits, (unsigned)nz);
#define SLAB_LAUNCH(E, T)                                                                                  \
  do {                                                                                                     \
    if (wt == 2) hipLaunchKernelGGL((sgemm_slab_kernel<2, E, T>), slab_grid, dim3(256), 0, st, a);         \
    else hipLaunchKernelGGL((sgemm_slab_kernel<1, E, T>), slab_grid, dim3(256), 0, st, a);                 \
  } while (0)
    if (tn) SLAB_LAUNCH(SE_PLAIN, true);
    else if (epi == SE_SIM) SLAB_LAUNCH(SE_SIM, false);
    else if (epi == SE_COLSCALE) SLAB_LAUNCH(SE_COLSCALE, false);
    else SLAB_LAUNCH(SE_PLAIN, false);
#undef SLAB_LAUNCH
  } else {
#define SG_LAUNCH(AK, BK, E)                                                                                   \
  do {                                                                                                         \
    if (vec) hipLaunchKernelGGL((sgemm_kernel<AK, BK, E, true>), dim3(grid, splits, nz), dim3(256), 0, st, a); \
    else hipLaunchKernelGGL((sgemm_kernel<AK, BK, E, false>), dim3(grid, splits, nz), dim3(256), 0, st, a);    \
  } while (0)
  if (epi == SE_SIM) {
    if (a.a_kc && a.b_kc) SG_LAUNCH(true, true, SE_SIM);
    else return hipErrorInvalidValue;
  } else if (epi == SE_COLSCALE) {
    if (a.a_kc && a.b_kc) SG_LAUNCH(true, true, SE_COLSCALE);
    else return hipErrorInvalidValue;
  } else {
    if (a.a_kc && a.b_kc) SG_LAUNCH(true, true, SE_PLAIN);
    else if (a.a_kc && !a.b_kc) SG_LAUNCH(true, false, SE_PLAIN);
    else if (!a.a_kc && !a.b_kc) SG_LAUNCH(false, false, SE_PLAIN);
    else return hipErrorInvalidValue;
  }
#undef SG_LAUNCH
  }
  if (a.sym) {
    const int nb = (a.M + 31) / 32;
    hipLaunchKernelGGL(splitk_reduce_sym_kernel, dim3(nb * (nb + 1) / 2, 1, nz), dim3(256), 0, st,
                       splits > 1 ? (const float *)part : (const float *)out, splits, out_elems, a.M, a.ldc, out,
                       splits > 1 ? a.zpart : a.zc, a.zc);
  } else if (splits > 1) {
    hipLaunchKernelGGL(splitk_reduce_kernel, dim3((unsigned)((out_elems + 255) / 256), 1, nz), dim3(256), 0, st, part,
                       splits, out_elems, out_elems, out, a.zpart, a.zc);
  }
  return hipGetLastError();
}

// --------------------------------------------------------------------------------------- similarity helpers
// 1 / |x_r| of every pool row (fp64 sum of squares); 0 for a zero row
__global__ __launch_bounds__(256) void rownorm_kernel(const float *X, int N, int F, float *rinv) {
  const int row = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
  if (row >= N) return;
  const float *x = X + (long long)row * F;
  double s = 0.0;
  for (int j = lane; j < F; j += 64) {
    const double v = x[j];
    s += v * v;
  }
  s = wave_sum(s);
  if (lane == 0) rinv[row] = s > 0.0 ? (float)(1.0 / sqrt(s)) : 0.f;
}

// rows, inverse norms and timestamps of one subsample gathered into dense arrays; an index outside [0, N) raises
// the flag and is replaced by 0
__global__ __launch_bounds__(256) void gather_kernel(const float *X, const float *rinv, const float *t, const int *idx,
                                                     int N, int F, float *Xs, float *cs, float *tc, int *flag,
                                                     long long zidx, long long zw, long long zflag) {
  const int h = blockIdx.x;
  idx = in_slot(idx, zidx);
  Xs = in_slot(Xs, zw);
  cs = in_slot(cs, zw);
  tc = in_slot(tc, zw);
  flag = in_slot(flag, zflag);
  int s = idx[h];
  if (s < 0 || s >= N) {
    if (threadIdx.x == 0) atomicOr(flag, 1);
    s = 0;
  }
  const float *src = X + (long long)s * F;
  float *dst = Xs + (long long)h * F;
  for (int j = threadIdx.x; j < F; j += 256) dst[j] = src[j];
  if (threadIdx.x == 0) {
    cs[h] = rinv[s];
    tc[h] = t[s];
  }
}

// d_r: one wavefront per row, fp64 sum
__global__ __launch_bounds__(256) void rowsum_kernel(const float *A, int N, int n, int lda, float *dr, long long zw) {
  A = in_slot(A, zw);
  dr = in_slot(dr, zw);
  const int row = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
  if (row >= N) return;
  const float *a = A + (long long)row * lda;
  double s = 0.0;
  for (int j = lane; j < n; j += 64) s += (double)a[j];
  s = wave_sum(s);
  if (lane == 0) dr[row] = (float)s;
}

// d_c in two deterministic stages: partial sums of COL_CHUNKS row ranges, then their sum in order
constexpr int COL_CHUNKS = 64;
__global__ __launch_bounds__(256) void colsum_partial_kernel(const float *A, int N, int n, int lda, double *part,
                                                             long long zw) {
  A = in_slot(A, zw);
  part = in_slot(part, zw);
  __shared__ double red[4][64];
  const int c = threadIdx.x & 63, ph = threadIdx.x >> 6;
  const int col = blockIdx.x * 64 + c;
  const int rows_per = (N + COL_CHUNKS - 1) / COL_CHUNKS;
  const int r0 = blockIdx.y * rows_per, r1 = min(N, r0 + rows_per);
  double s = 0.0;
  if (col < n)
    for (int r = r0 + ph; r < r1; r += 4) s += (double)A[(long long)r * lda + col];
  red[ph][c] = s;
  __syncthreads();
  if (ph == 0 && col < n) part[(long long)blockIdx.y * n + col] = ((red[0][c] + red[1][c]) + red[2][c]) + red[3][c];
}

// Both sums in one pass over A for up to 64 NC columns: the same row ranges and phases, a wavefront's lanes across a row, the
// column sums of its phase in registers.  What bounds it: the pass over A (three of 215 MB: 390 us as two kernels, 182 here).
template <int NC>
__global__ __launch_bounds__(256) void degree_sums_kernel(const float *A, int N, int n, int lda, float *dr, double *part, long long zw) {
  A = in_slot(A, zw);
  dr = in_slot(dr, zw);
  part = in_slot(part, zw);
  __shared__ double red[4][64];
  const int lane = threadIdx.x & 63, ph = threadIdx.x >> 6;
  const int rows_per = (N + COL_CHUNKS - 1) / COL_CHUNKS;
  const int r0 = blockIdx.x * rows_per, r1 = min(N, r0 + rows_per);
  double cs[NC];
#pragma unroll
  for (int c = 0; c < NC; ++c) cs[c] = 0.0;
  for (int r = r0 + ph; r < r1; r += 4) {
    const float *a = A + (long long)r * lda;
    float v[NC];
#pragma unroll
    for (int c = 0; c < NC; ++c) v[c] = a[min(lane + 64 * c, n - 1)];
    double s = 0.0;
#pragma unroll
    for (int c = 0; c < NC; ++c) {
      const double d = lane + 64 * c < n ? (double)v[c] : 0.0;
      s += d;
      cs[c] += d;
    }
    s = wave_sum(s);
    if (lane == 0) dr[r] = (float)s;
  }
#pragma unroll
  for (int c = 0; c < NC; ++c) {
    __syncthreads();
    red[ph][lane] = cs[c];
    __syncthreads();
    if (ph == 0 && lane + 64 * c < n) part[(long long)blockIdx.x * n + lane + 64 * c] = ((red[0][lane] + red[1][lane]) + red[2][lane]) + red[3][lane];
  }
}

__global__ __launch_bounds__(256) void colsum_final_kernel(const double *part, int n, float *dc, long long zw) {
  part = in_slot(part, zw);
  dc = in_slot(dc, zw);
  const int col = blockIdx.x * 256 + threadIdx.x;
  if (col >= n) return;
  double s = 0.0;
  for (int b = 0; b < COL_CHUNKS; ++b) s += part[(long long)b * n + col];
  dc[col] = (float)s;
}

__global__ __launch_bounds__(256) void fill_int_kernel(int *p, int count, int v, long long zp) {
  p = in_slot(p, zp);
  const int i = blockIdx.x * 256 + threadIdx.x;
  if (i < count) p[i] = v;
}

__global__ __launch_bounds__(256) void degree_check_kernel(const float *dr, int N, const float *dc, int n, int *flag,
                                                           long long zw, long long zflag) {
  dr = in_slot(dr, zw);
  dc = in_slot(dc, zw);
  flag = in_slot(flag, zflag);
  const int i = blockIdx.x * 256 + threadIdx.x;
  if (i < N + n) {
    const float v = i < N ? dr[i] : dc[i - N];
    if (!(v > 0.f) || !isfinite(v)) atomicOr(flag, 1);
  }
}

// `guard` (may be null): a device flag raised by the degree check; the matrix is left alone when it is set.  Rows lie lda
// floats apart; what lies between (a workspace matrix with padded rows) becomes zero.  A workgroup takes NORM_ROWS rows of 256 VEC
// columns: the reciprocal roots of its rows and columns are formed once, so that the pass is bound by its bytes (three matrices of
// 215 MB: 656 us with both roots per element, 250 here).
constexpr int NORM_ROWS = 8;
template <int VEC>
__global__ __launch_bounds__(256) void normalise_kernel(float *A, const float *dr, const float *dc, int N, int n, int lda,
                                                        const int *guard, long long zw, long long zflag) {
  if (guard && *in_slot(guard, zflag)) return;
  A = in_slot(A, zw);
  dr = in_slot(dr, zw);
  dc = in_slot(dc, zw);
  __shared__ float ir[NORM_ROWS];
  const int nblk = (lda + 256 * VEC - 1) / (256 * VEC);
  const int r0 = blockIdx.x / nblk * NORM_ROWS, h = (blockIdx.x % nblk * 256 + threadIdx.x) * VEC;
  if (threadIdx.x < NORM_ROWS && r0 + (int)threadIdx.x < N) ir[threadIdx.x] = 1.f / sqrtf(dr[r0 + threadIdx.x]);
  __syncthreads();
  if (h >= lda) return;
  float ic[VEC];
#pragma unroll
  for (int e = 0; e < VEC; ++e) ic[e] = h + e < n ? 1.f / sqrtf(dc[h + e]) : 0.f;
  const int rows = min(NORM_ROWS, N - r0);
  float *a = A + (long long)r0 * lda + h;
#pragma unroll 4
  for (int r = 0; r < rows; ++r, a += lda) {
    if constexpr (VEC == 4) {
      float4 v = *(const float4 *)a;
      v.x = h < n ? v.x * (ir[r] * ic[0]) : 0.f;
      v.y = h + 1 < n ? v.y * (ir[r] * ic[1]) : 0.f;
      v.z = h + 2 < n ? v.z * (ir[r] * ic[2]) : 0.f;
      v.w = h + 3 < n ? v.w * (ir[r] * ic[3]) : 0.f;
      *(float4 *)a = v;
    } else {
      *a = h < n ? *a * (ir[r] * ic[0]) : 0.f;
    }
  }
}

// rows of n floats copied to rows of ld floats, zeros behind them
__global__ __launch_bounds__(256) void pad_rows_kernel(const float *src, int n, float *dst, int ld, long long zdst) {
  dst = in_slot(dst, zdst);
  for (int j = threadIdx.x; j < ld; j += 256) dst[(long long)blockIdx.x * ld + j] = j < n ? src[(long long)blockIdx.x * n + j] : 0.f;
}

// -------------------------------------------------------------------------- orthonormalisation (Cholesky QR)
// v_mfma_f64_16x16x4_f64: lane l supplies row l % 16, k = l / 16 of either operand; result i of lane l is row l / 16 + 4 i,
// column l % 16.
typedef double f64x4 __attribute__((ext_vector_type(4)));

// Partial Gram matrices of kb vectors of length n over ranges of their elements, fp64: part[b][a][c] = sum_j y_a[j] y_c[j] for the
// blocks of 16 x 16 on and below the diagonal (the others are not written).  Vector a's element j is Y[a * sv + j] (KC) or
// Y[j * sv + a] (rows of whole, aligned 16-byte chunks).
//
// Every entry is one chain of float64 multiply-adds over the elements of its range in ascending order, from zero: the matrix
// instruction adds its four products one after the other, each with the rounding of a fused multiply-add (checked bit by bit against
// fma).  The order counts: the factor of these sums is rounded to float32 behind a matrix of condition up to 1e12 and Lloyd's iteration
// amplifies what is left; four interleaved chains, or ranges of another length, move 1 % of the labels of a large pool.
//
// 32 elements at a time go through LDS as float32 (the next ones are on their way into registers meanwhile); wavefront w multiplies the
// blocks w, w + 8, ... of the lower triangle, counted row by row.  Bound by the float64 matrix rate where ranges are long (32768
// elements: 256 a range), by the first loads where they are short.  Three subsamples, 128 vectors of 1640 elements: 42 us on the vector
// units (64 outputs a thread, operands from LDS), 8.2 here; 32 vectors of 160: 13 and 3.0; 128 of 32768: 52 here.
template <int NB, bool KC, bool V4>
__global__ __launch_bounds__(512) void gram_partial_kernel(const float *Y, int kb, int n, long long sv, int jchunk, double *part,
                                                           long long zy, long long zw) {
  constexpr int BLK = NB * (NB + 1) / 2, MINE = (BLK + 7) / 8, KP = 16 * NB, JB = 32;
  constexpr int UNITS = KP * JB / 4, NL = (UNITS + 511) / 512;          // 16-byte chunks of a stage, per thread
  // A fragment (16 vectors, 4 elements) is read without bank conflicts: rows of 36 floats, one a vector (KC), or of 16 mod 64, one an element.
  constexpr int LD = KC ? JB + 4 : KP + (80 - KP % 64) % 64;
  __shared__ __align__(16) float ys[2][KC ? KP * LD : JB * LD];
  Y = in_slot(Y, zy);
  part = in_slot(part, zw);
  const int tid = threadIdx.x, lane = tid & 63, row = lane & 15, g = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int j0 = blockIdx.x * jchunk, j1 = min(n, j0 + jchunk);
  float4 r[NL];
  auto load = [&](int jb) {
#pragma unroll
    for (int i = 0; i < NL; ++i) {
      const int u = tid + 512 * i;
      const int a = KC ? u / (JB / 4) : u % (KP / 4) * 4, j = jb + (KC ? u % (JB / 4) * 4 : u / (KP / 4));
      if (!KC || V4) {                            // KC: n a multiple of 4
        const float *p = KC ? Y + (long long)min(a, kb - 1) * sv + min(j, n - 4) : Y + (long long)min(j, n - 1) * sv + min(a, kb - 4);
        const float4 t = *(const float4 *)p;
        const bool in = a < kb && j < j1;
        r[i] = make_float4(in ? t.x : 0.f, in ? t.y : 0.f, in ? t.z : 0.f, in ? t.w : 0.f);
      } else {
        float t[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) t[e] = Y[(long long)min(a, kb - 1) * sv + min(j + e, n - 1)];
        r[i] = make_float4(a < kb && j < j1 ? t[0] : 0.f, a < kb && j + 1 < j1 ? t[1] : 0.f, a < kb && j + 2 < j1 ? t[2] : 0.f,
                           a < kb && j + 3 < j1 ? t[3] : 0.f);
      }
    }
  };
  int p[MINE], q[MINE], fa[MINE], fb[MINE];       // the wavefront's blocks; places of their fragments
  f64x4 acc[MINE];
#pragma unroll
  for (int b = 0; b < MINE; ++b) {
    tri_decode(min(wave + 8 * b, BLK - 1), p[b], q[b]);
    p[b] = __builtin_amdgcn_readfirstlane(p[b]);
    q[b] = __builtin_amdgcn_readfirstlane(q[b]);
    fa[b] = KC ? (16 * p[b] + row) * LD + g : g * LD + 16 * p[b] + row;
    fb[b] = KC ? (16 * q[b] + row) * LD + g : g * LD + 16 * q[b] + row;
    acc[b] = (f64x4){0.0, 0.0, 0.0, 0.0};
  }
  load(j0);
  int s = 0;
  for (int jb = j0; jb < j1; jb += JB, s ^= 1) {
    // (this buffer's last readers were done before the barrier of the stage in between)
#pragma unroll
    for (int i = 0; i < NL; ++i) {
      const int u = tid + 512 * i;
      if (u < UNITS) *(float4 *)(ys[s] + (KC ? u / (JB / 4) * LD + u % (JB / 4) * 4 : u / (KP / 4) * LD + u % (KP / 4) * 4)) = r[i];
    }
    __syncthreads();
    if (jb + JB < j1) load(jb + JB);
#pragma unroll
    for (int e = 0; e < JB / 4; ++e)
#pragma unroll
      for (int b = 0; b < MINE; ++b) {
        if (8 * b + 8 > BLK && wave + 8 * b >= BLK) continue;           // uniform
        const int at = KC ? 4 * e : 4 * e * LD;
        acc[b] = __builtin_amdgcn_mfma_f64_16x16x4f64((double)ys[s][fa[b] + at], (double)ys[s][fb[b] + at], acc[b], 0, 0, 0);
      }
  }
  double *const out = part + (long long)blockIdx.x * kb * kb;
#pragma unroll
  for (int b = 0; b < MINE; ++b) {
    if (wave + 8 * b >= BLK) continue;
    const int c = 16 * q[b] + row;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int rr = 16 * p[b] + g + 4 * i;
      if (rr < kb && c < kb) out[rr * kb + c] = acc[b][i];
    }
  }
}

// the ranges' partial matrices added in order, the lower triangle written to both sides of the diagonal
__global__ __launch_bounds__(256) void gram_reduce_kernel(const double *part, int nparts, int kb, double *W, long long zw) {
  part = in_slot(part, zw);
  W = in_slot(W, zw);
  const int i = blockIdx.x * 256 + threadIdx.x, kk = kb * kb, r = i / kb, c = i - r * kb;
  if (i >= kk || c > r) return;
  double s = 0.0;
  int b = 0;
  for (; b + 16 <= nparts; b += 16) {        // sixteen loads in flight, added in order
    double t[16];
#pragma unroll
    for (int q = 0; q < 16; ++q) t[q] = part[(long long)(b + q) * kk + i];
#pragma unroll
    for (int q = 0; q < 16; ++q) s += t[q];
  }
  for (; b < nparts; ++b) s += part[(long long)b * kk + i];
  W[i] = s;
  W[c * kb + r] = s;
}

// 1 / x and x^-1/2 to fp64 rounding level: hardware estimate, two Newton steps
__device__ __forceinline__ double nr_rcp(double x) {
  double r = __builtin_amdgcn_rcp(x);
  r = r * (2.0 - x * r);
  return r * (2.0 - x * r);
}
__device__ __forceinline__ double nr_rsq(double x) {
  double r = __builtin_amdgcn_rsq(x);
  r = r * (1.5 - 0.5 * x * r * r);
  return r * (1.5 - 0.5 * x * r * r);
}

// lane N's value of a row of 16 lanes to all of the row
template <int N>
__device__ __forceinline__ double row_bcast(double v) {
  const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(v), 0x150 + N, 0xF, 0xF, true);
  const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(v), 0x150 + N, 0xF, 0xF, true);
  return __hiloint2double(hi, lo);
}
// a[c] += (lane c's sc) * ma and b[c] += (lane c's sc) * mb, c = C .. 15: the broadcast is part of the multiply-add
template <int C>
__device__ __forceinline__ void eliminate_columns(double (&a)[16], double (&b)[16], double sc, double ma, double mb) {
  if constexpr (C < 16) {
    asm("v_fmac_f64_dpp %0, %1, %2 row_newbcast:%3 row_mask:0xf bank_mask:0xf" : "+v"(a[C]) : "v"(sc), "v"(ma), "n"(C));
    asm("v_fmac_f64_dpp %0, %1, %2 row_newbcast:%3 row_mask:0xf bank_mask:0xf" : "+v"(b[C]) : "v"(sc), "v"(mb), "n"(C));
    eliminate_columns<C + 1>(a, b, sc, ma, mb);
  }
}
// columns J .. 15 of the elimination of a 16 x 16 block, lane R (of each 16) its row R in a, and of 16 other rows, one a lane, in b; piv, inv:
// lane R's own pivot and its reciprocal
template <int J>
__device__ __forceinline__ void eliminate(double (&a)[16], double (&b)[16], double &piv, double &inv, int row, int check, bool &bad) {
  if constexpr (J < 16) {
    asm("s_nop 1" : "+v"(a[J]));                  // written by the assembly above, which the compiler does not see into, and read across lanes next
    double p = row_bcast<J>(a[J]);
    const bool no = !(p > 0.0) || !(p < INFINITY);
    bad = bad || no || (check && p < 0.25);
    p = no ? 1.0 : p;
    const bool own = row == J;
    const double r = nr_rcp(p);
    piv = own ? p : piv;
    inv = own ? r : inv;
    const double col = a[J], ma = -(own ? 1.0 : col), mb = -b[J];
    double sc;                                    // a value read across lanes has to be two instructions old: the wait is part of it
    asm("v_mul_f64 %0, %1, %2\n\ts_nop 1" : "=v"(sc) : "v"(col), "v"(r));
#pragma unroll
    for (int c = J + 1; c < 16; ++c) a[c] = own ? 0.0 : a[c];
    eliminate_columns<J + 1>(a, b, sc, ma, mb);
    eliminate<J + 1>(a, b, piv, inv, row, check, bad);
  }
}

// Inverse Cholesky factor of W + shift I (= Lc Lc^T, Lc lower), one workgroup.  The shift, shift_rel times the largest
// diagonal entry, keeps the factorisation alive when the rows are numerically dependent (shifted Cholesky QR: the
// rows come out better conditioned, not yet orthonormal, and the next pass finishes).
//
// The square-root-free sweep on one kb x kb array S in LDS (padded with the identity to whole blocks of 16).  After column j, rows R > j of
// the columns C > j hold the trailing matrix, rows R <= j of the columns C > j the inverse being built, r_CR at S[R][C], r's unit diagonal
// implicit.  At column j, with pivot p_j = S[j][j], every element of the columns C > j takes
//   S[R][C] = fma(-g(R), g(C) (1 / p_j), S[R][C]),   g(x) = S[x][j] for x != j, g(j) = 1,
// where row j starts from zero; at the end Lc^-1 = diag(p)^-1/2 r.  An element is one chain of multiply-adds over ascending j whatever the
// blocking: the values go to float32 behind a matrix of condition up to 1e12, so another sequence of roundings gives other labels.
//
// Sixteen columns at a time.  Two wavefronts eliminate block column p: lane R of each 16 keeps row R of the diagonal block, and a row of one other
// block beside it, the scaled column broadcast within the multiply-adds (both take the diagonal block, so nothing passes between
// them).  Then S[R][C] of the columns beyond takes its 16 products on the float64 matrix cores, which add them one after the other with
// the rounding of fma, a block a wavefront: column p + 1 first, the others while p + 1 is eliminated.  Blocks p < R < C are never read
// before their row starts from zero and are left alone.  Two barriers a block column; the chain of 16 pivots a block (reciprocal,
// broadcast, multiply-add) is what bounds it.  Three at a time, kb = 128: 114 us with one column and one barrier at a time, 50 so; kb = 32:
// 25 and 13.6.
// W: the matrix, or the partial sums of `parts` ranges (their triangle on and below the diagonal), added in order.
// Out: Rinv[kb, kb] fp32 = Lc^-1 (lower triangular), so that Rinv Y has orthonormal rows when the shift is
// negligible.  With `check` set (the last pass, whose input should already be near orthonormal) the kernel returns the
// identity at once when W is the identity to 1e-5, and a pivot below 1/4 raises the flag: the block has no full
// rank.  A non-positive pivot always raises it.
__global__ __launch_bounds__(1024) void chol_inv_kernel(const double *W, int parts, int kb, double shift_rel, int check,
                                                         float *Rinv, int *flag, long long zw, long long zflag) {
  W = in_slot(W, zw);
  Rinv = in_slot(Rinv, zw);
  flag = in_slot(flag, zflag);
  extern __shared__ double cs_[];
  const int nb = (kb + 15) / 16, kp = 16 * nb, ld = kp + 4;
  double *const S = cs_;
  __shared__ double redm[16], redd[16], pivs[KB_MAX], invs[2][16];
  const int tid = threadIdx.x, lane = tid & 63, row = lane & 15, g = lane >> 4;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  double dmax = 0.0, dev = 0.0;
  for (int u = tid; u < kp * kp; u += 1024) {
    const int R = u / kp, C = u - R * kp;
    const bool in = R < kb && C < kb;
    const int hi = R < C ? C : R, lo = R < C ? R : C;
    const double *const e = W + (in ? hi * kb + lo : 0);
    double v = *e;
    for (int b = 1; b < parts; ++b) v += e[(long long)b * kb * kb];
    const double one = R == C ? 1.0 : 0.0, x = in ? v : one;
    S[R * ld + C] = x;
    if (in && R == C) dmax = fmax(dmax, v);
    dev = fmax(dev, fabs(x - one));
    if (!(x == x)) dev = INFINITY;
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    dmax = fmax(dmax, __shfl_xor(dmax, o, 64));
    dev = fmax(dev, __shfl_xor(dev, o, 64));
  }
  if (lane == 0) {
    redm[w] = dmax;
    redd[w] = dev;
  }
  __syncthreads();
#pragma unroll
  for (int q = 0; q < 16; ++q) {
    dmax = fmax(dmax, redm[q]);
    dev = fmax(dev, redd[q]);
  }
  // last pass only: rows that are already orthonormal to fp32 level (|W - I| <= 1e-5 everywhere) are left as they are
  if (check && dev <= 1e-5) {                     // the same value in every thread: the whole workgroup leaves together
    for (int u = tid; u < kb * kb; u += 1024) Rinv[u] = u / kb == u % kb ? 1.f : 0.f;
    return;
  }
  const double shift = shift_rel * dmax;
  if (tid < kb) S[tid * ld + tid] += shift;
  __syncthreads();

  // Block column p: wavefront w eliminates the diagonal block and, beside it, the rows of four others, one a group of 16 lanes.  Only wavefront 0
  // writes the diagonal block, and only above its diagonal, where nobody reads it before the next barrier.
  const int panel_waves = max(1, (nb + 2) / 4);
  auto panel = [&](int p) {
    double *const P = S + 16 * p * ld + 16 * p;
    const int o = 4 * w + g, R = o < p ? o : o + 1;
    const bool live = o < nb - 1;
    double *const O = S + (16 * (live ? R : p) + row) * ld + 16 * p;
    double a[16], b[16], piv = 1.0, inv = 1.0;
#pragma unroll
    for (int c = 0; c < 16; ++c) {
      a[c] = c <= row ? P[row * ld + c] : 0.0;    // above the diagonal a row starts from zero
      b[c] = live ? O[c] : 0.0;
    }
    bool bad = false;
    eliminate<0>(a, b, piv, inv, row, check, bad);
    if (bad && lane == 0) atomicOr(flag, 2);
    if (live) {
#pragma unroll
      for (int c = 0; c < 16; ++c) O[c] = b[c];
    }
    if (w == 0 && g == 0) {
#pragma unroll
      for (int c = 0; c < 16; ++c)
        if (c > row) P[row * ld + c] = a[c];
      pivs[16 * p + row] = piv;
      invs[p & 1][row] = inv;
    }
  };
  // the 16 columns of block column p taken from block (R, C), C > p
  auto update = [&](int R, int C, int p) {
    const double *const m = S + (16 * R + row) * ld + 16 * p, *const c = S + (16 * C + row) * ld + 16 * p;
    double *const B = S + 16 * R * ld + 16 * C + row;
    f64x4 acc = {0.0, 0.0, 0.0, 0.0};             // block row p starts from zero
    if (R != p) {
#pragma unroll
      for (int i = 0; i < 4; ++i) acc[i] = B[(g + 4 * i) * ld];
    }
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int k = g + 4 * e;
      double x = m[k];
      if (R == p) x = k < row ? 0.0 : k == row ? 1.0 : x;
      acc = __builtin_amdgcn_mfma_f64_16x16x4f64(-x, c[k] * invs[p & 1][k], acc, 0, 0, 0);
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) B[(g + 4 * i) * ld] = acc[i];
  };
  for (int p = 0;; ++p) {
    if (w < panel_waves) {
      panel(p);
    } else if (p > 0) {                           // block column p - 1 from the columns C = p + 1 + i: of each the rows up to p - 1 and from C on
      int u = w - panel_waves;
      for (int i = 0; i + p + 1 < nb; ++i) {
        for (; u < nb - 1 - i; u += 16 - panel_waves) update(u < p ? u : u + i + 1, p + 1 + i, p - 1);
        u -= nb - 1 - i;
      }
    }
    __syncthreads();
    if (p + 1 == nb) break;
    if (w < nb) update(w, p + 1, p);
    __syncthreads();
  }
  // S[R][C] with R < C is r_CR: row C of the inverse; everything above the diagonal of Rinv is zero
  for (int C = w; C < kb; C += 16) {
    const double root = sqrt(pivs[C]);
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int R = lane + 64 * h;
      float v = 0.f;
      if (64 * h <= C) v = R < C ? (float)(S[min(R, kp - 1) * ld + C] / root) : R == C ? (float)(1.0 / root) : 0.f;
      if (R < kb) Rinv[C * kb + R] = v;
    }
  }
}

// ------------------------------------------------------------------------------- Rayleigh-Ritz (Jacobi)
// sum over each row of 16 lanes, every lane receiving it: four butterfly steps on the data-parallel-primitive paths
// (quad permutes, mirror within 8, mirror within 16), no LDS traffic.  All lanes of a row add the same pairs in the
// same tree, so they hold bitwise the same result.
template <int CTRL>
__device__ __forceinline__ double dpp_move(double v) {
  int lo = __double2loint(v), hi = __double2hiint(v);
  lo = __builtin_amdgcn_update_dpp(0, lo, CTRL, 0xF, 0xF, true);
  hi = __builtin_amdgcn_update_dpp(0, hi, CTRL, 0xF, 0xF, true);
  return __hiloint2double(hi, lo);
}
__device__ __forceinline__ double row16_sum(double v) {
  v += dpp_move<0xB1>(v);    // quad_perm [1, 0, 3, 2]
  v += dpp_move<0x4E>(v);    // quad_perm [2, 3, 0, 1]
  v += dpp_move<0x141>(v);   // row_half_mirror
  v += dpp_move<0x140>(v);   // row_mirror
  return v;
}

// Eigenvectors of the symmetric positive semi-definite T[kb, kb] (fp64) by one-sided Jacobi rotations on the rows of
// a copy M of T (LDS): rotations from the left make the rows mutually orthogonal; then row j = lambda_j v_j^T.  The
// kb / 2 pairs of a round are disjoint (round-robin schedule) and rotate concurrently, one pair per row of 16 lanes (as many
// as there are pairs, in whole wavefronts), lane e holding elements e, e + 16, ....  The squared row norms are carried along (a
// rotation by tangent t moves t * <x, y> from one to the other) and recomputed at the start of every sweep, so a pair
// costs one reduction.  Rows whose norm is below 10^-11 of the largest are rounding noise and are left alone.  Out:
// the k eigenvectors of largest eigenvalue as rows of Wk[k, kb], sigma[k] = lambda^1/2 (descending) and inv_sigma[k] =
// lambda^-1/2 (0 where lambda = 0).
//
// What bounds it: the length of a round (read, reduce, rotation, write, barrier), kb - 1 of them in each of about nine sweeps; at kb = 128 also
// the vector instructions of sixteen wavefronts.  So there are no wavefronts without a pair, no chunks beyond kb, no remainder by
// kb - 1 (its division was a third of the chain) and no square root in the test.  kb = 32: 181 -> 107 us, 128: 1664 -> 1572, same bits.
// (Two reciprocal square roots in place of the rotation's four steps: 86 and 1340, but other last bits, which move labels.  Eight lanes a pair
// instead of sixteen, half the scalar part: a third slower at 64 and at 128.)
template <int NC>      // chunks of 16 elements a row
__global__ __launch_bounds__(NC <= 2 ? 256 : NC <= 4 ? 512 : 1024) void jacobi_kernel(const double *T, int kb, int k, int max_sweeps, float *Wk,
                                                       float *inv_sigma, float *sigma, long long zw, long long zsigma) {
  T = in_slot(T, zw);
  Wk = in_slot(Wk, zw);
  inv_sigma = in_slot(inv_sigma, zw);
  sigma = in_slot(sigma, zsigma);
  extern __shared__ double Ms[];
  __shared__ int rotated;
  __shared__ double nrm2[KB_MAX];
  __shared__ double amax;
  const int tid = threadIdx.x, e = tid & 15, grp = tid >> 4, threads = blockDim.x, groups = threads >> 4;
  const int ldm = kb + 2;
  for (int u = tid; u < kb * kb; u += threads) {
    const int i = u / kb, j = u % kb;
    Ms[i * ldm + j] = 0.5 * (T[i * kb + j] + T[j * kb + i]);
  }
  if (tid == 0) rotated = 0;
  __syncthreads();
  const int half = kb / 2, ring = kb - 1;
  for (int sweep = 0; sweep <= max_sweeps; ++sweep) {
    for (int j = grp; j < kb; j += groups) {
      double s = 0.0;
      for (int c = e; c < kb; c += 16) {
        const double x = Ms[j * ldm + c];
        s = fma(x, x, s);
      }
      s = row16_sum(s);
      if (e == 0) nrm2[j] = s;
    }
    __syncthreads();
    if (sweep == max_sweeps) break;       // the norms are exact again: ready for the ranking below
    if (tid < 64) {
      double m = tid < kb ? nrm2[tid] : 0.0;
      if (tid + 64 < kb) m = fmax(m, nrm2[tid + 64]);
#pragma unroll
      for (int o = 32; o > 0; o >>= 1) m = fmax(m, __shfl_xor(m, o, 64));
      if (tid == 0) amax = fmax(m, 0.0);
    }
    __syncthreads();
    const double floor2 = 1e-22 * amax;
    for (int round = 0; round < ring; ++round) {
      // all 64 lanes of a wavefront run the reduction (the 16-lane groups without a pair add zeros)
      const bool live = grp < half;
      const int pr = live ? grp : 0;
      const int up = round + pr, down = round - pr;             // modulo ring
      const int a = up >= ring ? up - ring : up, b = pr == 0 ? ring : down < 0 ? down + ring : down;
      double *ra = Ms + a * ldm, *rb = Ms + b * ldm;
      double x[NC], y[NC];
      double ga = 0.0;
#pragma unroll
      for (int i = 0; i < NC; ++i) {
        const int c = e + 16 * i;
        const bool ok = live && c < kb;
        x[i] = ok ? ra[c] : 0.0;
        y[i] = ok ? rb[c] : 0.0;
        ga = fma(x[i], y[i], ga);
      }
      ga = row16_sum(ga);
      const double al = nrm2[a], be = nrm2[b];
      // |<x, y>| > 1e-11 |x| |y|, by its square where that is certain to decide alike
      const double sq = ga * ga, lim = 1e-22 * (al * be);
      bool turn = sq > lim;
      if (!(fabs(sq - lim) > 1e-12 * lim && lim > 1e-280 && lim < 1e280)) turn = fabs(ga) > 1e-11 * sqrt(al * be);
      if (live && fmin(al, be) > floor2 && turn) {
        // the rotation from hardware reciprocal / reciprocal-square-root estimates refined by Newton steps: a correctly rounded
        // division and square root cost several times the rest of the round, and any (c, s) with c^2 + s^2 = 1 to rounding keeps the
        // rows' span; the sweeps converge on the same vectors, but a formula of other roundings ends on other last bits
        // and so on other labels
        const double zeta = (be - al) * nr_rcp(2.0 * ga);
        const double h2 = fma(zeta, zeta, 1.0);
        const double tt = copysign(1.0, zeta) * nr_rcp(fabs(zeta) + h2 * nr_rsq(h2));
        const double c_ = nr_rsq(fma(tt, tt, 1.0)), s_ = c_ * tt;
#pragma unroll
        for (int i = 0; i < NC; ++i) {
          const int c = e + 16 * i;
          if (c < kb) {
            ra[c] = c_ * x[i] - s_ * y[i];
            rb[c] = s_ * x[i] + c_ * y[i];
          }
        }
        if (e == 0) {
          nrm2[a] = al - tt * ga;
          nrm2[b] = be + tt * ga;
          rotated = 1;
        }
      }
      __syncthreads();
    }
    const int any = rotated;
    __syncthreads();
    if (tid == 0) rotated = 0;
    __syncthreads();
    if (!any) break;                      // nothing moved in this sweep: the carried norms are the exact ones
  }
  __syncthreads();
  // eigenvalues = row norms; rank them (descending, ties to the lower row)
  for (int j = grp; j < kb; j += groups) {
    int rank = 0;
    const double mine = nrm2[j] > 0.0 ? nrm2[j] : 0.0;
    for (int i = 0; i < kb; ++i) {
      const double o = nrm2[i] > 0.0 ? nrm2[i] : 0.0;
      rank += (o > mine || (o == mine && i < j)) ? 1 : 0;
    }
    if (rank < k) {
      const double lam = sqrt(mine);
      const double inv = lam > 0.0 ? 1.0 / lam : 0.0;
      for (int c = e; c < kb; c += 16) Wk[rank * kb + c] = (float)(Ms[j * ldm + c] * inv);
      if (e == 0) {
        sigma[rank] = (float)sqrt(lam);
        inv_sigma[rank] = lam > 0.0 ? (float)(1.0 / sqrt(lam)) : 0.f;
      }
    }
  }
}

// ------------------------------------------------------------------------------------------------- k-means
__device__ __forceinline__ int clamp_label(int v, int k) { return v < 0 ? 0 : (v >= k ? k - 1 : v); }

__global__ __launch_bounds__(256) void kmeans_init_kernel(const float *U, int N, int d, int k, const int *init_idx,
                                                          float *centres, int *flag, long long zu, long long zinit,
                                                          long long zflag) {
  U = in_slot(U, zu);
  init_idx = in_slot(init_idx, zinit);
  centres = in_slot(centres, zu);
  flag = in_slot(flag, zflag);
  const int c = blockIdx.x;
  int r = init_idx[c];
  if (r < 0 || r >= N) {
    if (threadIdx.x == 0) atomicOr(flag, 1);
    r = 0;
  }
  for (int j = threadIdx.x; j < d; j += 256) centres[c * d + j] = U[(long long)r * d + j];
}

// Control words of one k-means run (device, ints): KM_COUNT + it % 3 = labels changed by pass it, KM_DONE = 1 once a pass has
// changed nothing, KM_PASSES = assignment passes run.  Every kernel of a pass leaves at once
// when KM_DONE is up, so the host may enqueue passes ahead of knowing whether they are needed.  Three counters: while pass
// it adds to its own, it reads that of pass it - 1 and clears that of pass it + 1, which was last read in pass it - 1.
constexpr int KM_DONE = 2, KM_PASSES = 3, KM_COUNT = 4;

// Pass `it`: assignment, and the sums of the clusters it touched.  One workgroup = one range of rows (rows_per of them, taken in
// batches of KM_ROWS), the centres in LDS (rows of 16 NC + 4 floats, zeros behind the d-th).
//
// Assignment.  The label of a row u is the centre c with the least s(c) = sum (u_j - c_j)^2, a chain of float32 multiply-adds
// over ascending j, ties to the lowest centre.  The products u . c of 16 rows and 16 centres at a time come from the float32 matrix
// cores (fragments 16 c + 4 g + u of both operands, so 16-byte reads), which gives D(c) = |c|^2 - 2 u . c.  With
// K = (5 d + 16) 2^-24, D(c) and s(c) - |u|^2 are within K (|u|^2 + |c|^2) of each other: 2^-23 d (|u|^2 + |c|^2) for the products
// (half a unit more than round to nearest per step), (d + 4) 2^-24 (..) for |c|^2 and the last addition, (d + 3) 2^-24 |u - c|^2 for
// the chain.  So the least D(c) names the label when every other D(c) (1 - K) lies above it by 2 K (|u|^2 + |c|^2) and more; the other
// rows (ties, NaN and infinities among them) are queued and a wavefront evaluates s(c) itself for each, a centre a lane.  On the
// embedding of a pool of 32768 samples in 100 dimensions fewer than one row in a thousand is queued.
//
// Sums.  A range whose labels stay as they were keeps its sums from the last pass; so do the clusters of a changed range that no
// row entered or left.  Wavefront w takes the clusters w, w + 8, ...: the rows of a cluster come out of a ballot in ascending
// order, lane l adds dimensions l and l + 64 in float64 in that order.  pcnt = 0 stands for sums that were never written.
//
// Three subsamples of 32768 rows, 100 centres in 100 dimensions: 83 us in the first pass, 42 in the late ones, where one
// subsample took 48 for an assignment on the vector units and 32 for sums by LDS atomics.  The products are what is left:
// 392 instructions of 32 cycles a wavefront, on 384 workgroups, so half the compute units have two.
constexpr int KM_ROWS = 256;
// Up to 16 KM_STAGE_NC dimensions, the rows of a range of one batch stay in LDS for the sums, whose chains of eight rows a round trip were
// the longest part of a pass.  k-means of 500 to 65536 samples, 2 to 16 dimensions, 2 to 128 clusters, 16 passes: 2 - 10 % faster (1536
// samples, 8 of each 290 -> 270 us; 32768 446 -> 436).  With 17 to 32 dimensions too nothing gained, with 33 to 48 1 % slower; with the rows
// requested in front of the centres, beside the loads of the sums, 32768 samples took 5 % longer.
constexpr int KM_STAGE_NC = 1;
typedef float kmv4 __attribute__((ext_vector_type(4)));

// `own` (it > 0, no kmeans_finish_kernel in between): every workgroup starts from the sums of the pass before and forms the centres
// itself, with the arithmetic of that kernel.  A cluster that has become empty keeps the centre that workgroup 0 has put to memory in an
// earlier pass (it writes those that are not empty, the others are only read).
//
// Nothing orders the workgroups of a launch: beside other work one may start after another has ended.  So, where passes are `own`,
// no location that a workgroup of the launch reads is written by another one in it: a pass reads the sums and counts of the pass before
// (psum_in, pcnt_in) and writes all of its range's to the other of two copies (psum, pcnt), the ones that it keeps copied over; a centre is
// either read by all (its cluster is empty) or written by workgroup 0 (it is not), and which of the two follows from the counts
// of the pass before; labels are each range's own; the control words are read as said above, `dirty` is only set.  Without `own` the
// two copies are one (psum_in == psum), which a workgroup reads and writes in its own range alone.
template <int NC, bool V4, bool STAGE>
__global__ __launch_bounds__(512) void kmeans_pass_kernel(const float *U, int N, int d, float *centres, int k, int rows_per,
                                                          int *labels, const double *psum_in, const int *pcnt_in, double *psum, int *pcnt,
                                                          int *dirty, int *ctl, int it, int own,
                                                          long long zu, long long zlab, long long zw, long long zctl) {
  ctl = in_slot(ctl, zctl);
  if (ctl[KM_DONE]) return;
  if (own && ctl[KM_COUNT + (it - 1) % 3] == 0) {           // the pass before changed nothing
    if (blockIdx.x == 0 && threadIdx.x == 0) ctl[KM_DONE] = 1;
    return;
  }
  if (blockIdx.x == 0 && threadIdx.x == 0) ctl[KM_COUNT + (it + 1) % 3] = 0;
  U = in_slot(U, zu);
  centres = in_slot(centres, zu);
  labels = in_slot(labels, zlab);
  const bool copies = psum_in != psum && it > 0;            // (the first pass keeps nothing)
  psum_in = in_slot(psum_in, zw);
  pcnt_in = in_slot(pcnt_in, zw);
  psum = in_slot(psum, zw);
  pcnt = in_slot(pcnt, zw);
  dirty = in_slot(dirty, zw);
  constexpr int DP = 16 * NC, S = DP + 4, NW = 8;
  extern __shared__ float sm[];
  const int k16 = (k + 15) & ~15;
  float *const cs = sm, *const cn = sm + k16 * S;
  float *const us = cn + k16;                     // STAGE: the rows of the range, laid out as the centres
  __shared__ int lab_s[KM_ROWS], queue[KM_ROWS], queued, changed, touched[KB_MAX];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, ql = lane & 15, g = lane >> 4;
  const float kappa = (float)(5 * d + 16) * 5.9604645e-8f;
  if (blockIdx.x == 0 && tid == 0) atomicAdd(&ctl[KM_PASSES], 1);
  if (tid == 0) {
    queued = 0;
    changed = 0;
  }
  if (tid < KB_MAX) touched[tid] = it == 0;       // the first pass writes every count
  // The sums and counts of before go to this pass's copy at once; the clusters that turn out to be touched are written again below, barriers
  // later (so that their loads lie beside the others: at the end, for the kept ones alone, a clustering of 1536 samples is 2 % slower).
  double *const ps = psum + (long long)blockIdx.x * k * d;
  if (copies && tid < k) pcnt[blockIdx.x * k + tid] = pcnt_in[blockIdx.x * k + tid];
  for (int u = tid; u < k16 * DP; u += 512) {
    const int c = u / DP, j = u - c * DP;
    const bool in = c < k && j < d;
    const double kept = copies && in ? psum_in[((long long)blockIdx.x * k + c) * d + j] : 0.0;
    float v = 0.f;
    bool stored = in;                             // the centre is the one in memory
    if (own && in) {
      double tot = 0.0;
      int m = 0;
      constexpr int AHEAD = 16;                   // that many ranges' loads in flight
      for (int b = 0; b < (int)gridDim.x; b += AHEAD) {
        double t[AHEAD];
        int q[AHEAD];
#pragma unroll
        for (int i = 0; i < AHEAD; ++i) {
          const int bb = min(b + i, (int)gridDim.x - 1);
          q[i] = pcnt_in[bb * k + c];
          t[i] = psum_in[((long long)bb * k + c) * d + j];
        }
        // (a count of 0: sums of an earlier pass, or none)  Up to 16 dimensions, the additions are selects behind all loads.  The compiler may make
        // a branch of each otherwise, or of the first sum's load, which then is a round trip of its own (a pass of 128 ranges 23 -> 25 us, of 256
        // 51 -> 56).  With more dimensions the selects' masks spill scalar registers, which passes that are not `own` pay for too: 300000 samples
        // of 24 1.5 % slower.
        if constexpr (NC == 1) {
          asm volatile("" ::: "memory");
#pragma unroll
          for (int i = 0; i < AHEAD; ++i) {
            const bool have = b + i < (int)gridDim.x && q[i] > 0;
            tot += have ? t[i] : 0.0;
            m += have ? q[i] : 0;
          }
        } else {
#pragma unroll
          for (int i = 0; i < AHEAD; ++i)
            if (b + i < (int)gridDim.x && q[i] > 0) {
              tot += t[i];
              m += q[i];
            }
        }
      }
      stored = m <= 0;
      if (!stored) {
        v = (float)(tot / (double)m);
        if (blockIdx.x == 0) centres[c * d + j] = v;
      }
    }
    if (stored) v = centres[c * d + j];
    if (copies && in) ps[c * d + j] = kept;
    cs[c * S + j] = v;
  }
  __syncthreads();
  {
    const int c = tid >> 2, q = tid & 3;          // four lanes a centre
    float s = 0.f;
    if (c < k16)
#pragma unroll
      for (int i = 0; i < NC; ++i) {
        const kmv4 v = *(const kmv4 *)(cs + c * S + 16 * i + 4 * q);
        s = fmaf(v[0], v[0], s);
        s = fmaf(v[1], v[1], s);
        s = fmaf(v[2], v[2], s);
        s = fmaf(v[3], v[3], s);
      }
    s += __shfl_xor(s, 1, 64);
    s += __shfl_xor(s, 2, 64);
    if (c < k16 && q == 0) cn[c] = c < k ? s * (1.f - kappa) : INFINITY;
  }
  __syncthreads();

  const int r0 = blockIdx.x * rows_per, r1 = min(N, r0 + rows_per);
  for (int b0 = r0; b0 < r1; b0 += KM_ROWS) {
    kmv4 uf[2][NC];
    float un[2], v1[2], v2[2];
    int i1[2];
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      const float *u = U + (long long)min(b0 + wave * 32 + 16 * j + ql, N - 1) * d;
#pragma unroll
      for (int c = 0; c < NC; ++c) {
        const int f = 16 * c + 4 * g;
        if (V4) {
          const kmv4 v = *(const kmv4 *)(u + min(f, d - 4));
          uf[j][c] = f < d ? v : (kmv4){0.f, 0.f, 0.f, 0.f};
        } else {
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const float v = u[min(f + e, d - 1)];
            uf[j][c][e] = f + e < d ? v : 0.f;
          }
        }
        if constexpr (STAGE) *(kmv4 *)(us + (wave * 32 + 16 * j + ql) * S + f) = uf[j][c];
      }
    }
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      float s = 0.f;
#pragma unroll
      for (int c = 0; c < NC; ++c)
#pragma unroll
        for (int e = 0; e < 4; ++e) s = fmaf(uf[j][c][e], uf[j][c][e], s);
      s += __shfl_xor(s, 16, 64);
      s += __shfl_xor(s, 32, 64);
      un[j] = s;
      v1[j] = v2[j] = INFINITY;
      i1[j] = 0x7fffffff;
    }
    for (int kt = 0; kt < k16; kt += 16) {
      kmv4 acc[2] = {{0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}};
#pragma unroll
      for (int c = 0; c < NC; ++c) {
        const kmv4 kf = *(const kmv4 *)(cs + (kt + ql) * S + 16 * c + 4 * g);
#pragma unroll
        for (int e = 0; e < 4; ++e)
#pragma unroll
          for (int j = 0; j < 2; ++j) acc[j] = __builtin_amdgcn_mfma_f32_16x16x4f32(kf[e], uf[j][c][e], acc[j], 0, 0, 0);
      }
      const kmv4 c4 = *(const kmv4 *)(cn + kt + 4 * g);
#pragma unroll
      for (int j = 0; j < 2; ++j)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const float v = fmaf(-2.f, acc[j][r], c4[r]);
          const bool less = v < v1[j];
          v2[j] = less ? v1[j] : fminf(v2[j], v);
          i1[j] = less ? kt + 4 * g + r : i1[j];
          v1[j] = less ? v : v1[j];
        }
    }
#pragma unroll
    for (int j = 0; j < 2; ++j) {
#pragma unroll
      for (int o = 16; o <= 32; o <<= 1) {
        const float a1 = __shfl_xor(v1[j], o, 64), a2 = __shfl_xor(v2[j], o, 64);
        const int ai = __shfl_xor(i1[j], o, 64);
        const bool other = a1 < v1[j] || (a1 == v1[j] && ai < i1[j]);
        v2[j] = fminf(other ? v1[j] : v2[j], other ? a2 : a1);
        v1[j] = other ? a1 : v1[j];
        i1[j] = other ? ai : i1[j];
      }
      const int rr = wave * 32 + 16 * j + ql;
      if (g == 0 && b0 + rr < r1) {
        const float cb = i1[j] < k ? cn[i1[j]] : INFINITY;
        if (v2[j] - v1[j] > 2.2f * kappa * (cb + un[j]) + 1e-34f) lab_s[rr] = i1[j];
        else queue[atomicAdd(&queued, 1)] = rr;
      }
    }
    __syncthreads();
    for (int q = wave; q < queued; q += NW) {
      const int rr = queue[q];
      const float *u = U + (long long)(b0 + rr) * d;
      const float *ca = cs + (lane < k ? lane : 0) * S, *cb = cs + (lane + 64 < k ? lane + 64 : 0) * S;
      float sa = 0.f, sb = 0.f;
      for (int j = 0; j < d; ++j) {
        const float v = u[j], ta = v - ca[j], tb = v - cb[j];
        sa = fmaf(ta, ta, sa);
        sb = fmaf(tb, tb, sb);
      }
      float best = INFINITY;
      int besti = 0x7fffffff;
      if (lane < k && sa < best) { best = sa; besti = lane; }
      if (lane + 64 < k && sb < best) { best = sb; besti = lane + 64; }
#pragma unroll
      for (int o = 1; o < 64; o <<= 1) {
        const float s = __shfl_xor(best, o, 64);
        const int c = __shfl_xor(besti, o, 64);
        if (s < best || (s == best && c < besti)) { best = s; besti = c; }
      }
      if (lane == 0) lab_s[rr] = besti;
    }
    __syncthreads();
    bool moved = false;
    if (tid < KM_ROWS && b0 + tid < r1) {
      const int was = labels[b0 + tid], is = lab_s[tid];
      moved = was != is;
      if (moved) {
        labels[b0 + tid] = is;
        touched[clamp_label(is, k)] = 1;
        if (was >= 0) touched[clamp_label(was, k)] = 1;
      }
    }
    const int n = (int)__popcll(__builtin_amdgcn_ballot_w64(moved));
    if (n && lane == 0) {
      atomicAdd(&ctl[KM_COUNT + it % 3], n);
      changed = 1;
    }
    if (tid == 0) queued = 0;
    __syncthreads();                              // before the next batch queues rows and writes labels
  }
  if (!changed) return;                           // the same value in every thread

  for (int c = wave; c < k; c += NW) {
    if (!touched[c]) continue;
    double s0 = 0.0, s1 = 0.0;
    int count = 0;
    const int ja = min(lane, d - 1), jb = min(lane + 64, d - 1);
    for (int b0 = r0; b0 < r1; b0 += KM_ROWS) {
#pragma unroll
      for (int q = 0; q < KM_ROWS / 64; ++q) {
        const int row = b0 + 64 * q + lane;
        const int l = b0 == r0 && r1 - r0 <= KM_ROWS ? lab_s[64 * q + lane] : labels[min(row, r1 - 1)];
        unsigned long long rows = __builtin_amdgcn_ballot_w64(row < r1 && clamp_label(l, k) == c);
        count += (int)__popcll(rows);
        const float *base = U + (long long)(b0 + 64 * q) * d;
        while (rows) {                            // eight rows at a time (the last one repeated), added in ascending order
          float a[8], b[8];
          int have = 0;
#pragma unroll
          for (int i = 0; i < 8; ++i) {
            const int r = (int)__builtin_ctzll(rows);
            if constexpr (STAGE) {
              a[i] = us[(64 * q + r) * S + ja];
            } else {
              a[i] = base[(long long)r * d + ja];
              b[i] = base[(long long)r * d + jb];
            }
            have = i + 1;
            const unsigned long long rest = rows & (rows - 1);
            if (!rest) { rows = 0; break; }
            rows = rest;
          }
#pragma unroll
          for (int i = 0; i < 8; ++i)
            if (i < have) {
              s0 += (double)a[i];
              if constexpr (!STAGE) s1 += (double)b[i];
            }
        }
      }
    }
    if (count) {
      if (lane < d) ps[c * d + lane] = s0;
      if (lane + 64 < d) ps[c * d + lane + 64] = s1;
    }
    if (lane == 0) {
      pcnt[blockIdx.x * k + c] = count;
      dirty[c] = 1;
    }
  }
}

// New centres of the clusters touched since this kernel last ran, one workgroup each: the ranges' sums added in order (an empty cluster
// keeps its centre); a pass `it` that changed nothing raises KM_DONE.
__global__ __launch_bounds__(128) void kmeans_finish_kernel(const double *psum, const int *pcnt, int nb, int k, int d,
                                                           float *centres, int *dirty, int *ctl, int it, long long zu, long long zw,
                                                           long long zctl) {
  ctl = in_slot(ctl, zctl);
  if (ctl[KM_DONE]) return;
  psum = in_slot(psum, zw);
  pcnt = in_slot(pcnt, zw);
  dirty = in_slot(dirty, zw);
  centres = in_slot(centres, zu);
  if (ctl[KM_COUNT + it % 3] == 0) {
    if (blockIdx.x == 0 && threadIdx.x == 0) ctl[KM_DONE] = 1;
    return;
  }
  const int c = blockIdx.x, j = threadIdx.x;
  if (!dirty[c]) return;
  __syncthreads();
  if (j == 0) dirty[c] = 0;
  if (j >= d) return;
  double tot = 0.0;
  int m = 0;
  constexpr int AHEAD = 32;
  for (int b = 0; b < nb; b += AHEAD) {
    double t[AHEAD];
    int q[AHEAD];
#pragma unroll
    for (int i = 0; i < AHEAD; ++i) {
      const int bb = min(b + i, nb - 1);
      q[i] = pcnt[bb * k + c];
      t[i] = psum[((long long)bb * k + c) * d + j];
    }
#pragma unroll
    for (int i = 0; i < AHEAD; ++i)
      if (b + i < nb && q[i] > 0) {               // a count of 0: sums of an earlier pass, or none
        tot += t[i];
        m += q[i];
      }
  }
  if (m > 0) centres[c * d + j] = (float)(tot / (double)m);
}

// ---------------------------------------------------------------------------------------------- aggregation
__global__ __launch_bounds__(256) void contingency_kernel(const int *a, const int *b, int N, int k, int *T) {
  const int r = blockIdx.x * 256 + threadIdx.x;
  if (r < N) atomicAdd(&T[clamp_label(a[r], k) * k + clamp_label(b[r], k)], 1);
}

// Greedy renaming, one workgroup: take the largest remaining count (ties to the lowest flat index), fix perm[column] = row, retire the
// row and the column, and so on.  Count and index make one 64-bit key, (count << 32) | (2^31 - 1 - flat index), so no two entries
// are equal (within a row or a column the position there will do), and then an entry that is the largest of its row and of its column among the live ones is taken by the greedy order whatever
// else is in the table: nothing that could retire its row or column comes before it.  So a round takes all such entries at once (the
// largest of the table is one of them, so there are at most k rounds: a handful for counts that differ, nearly k where most are equal and
// small), and only rows and columns whose partner has retired look again.  Table in LDS, eight lanes a row, then eight lanes a column.
// A round is bound by its LDS round trips and barriers, 1 us.  One entry a round, all keys in registers, one barrier: 16 us at 8 labels,
// 170 at 100, whatever the table.  Here 5 at 8; at 100 it depends on the table: 92 - 118 for pools whose subsamples agree for the most part, 180
// for one without such classes, where the counts are small and most of them equal.
__device__ __forceinline__ long long max8(long long m) {          // over eight adjacent lanes
#pragma unroll
  for (int o = 1; o < 8; o <<= 1) {
    const long long x = __shfl_xor(m, o, 64);
    m = x > m ? x : m;
  }
  return m;
}
__global__ __launch_bounds__(1024) void greedy_match_kernel(const int *T, int k, int *perm) {
  extern __shared__ int gt_[];                    // [k][k + 1]
  __shared__ int row_best[KB_MAX], col_best[KB_MAX], left;        // column of a row's largest, row of a column's; -1: retired
  const int tid = threadIdx.x, l = tid & 7, me = tid >> 3, ld = k + 1;
  for (int u = tid; u < k * k; u += 1024) gt_[u / k * ld + u % k] = T[u];
  if (tid < KB_MAX) row_best[tid] = col_best[tid] = tid < k ? 0 : -1;
  if (tid == 0) left = k;
  __syncthreads();
  for (bool first = true; left > 0; first = false) {          // `left`: the same in every thread, written behind a barrier, before one
    long long mr = -1, mc = -1;
    // a largest entry stays what it is until its partner retires
    const int rb = me < k ? row_best[me] : -1, cb = me < k ? col_best[me] : -1;
    const bool row = rb >= 0 && (first || col_best[rb] < 0), col = cb >= 0 && (first || row_best[cb] < 0);
    if (row) {
      int v = -1, at = 0;
      for (int c0 = l; c0 < k; c0 += 64) {          // eight pairs of reads in flight
        int t[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) {
          const int cc = min(c0 + 8 * i, k - 1), e = gt_[me * ld + cc];
          t[i] = c0 + 8 * i < k && col_best[cc] >= 0 ? e : -1;
        }
#pragma unroll
        for (int i = 0; i < 8; ++i) {
          at = t[i] > v ? c0 + 8 * i : at;
          v = t[i] > v ? t[i] : v;
        }
      }
      if (v >= 0) mr = ((long long)v << 32) | (long long)(unsigned)(0x7fffffff - at);
    }
    if (col) {
      int v = -1, at = 0;
      for (int c0 = l; c0 < k; c0 += 64) {          // eight pairs of reads in flight
        int t[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) {
          const int cc = min(c0 + 8 * i, k - 1), e = gt_[cc * ld + me];
          t[i] = c0 + 8 * i < k && row_best[cc] >= 0 ? e : -1;
        }
#pragma unroll
        for (int i = 0; i < 8; ++i) {
          at = t[i] > v ? c0 + 8 * i : at;
          v = t[i] > v ? t[i] : v;
        }
      }
      if (v >= 0) mc = ((long long)v << 32) | (long long)(unsigned)(0x7fffffff - at);
    }
    mr = max8(mr);
    mc = max8(mc);
    __syncthreads();                              // everyone has read what is live
    if (me < k && l == 0) {
      if (mr >= 0) row_best[me] = 0x7fffffff - (int)(unsigned)(mr & 0xffffffffll);
      if (mc >= 0) col_best[me] = 0x7fffffff - (int)(unsigned)(mc & 0xffffffffll);
    }
    __syncthreads();
    const int q = tid < k ? row_best[tid] : -1;
    const bool take = q >= 0 && col_best[q] == tid;
    __syncthreads();
    if (take) {
      perm[q] = tid;
      row_best[tid] = -1;
      col_best[q] = -1;
      atomicSub(&left, 1);
    }
    __syncthreads();
  }
}

__global__ __launch_bounds__(256) void identity_perm_kernel(int *perm, int k) {
  const int i = blockIdx.x * 256 + threadIdx.x;
  if (i < k) perm[i] = i;
}

__global__ __launch_bounds__(256) void vote_kernel(const int *labels, const int *perm, int m, int N, int k, int *out) {
  const int r = blockIdx.x * 256 + threadIdx.x;
  if (r >= N) return;
  int name[M_MAX];
  for (int i = 0; i < m; ++i) name[i] = perm[i * k + clamp_label(labels[(long long)i * N + r], k)];
  int best = 0, pick = name[0];
  for (int i = 0; i < m; ++i) {
    int votes = 0;
    for (int q = 0; q < m; ++q) votes += name[q] == name[i] ? 1 : 0;
    if (votes > best) {      // strict: the earliest vector among the most frequent names wins
      best = votes;
      pick = name[i];
    }
  }
  out[r] = pick;
}

// ------------------------------------------------------------------------------------------- host side
struct Carve {
  char *base;
  size_t off = 0;
  explicit Carve(void *b) : base(static_cast<char *>(b)) {}
  template <class T>
  T *take(size_t count) {
    off = (off + 255) & ~size_t(255);
    T *p = base ? reinterpret_cast<T *>(base + off) : nullptr;
    off += count * sizeof(T);
    return p;
  }
};

// element ranges of the partial Gram matrices: at most 128 of them, whole multiples of the 32 elements that a workgroup takes at a time
int gram_chunk(int len) { return (((len + 127) / 128) + 31) / 32 * 32; }
int gram_parts(int len) { return (len + gram_chunk(len) - 1) / gram_chunk(len); }

// row ranges of the k-means partial sums: at most 256 of them, at least 256 rows each
int kmeans_rows_per(int N) {
  const int r = (N + 255) / 256;
  return r < 256 ? 256 : r;
}
int kmeans_blocks(int N) { return (N + kmeans_rows_per(N) - 1) / kmeans_rows_per(N); }
// A pass forms its centres itself, a launch less, where every workgroup can read all sums in a few round trips: the whole clustering is
// 3 - 6 % faster up to 9216 sums (1536 samples, 8 clusters 842 -> 815 us; 4000, 16: 1355 -> 1276; 4000, 24: 1780 -> 1731), 4 - 5 % slower at
// 13800 and 18400.
constexpr long long KM_OWN = 10240;
bool kmeans_own(int N, int d, int k) { return (long long)kmeans_blocks(N) * k * d <= KM_OWN; }

struct SimWork {
  float *rinv, *Xs, *cs, *tc;
  double *colpart;
  int *flag;
  size_t bytes;
  SimWork(void *w, int N, int F, int n) {
    Carve c(w);
    flag = c.take<int>(64);
    rinv = c.take<float>(N);
    Xs = c.take<float>((size_t)n * F);
    cs = c.take<float>(n);
    tc = c.take<float>(n);
    colpart = c.take<double>((size_t)COL_CHUNKS * n);
    bytes = c.off + 256;
  }
};

struct EmbedWork {
  float *G, *Q, *Y, *Z, *Bm, *Wk, *isig, *Rinv, *spart;
  size_t spart_elems;
  double *part, *W;
  int *flag;
  size_t bytes;
  EmbedWork(void *w, int N, int n, int k, int kb) {
    Carve c(w);
    flag = c.take<int>(64);
    G = c.take<float>((size_t)n * n);
    Q = c.take<float>((size_t)kb * n);
    Y = c.take<float>((size_t)kb * n);
    Z = c.take<float>((size_t)kb * n);
    Bm = c.take<float>((size_t)N * kb);
    Wk = c.take<float>((size_t)k * kb);
    isig = c.take<float>(k);
    Rinv = c.take<float>((size_t)kb * kb);
    spart_elems = (size_t)5 * n * n;
    spart = c.take<float>(spart_elems);
    const int parts = gram_parts(n) > gram_parts(N) ? gram_parts(n) : gram_parts(N);
    part = c.take<double>((size_t)parts * kb * kb);
    W = c.take<double>((size_t)kb * kb);
    bytes = c.off + 256;
  }
};

struct SmallWork {      // k-means (N rows of d dimensions), aggregation, normalisation
  int *flag, *T, *perm, *pcnt, *dirty;
  double *psum;
  size_t count;         // of one copy
  size_t bytes;
  SmallWork(void *w, int N, int d, int k) {
    Carve c(w);
    flag = c.take<int>(64);
    T = c.take<int>((size_t)k * k);
    perm = c.take<int>((size_t)M_MAX * k);
    // two copies of the k-means sums and counts where the passes form the centres (sums: at most 2 KM_OWN then, reserved for larger
    // problems as well, so that a workspace for d dimensions and k clusters also does for fewer)
    count = (size_t)kmeans_blocks(N) * k;
    pcnt = c.take<int>(2 * count);
    dirty = c.take<int>(k);
    psum = c.take<double>(std::max(count * d, std::min(2 * count * d, (size_t)(2 * KM_OWN))));
    bytes = c.off + 256;
  }
};

// rows of the matrices with n columns in the workspace are padded to whole 16-byte loads
int padded(int n) { return (n + 3) & ~3; }

struct ClusterWork {
  float *A, *dr, *dc, *U, *sigma, *centres;
  int *flags;           // [MAX_SLOTS][SLOT_WORDS], those of the group in its first subsample's workspace
  void *sub;            // region handed to the calls above
  size_t sub_bytes, bytes;
  ClusterWork(void *w, int N, int F, int n, int k, int kb) {
    Carve c(w);
    A = c.take<float>((size_t)N * padded(n));
    dr = c.take<float>(N);
    dc = c.take<float>(n);
    U = c.take<float>((size_t)N * k);
    sigma = c.take<float>(k);
    centres = c.take<float>((size_t)k * k);
    flags = c.take<int>(64);
    // the k-means region is sized for rows of up to kb dimensions, so that the one size also covers qc_tap_kmeans
    // on an embedding of the whole iteration block
    size_t s1 = SimWork(nullptr, N, F, n).bytes, s2 = EmbedWork(nullptr, N, padded(n), k, kb).bytes, s3 = SmallWork(nullptr, N, kb, kb).bytes;
    sub_bytes = s1 > s2 ? s1 : s2;
    if (s3 > sub_bytes) sub_bytes = s3;
    sub = c.take<char>(sub_bytes);
    bytes = c.off + 256;
  }
};

int check_dims(int N, int F, int n, int k, int kb) {
  if (N < 1 || F < 1 || n < 1 || k < 1 || kb < 1) TAP_FAIL(QC_ERR_SHAPE, "N, F, n, k, kb must be positive");
  if (kb > KB_MAX || kb % 8) TAP_FAIL(QC_ERR_UNSUPPORTED, "kb must be a multiple of 8 and at most %d (got %d)", KB_MAX, kb);
  if (k > kb) TAP_FAIL(QC_ERR_SHAPE, "k (%d) exceeds kb (%d)", k, kb);
  if (kb > n) TAP_FAIL(QC_ERR_SHAPE, "kb (%d) exceeds the subsample size n (%d)", kb, n);
  if (n > N) TAP_FAIL(QC_ERR_SHAPE, "n (%d) exceeds N (%d)", n, N);
  if ((long long)N * (n > F ? n : F) >= (1ll << 31)) TAP_FAIL(QC_ERR_UNSUPPORTED, "N * max(n, F) must be below 2^31");
  return QC_OK;
}

// reads a device flag word after waiting for the stream
int read_flag(const int *flag, hipStream_t st, int *out) {
  TAP_HIP(hipMemcpyAsync(out, flag, sizeof(int), hipMemcpyDeviceToHost, st));
  TAP_HIP(hipStreamSynchronize(st));
  return QC_OK;
}

// optional timing of the similarity contraction (the dominant kernel) with events on the caller's stream
struct SimProfile {
  bool on = false;
  std::vector<std::pair<hipEvent_t, hipEvent_t>> ev;
  size_t used = 0;
  int products = 0;
};
SimProfile g_prof;

// Each stage below works on a group of nz subsamples in one launch per kernel (grid z), whose workspaces lie `zw` bytes apart
// (0 with a single one), and takes `ext`: null = use the flag word in its own workspace and report the error before
// returning (the stage waits for the stream); non-null = raise that device flag instead (SLOT_WORDS words from one subsample's to
// the next) and only enqueue: the caller reads the flags of all stages later.
constexpr int MAX_SLOTS = 3;
constexpr int SLOT_WORDS = 16;          // a subsample's flags (index, degree, rank, initial centres), then its k-means control words
constexpr int SLOT_CTL = 4;
constexpr long long ZF = SLOT_WORDS * sizeof(int);
struct Group {
  int nz;
  long long zw;
};

// idx of the group's subsamples lie one behind the other; A has rows of lda floats
int similarity_impl(const float *X, const float *t, int N, int F, const int *idx, int n, float alpha, float *A, int lda,
                    float *d_r, float *d_c, void *work, Group gr, hipStream_t st, int *ext = nullptr) {
  SimWork w(work, N, F, n);
  int *fl = ext ? ext : w.flag;
  const unsigned nz = (unsigned)gr.nz;
  if (!ext) hipLaunchKernelGGL(fill_int_kernel, dim3(1), dim3(256), 0, st, w.flag, 64, 0, 0ll);
  hipLaunchKernelGGL(rownorm_kernel, dim3((N + 3) / 4), dim3(256), 0, st, X, N, F, w.rinv);      // once for the whole group
  hipLaunchKernelGGL(gather_kernel, dim3(n, 1, nz), dim3(256), 0, st, X, w.rinv, t, idx, N, F, w.Xs, w.cs, w.tc, fl,
                     (long long)n * sizeof(int), gr.zw, ZF);
  TAP_HIP(hipGetLastError());
  SgemmArgs g{};
  g.A = X; g.sam = F; g.sak = 1;
  g.B = w.Xs; g.sbn = F; g.sbk = 1; g.zb = gr.zw;
  g.C = A; g.ldc = lda; g.zc = gr.zw;
  g.M = N; g.N = n; g.K = F;
  g.rs = w.rinv; g.cs = w.cs; g.tr = t; g.tc = w.tc; g.alpha = alpha; g.zcs = gr.zw; g.ztc = gr.zw;
  if (g_prof.on) {
    if (g_prof.used == g_prof.ev.size()) {
      hipEvent_t a, b;
      TAP_HIP(hipEventCreate(&a));
      TAP_HIP(hipEventCreate(&b));
      g_prof.ev.emplace_back(a, b);
    }
    TAP_HIP(hipEventRecord(g_prof.ev[g_prof.used].first, st));
  }
  TAP_HIP(sgemm(g, SE_SIM, gr.nz, st));
  if (g_prof.on) {
    TAP_HIP(hipEventRecord(g_prof.ev[g_prof.used++].second, st));
    g_prof.products += gr.nz;
  }
  // (26 blocks of columns, 175 registers, cover a twentieth of a pool of 33000; wider ones were not measured against the two passes)
#define DEGREE_SUMS(NC) hipLaunchKernelGGL(degree_sums_kernel<NC>, dim3(COL_CHUNKS, 1, nz), dim3(256), 0, st, A, N, n, lda, d_r, w.colpart, gr.zw)
  if (n <= 64 * 3) DEGREE_SUMS(3);
  else if (n <= 64 * 8) DEGREE_SUMS(8);
  else if (n <= 64 * 16) DEGREE_SUMS(16);
  else if (n <= 64 * 26) DEGREE_SUMS(26);
  else {      // more columns than a wavefront keeps sums of
    hipLaunchKernelGGL(rowsum_kernel, dim3((N + 3) / 4, 1, nz), dim3(256), 0, st, A, N, n, lda, d_r, gr.zw);
    hipLaunchKernelGGL(colsum_partial_kernel, dim3((n + 63) / 64, COL_CHUNKS, nz), dim3(256), 0, st, A, N, n, lda, w.colpart, gr.zw);
  }
#undef DEGREE_SUMS
  hipLaunchKernelGGL(colsum_final_kernel, dim3((n + 255) / 256, 1, nz), dim3(256), 0, st, w.colpart, n, d_c, gr.zw);
  TAP_HIP(hipGetLastError());
  if (ext) return QC_OK;
  int flag = 0;
  TAP_RC(read_flag(w.flag, st, &flag));
  if (flag) TAP_FAIL(QC_ERR_RANGE, "a subsample index lies outside [0, %d)", N);
  return QC_OK;
}

int normalise_impl(float *A, const float *d_r, const float *d_c, int N, int n, int lda, void *work, Group gr, hipStream_t st,
                   int *ext = nullptr) {
  SmallWork w(work, 1, 1, 1);
  int *fl = ext ? ext : w.flag;
  const unsigned nz = (unsigned)gr.nz;
  if (!ext) hipLaunchKernelGGL(fill_int_kernel, dim3(1), dim3(256), 0, st, w.flag, 64, 0, 0ll);
  hipLaunchKernelGGL(degree_check_kernel, dim3((N + n + 255) / 256, 1, nz), dim3(256), 0, st, d_r, N, d_c, n, fl, gr.zw, ZF);
  TAP_HIP(hipGetLastError());
  if (!ext) {
    int flag = 0;
    TAP_RC(read_flag(w.flag, st, &flag));
    if (flag) TAP_FAIL(QC_ERR_RANGE, "a degree of the similarity matrix is not positive and finite");
  }
  // with a deferred check the kernel itself leaves the matrix alone when the flag is up
  const unsigned row_blocks = (unsigned)((N + NORM_ROWS - 1) / NORM_ROWS);
  if (lda % 4 == 0 && aligned16(A))
    hipLaunchKernelGGL(normalise_kernel<4>, dim3((unsigned)((lda + 1023) / 1024) * row_blocks, 1, nz), dim3(256), 0, st, A, d_r, d_c, N, n,
                       lda, ext ? (const int *)ext : (const int *)nullptr, gr.zw, ZF);
  else
    hipLaunchKernelGGL(normalise_kernel<1>, dim3((unsigned)((lda + 255) / 256) * row_blocks, 1, nz), dim3(256), 0, st, A, d_r, d_c, N, n,
                       lda, ext ? (const int *)ext : (const int *)nullptr, gr.zw, ZF);
  TAP_HIP(hipGetLastError());
  if (!ext) TAP_HIP(hipStreamSynchronize(st));
  return QC_OK;
}

hipError_t set_lds(const void *kern, size_t bytes) {
  return hipFuncSetAttribute(kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes);
}

// Gram matrix W of kb vectors of n elements: vector a's element j at Y[a * sv + j] (kc) or Y[j * sv + a]; zy: bytes from one
// subsample's vectors to the next
int gram(const float *Y, long long zy, bool kc, int kb, int n, long long sv, EmbedWork &w, Group gr, hipStream_t st, bool reduce = true) {
  const int nb = (kb + 15) / 16, parts = gram_parts(n);
  const bool v4 = kc && aligned16(Y) && sv % 4 == 0 && n % 4 == 0;
  const dim3 grid((unsigned)parts, 1, (unsigned)gr.nz);
#define GRAM_ONE(NB, K, V) \
  hipLaunchKernelGGL((gram_partial_kernel<NB, K, V>), grid, dim3(512), 0, st, Y, kb, n, sv, gram_chunk(n), w.part, zy, gr.zw)
#define GRAM_CASE(NB)                       \
  case NB:                                  \
    if (!kc) GRAM_ONE(NB, false, false);    \
    else if (v4) GRAM_ONE(NB, true, true);  \
    else GRAM_ONE(NB, true, false);         \
    break;
  switch (nb) {
    GRAM_CASE(1)
    GRAM_CASE(2)
    GRAM_CASE(3)
    GRAM_CASE(4)
    GRAM_CASE(5)
    GRAM_CASE(6)
    GRAM_CASE(7)
    GRAM_CASE(8)
    default: TAP_FAIL(QC_ERR_UNSUPPORTED, "at most %d vectors", KB_MAX);
  }
#undef GRAM_CASE
#undef GRAM_ONE
  if (!reduce) return QC_OK;
  hipLaunchKernelGGL(gram_reduce_kernel, dim3((kb * kb + 255) / 256, 1, (unsigned)gr.nz), dim3(256), 0, st, w.part, parts, kb, w.W, gr.zw);
  TAP_HIP(hipGetLastError());
  return QC_OK;
}

// one pass of shifted Cholesky QR on the rows of `in` [kb, n] into `out` (`in` and `out` must differ); zin: bytes from one
// subsample's rows to the next
int cholqr_pass(const float *in, long long zin, float *out, int kb, int n, int check, EmbedWork &w, Group gr, int *fl, hipStream_t st) {
  // The factorisation adds the ranges itself where they are few, which is a launch less: the whole clustering 2 % faster up to 4096 numbers
  // (kb = 32, n = 200: 968 -> 951 us), 1 % at 7000 - 13000, as fast at 16000, 1 % slower at 25600 and 9 % at 200000 (one workgroup reads them).
  const bool direct = (long long)gram_parts(n) * kb * kb <= 12288;
  TAP_RC(gram(in, zin, true, kb, n, n, w, gr, st, !direct));
  const int kp = (kb + 15) / 16 * 16;
  const size_t lds = (size_t)kp * (kp + 4) * sizeof(double);
  TAP_HIP(set_lds((const void *)chol_inv_kernel, lds));
  hipLaunchKernelGGL(chol_inv_kernel, dim3(1, 1, (unsigned)gr.nz), dim3(1024), lds, st, direct ? w.part : w.W, direct ? gram_parts(n) : 1, kb,
                     1e-12, check, w.Rinv, fl, gr.zw, ZF);
  TAP_HIP(hipGetLastError());
  SgemmArgs g{};
  g.A = w.Rinv; g.sam = kb; g.sak = 1; g.za = gr.zw;
  g.B = in; g.sbn = 1; g.sbk = n; g.zb = zin;
  g.C = out; g.ldc = n; g.zc = gr.zw;
  g.M = kb; g.N = n; g.K = kb;
  TAP_HIP(sgemm(g, SE_PLAIN, gr.nz, st));
  return QC_OK;
}

// rows of `in` made orthonormal into w.Q: three passes, which is enough for a block whose condition number is as
// large as 10^12 (the power iteration multiplies by L^T L, whose small eigenvalues are rounding noise in fp32); uses
// w.Z and w.Y as intermediates (`in` may be w.Y)
int orthonormalise(const float *in, long long zin, EmbedWork &w, int kb, int n, Group gr, int *fl, hipStream_t st) {
  TAP_RC(cholqr_pass(in, zin, w.Z, kb, n, 0, w, gr, fl, st));
  TAP_RC(cholqr_pass(w.Z, gr.zw, w.Y, kb, n, 0, w, gr, fl, st));
  TAP_RC(cholqr_pass(w.Y, gr.zw, w.Q, kb, n, 1, w, gr, fl, st));
  return QC_OK;
}

// Between two multiplications of the power iteration one pass is enough: the next product only needs rows that span
// the same space and are well conditioned (a single shifted pass leaves them orthonormal to about the square of the
// block's condition number times the fp64 rounding, far from dependent); `in` must not be w.Q
int recondition(const float *in, long long zin, EmbedWork &w, int kb, int n, Group gr, int *fl, hipStream_t st) {
  return cholqr_pass(in, zin, w.Q, kb, n, 0, w, gr, fl, st);
}

// L has rows of n floats and q0 rows of n0 <= n; the columns of L beyond n0 are zero.  The results U, sigma lie zout bytes apart.
int embed_impl(const float *L, int N, int n, int n0, int k, int kb, int iters, const float *q0, float *U, float *sigma, long long zout,
               void *work, Group gr, hipStream_t st, int *ext = nullptr) {
  EmbedWork w(work, N, n, k, kb);
  int *fl = ext ? ext : w.flag;
  const unsigned nz = (unsigned)gr.nz;
  if (!ext) hipLaunchKernelGGL(fill_int_kernel, dim3(1), dim3(256), 0, st, w.flag, 64, 0, 0ll);
  TAP_HIP(hipGetLastError());
  // G = L^T L drives the power iteration (its fp32 rounding only slows the convergence of directions whose singular
  // values are below about 3e-4 of the largest; the Rayleigh-Ritz step below works on L itself)
  SgemmArgs g{};
  g.A = L; g.sam = 1; g.sak = n; g.za = gr.zw;
  g.B = L; g.sbn = 1; g.sbk = n; g.zb = gr.zw;
  g.C = w.G; g.ldc = n; g.zc = gr.zw; g.zpart = gr.zw;
  g.M = n; g.N = n; g.K = N;
  g.sym = 1;
  TAP_HIP(sgemm(g, SE_PLAIN, gr.nz, st, w.spart, w.spart_elems));
  const float *start = q0;
  long long zstart = 0;
  if (n != n0) {
    hipLaunchKernelGGL(pad_rows_kernel, dim3(kb, 1, nz), dim3(256), 0, st, q0, n0, w.Y, n, gr.zw);
    start = w.Y;
    zstart = gr.zw;
  }
  if (iters > 0) TAP_RC(recondition(start, zstart, w, kb, n, gr, fl, st));
  else TAP_RC(orthonormalise(start, zstart, w, kb, n, gr, fl, st));
  SgemmArgs mul{};
  mul.A = w.Q; mul.sam = n; mul.sak = 1; mul.za = gr.zw;
  mul.B = w.G; mul.sbn = n; mul.sbk = 1; mul.zb = gr.zw;      // G is symmetric
  mul.C = w.Y; mul.ldc = n; mul.zc = gr.zw; mul.zpart = gr.zw;
  mul.M = kb; mul.N = n; mul.K = n; mul.zero_k = n - n0;
  for (int it = 0; it < iters; ++it) {
    TAP_HIP(sgemm(mul, SE_PLAIN, gr.nz, st, w.spart, w.spart_elems));
    if (it + 1 < iters) TAP_RC(recondition(w.Y, gr.zw, w, kb, n, gr, fl, st));
    else TAP_RC(orthonormalise(w.Y, gr.zw, w, kb, n, gr, fl, st));      // the final basis: orthonormal to fp32 level
  }
  // Rayleigh-Ritz on B = L Q^T [N, kb]: T = B^T B (fp64), its k leading eigenvectors W, U = B W^T diag(1 / sigma)
  SgemmArgs bm{};
  bm.A = L; bm.sam = n; bm.sak = 1; bm.za = gr.zw;
  bm.B = w.Q; bm.sbn = n; bm.sbk = 1; bm.zb = gr.zw;
  bm.C = w.Bm; bm.ldc = kb; bm.zc = gr.zw;
  bm.M = N; bm.N = kb; bm.K = n;
  TAP_HIP(sgemm(bm, SE_PLAIN, gr.nz, st));
  TAP_RC(gram(w.Bm, gr.zw, false, kb, N, kb, w, gr, st));
  const size_t lds = (size_t)kb * (kb + 2) * sizeof(double);
#define JACOBI_CASE(NC)                                                                                                          \
  case NC:                                                                                                                       \
    TAP_HIP(set_lds((const void *)jacobi_kernel<NC>, lds));                                                                      \
    hipLaunchKernelGGL(jacobi_kernel<NC>, dim3(1, 1, nz), dim3((unsigned)((kb * 8 + 63) / 64 * 64)), lds, st, w.W, kb, k, 30, w.Wk, w.isig, \
                       sigma, gr.zw, zout);                                                                                      \
    break;
  switch ((kb + 15) / 16) {
    JACOBI_CASE(1)
    JACOBI_CASE(2)
    JACOBI_CASE(3)
    JACOBI_CASE(4)
    JACOBI_CASE(5)
    JACOBI_CASE(6)
    JACOBI_CASE(7)
    JACOBI_CASE(8)
    default: TAP_FAIL(QC_ERR_UNSUPPORTED, "at most %d vectors", KB_MAX);
  }
#undef JACOBI_CASE
  TAP_HIP(hipGetLastError());
  SgemmArgs u{};
  u.A = w.Bm; u.sam = kb; u.sak = 1; u.za = gr.zw;
  u.B = w.Wk; u.sbn = kb; u.sbk = 1; u.zb = gr.zw;
  u.C = U; u.ldc = k; u.zc = zout;
  u.M = N; u.N = k; u.K = kb;
  u.cs = w.isig; u.zcs = gr.zw;
  TAP_HIP(sgemm(u, SE_COLSCALE, gr.nz, st));
  if (ext) return QC_OK;
  int flag = 0;
  TAP_RC(read_flag(w.flag, st, &flag));
  if (flag) TAP_FAIL(QC_ERR_RANGE, "the iteration block has no full rank (a zero start vector, or fewer than kb independent directions)");
  return QC_OK;
}

template <int NC>
auto kmeans_kernel(bool v4, bool stage) {
  if constexpr (NC <= KM_STAGE_NC)
    if (stage) return v4 ? kmeans_pass_kernel<NC, true, true> : kmeans_pass_kernel<NC, false, true>;
  return v4 ? kmeans_pass_kernel<NC, true, false> : kmeans_pass_kernel<NC, false, false>;
}

hipError_t launch_kmeans_pass(const float *U, int N, int d, float *centres, int k, int *labels, const SmallWork &w, int *ctl, int it, bool own,
                              long long zu, long long zlab, Group gr, hipStream_t st) {
  const int nc = (d + 15) / 16, k16 = (k + 15) / 16 * 16;
  const bool stage = nc <= KM_STAGE_NC && kmeans_rows_per(N) <= KM_ROWS;
  const size_t lds = ((size_t)k16 * (16 * nc + 4 + 1) + (stage ? (size_t)KM_ROWS * (16 * nc + 4) : 0)) * sizeof(float);
  const bool v4 = d % 4 == 0 && aligned16(U);
  const size_t out = kmeans_own(N, d, k) ? it & 1 : 0, in = kmeans_own(N, d, k) ? out ^ 1 : 0;
#define KM_CASE(NC)                                                                                                          \
  case NC: {                                                                                                                 \
    const auto kern = kmeans_kernel<NC>(v4, stage);                                                                          \
    const hipError_t e = it == 0 ? set_lds((const void *)kern, lds) : hipSuccess;                                            \
    if (e != hipSuccess) return e;                                                                                           \
    hipLaunchKernelGGL(kern, dim3(kmeans_blocks(N), 1, (unsigned)gr.nz), dim3(512), lds, st, U, N, d, centres, k, kmeans_rows_per(N), \
                       labels, w.psum + in * w.count * d, w.pcnt + in * w.count, w.psum + out * w.count * d, w.pcnt + out * w.count, \
                       w.dirty, ctl, it, own ? 1 : 0, zu, zlab, gr.zw, ZF);                                                  \
    break;                                                                                                                   \
  }
  switch (nc) {
    KM_CASE(1)
    KM_CASE(2)
    KM_CASE(3)
    KM_CASE(4)
    KM_CASE(5)
    KM_CASE(6)
    KM_CASE(7)
    KM_CASE(8)
    default: return hipErrorInvalidValue;
  }
#undef KM_CASE
  return hipGetLastError();
}

// Lloyd's iteration on the group's problems.  The passes decide on the device whether they still have work (see the control
// words above), so the host enqueues KM_BATCH passes and only then reads the control words; a problem is over when a pass
// has changed nothing, and the loop when all are.  U and the centres of the group lie zu bytes apart; `ext` holds the index
// check's flag of each problem (word 3) and its control words; null: a single problem whose index check is reported before
// the first pass, words in the workspace.  `words` (host, SLOT_WORDS a problem): all of them after the last pass.
constexpr int KM_BATCH = 8;

int kmeans_group(const float *U, long long zu, int N, int d, int k, const int *init_idx, int max_iter, int *labels, float *centres,
                 void *work, Group gr, hipStream_t st, int *ext, int *words) {
  const int nb = kmeans_blocks(N);
  const unsigned nz = (unsigned)gr.nz;
  SmallWork w(work, N, d, k);
  int *all = ext ? ext : w.flag, *ctl = all + SLOT_CTL;
  const long long zlab = (long long)N * sizeof(int);
  if (!ext) hipLaunchKernelGGL(fill_int_kernel, dim3(1), dim3(256), 0, st, all, 64, 0, 0ll);
  hipLaunchKernelGGL(fill_int_kernel, dim3((N * nz + 255) / 256), dim3(256), 0, st, labels, (int)(N * nz), -1, 0ll);
  hipLaunchKernelGGL(fill_int_kernel, dim3(1, 1, nz), dim3(256), 0, st, w.dirty, k, 0, gr.zw);
  hipLaunchKernelGGL(kmeans_init_kernel, dim3(k, 1, nz), dim3(256), 0, st, U, N, d, k, init_idx, centres, all + 3, zu,
                     (long long)k * sizeof(int), ZF);
  TAP_HIP(hipGetLastError());
  if (!ext) {
    int flag = 0;
    TAP_RC(read_flag(all + 3, st, &flag));
    if (flag) TAP_FAIL(QC_ERR_RANGE, "an initial-centre index lies outside [0, %d)", N);
  }
  const bool own = kmeans_own(N, d, k);
  for (int it0 = 0; it0 < max_iter; it0 += KM_BATCH) {
    const int it1 = it0 + KM_BATCH < max_iter ? it0 + KM_BATCH : max_iter;
    for (int it = it0; it < it1; ++it) {
      TAP_HIP(launch_kmeans_pass(U, N, d, centres, k, labels, w, ctl, it, own && it > it0, zu, zlab, gr, st));
      if (own && it + 1 < it1) continue;
      hipLaunchKernelGGL(kmeans_finish_kernel, dim3(k, 1, nz), dim3(128), 0, st, w.psum + (own ? it & 1 : 0) * w.count * d,
                         w.pcnt + (own ? it & 1 : 0) * w.count, nb, k, d, centres, w.dirty, ctl, it,
                         zu, gr.zw, ZF);
      TAP_HIP(hipGetLastError());
    }
    TAP_HIP(hipMemcpyAsync(words, all, (size_t)gr.nz * ZF, hipMemcpyDeviceToHost, st));
    TAP_HIP(hipStreamSynchronize(st));
    bool any = false;
    for (int z = 0; z < gr.nz; ++z) any = any || !words[z * SLOT_WORDS + SLOT_CTL + KM_DONE];
    if (!any) break;
  }
  return QC_OK;
}

int kmeans_impl(const float *U, int N, int d, int k, const int *init_idx, int max_iter, int *labels, float *centres,
                int *passes_out, void *work, hipStream_t st) {
  int words[SLOT_WORDS];
  TAP_RC(kmeans_group(U, 0, N, d, k, init_idx, max_iter, labels, centres, work, Group{1, 0}, st, nullptr, words));
  if (passes_out) *passes_out = words[SLOT_CTL + KM_PASSES];
  return QC_OK;
}

int aggregate_impl(const int *labels, int m, int N, int k, int *out, int *perm_out, void *work, hipStream_t st) {
  SmallWork w(work, 1, 1, k);
  hipLaunchKernelGGL(identity_perm_kernel, dim3((k + 255) / 256), dim3(256), 0, st, w.perm, k);
  for (int i = 1; i < m; ++i) {
    hipLaunchKernelGGL(fill_int_kernel, dim3((k * k + 255) / 256), dim3(256), 0, st, w.T, k * k, 0, 0ll);
    hipLaunchKernelGGL(contingency_kernel, dim3((N + 255) / 256), dim3(256), 0, st, labels, labels + (size_t)i * N, N, k, w.T);
    const size_t lds = (size_t)k * (k + 1) * sizeof(int);
    TAP_HIP(set_lds((const void *)greedy_match_kernel, lds));
    hipLaunchKernelGGL(greedy_match_kernel, dim3(1), dim3(1024), lds, st, w.T, k, w.perm + (size_t)i * k);
  }
  hipLaunchKernelGGL(vote_kernel, dim3((N + 255) / 256), dim3(256), 0, st, labels, w.perm, m, N, k, out);
  TAP_HIP(hipGetLastError());
  if (perm_out) TAP_HIP(hipMemcpyAsync(perm_out, w.perm, (size_t)m * k * sizeof(int), hipMemcpyDeviceToDevice, st));
  return QC_OK;
}

int check_work(const void *work, size_t have, size_t need) {
  if (!work) TAP_FAIL(QC_ERR_NULL, "work is NULL");
  if (!aligned16(work)) TAP_FAIL(QC_ERR_ALIGN, "work must be 16-byte aligned");
  if (have < need) TAP_FAIL(QC_ERR_WORKSPACE, "workspace of %zu bytes is too small (%zu needed)", have, need);
  return QC_OK;
}

}  // namespace

extern "C" {

int qc_tap_workspace_bytes(int N, int F, int n, int k, int kb, size_t *bytes_out) {
  if (!bytes_out) TAP_FAIL(QC_ERR_NULL, "bytes_out is NULL");
  TAP_RC(check_dims(N, F, n, k, kb));
  *bytes_out = ClusterWork(nullptr, N, F, n, k, kb).bytes;
  return QC_OK;
}

int qc_tap_profile_begin(void) {
  g_prof.on = true;
  g_prof.used = 0;
  g_prof.products = 0;
  return QC_OK;
}

int qc_tap_profile_end(float *sim_ms_out, int *launches_out) {
  if (!sim_ms_out || !launches_out) TAP_FAIL(QC_ERR_NULL, "an output pointer is NULL");
  if (!g_prof.on) TAP_FAIL(QC_ERR_STATE, "qc_tap_profile_begin was not called");
  g_prof.on = false;
  float total = 0.f;
  for (size_t i = 0; i < g_prof.used; ++i) {
    TAP_HIP(hipEventSynchronize(g_prof.ev[i].second));
    float ms = 0.f;
    TAP_HIP(hipEventElapsedTime(&ms, g_prof.ev[i].first, g_prof.ev[i].second));
    total += ms;
  }
  *sim_ms_out = total;
  *launches_out = g_prof.products;
  return QC_OK;
}

int qc_tap_similarity(const float *X, const float *t, int N, int F, const int *idx, int n, float alpha, float *A,
                      float *d_r, float *d_c, void *work, size_t work_bytes, void *stream) {
  if (!X || !t || !idx || !A || !d_r || !d_c) TAP_FAIL(QC_ERR_NULL, "a required pointer is NULL");
  if (N < 1 || F < 1 || n < 1) TAP_FAIL(QC_ERR_SHAPE, "N, F, n must be positive");
  if (n > N) TAP_FAIL(QC_ERR_SHAPE, "n (%d) exceeds N (%d)", n, N);
  if ((long long)N * (n > F ? n : F) >= (1ll << 31)) TAP_FAIL(QC_ERR_UNSUPPORTED, "N * max(n, F) must be below 2^31");
  if (!(alpha >= 0.f && alpha <= 1.f)) TAP_FAIL(QC_ERR_RANGE, "alpha must lie in [0, 1]");
  if (!aligned16(X) || !aligned16(A)) TAP_FAIL(QC_ERR_ALIGN, "X and A must be 16-byte aligned");
  TAP_RC(check_work(work, work_bytes, SimWork(nullptr, N, F, n).bytes));
  return similarity_impl(X, t, N, F, idx, n, alpha, A, n, d_r, d_c, work, Group{1, 0}, static_cast<hipStream_t>(stream));
}

int qc_tap_normalise(float *A, const float *d_r, const float *d_c, int N, int n, void *work, size_t work_bytes,
                     void *stream) {
  if (!A || !d_r || !d_c) TAP_FAIL(QC_ERR_NULL, "a required pointer is NULL");
  if (N < 1 || n < 1) TAP_FAIL(QC_ERR_SHAPE, "N and n must be positive");
  if ((long long)N * n >= (1ll << 31)) TAP_FAIL(QC_ERR_UNSUPPORTED, "N * n must be below 2^31");
  TAP_RC(check_work(work, work_bytes, SmallWork(nullptr, 1, 1, 1).bytes));
  return normalise_impl(A, d_r, d_c, N, n, n, work, Group{1, 0}, static_cast<hipStream_t>(stream));
}

int qc_tap_embed(const float *L, int N, int n, int k, int kb, int iters, const float *q0, float *U, float *sigma,
                 void *work, size_t work_bytes, void *stream) {
  if (!L || !q0 || !U || !sigma) TAP_FAIL(QC_ERR_NULL, "a required pointer is NULL");
  TAP_RC(check_dims(N, 1, n, k, kb));
  if (iters < 0 || iters > 1000) TAP_FAIL(QC_ERR_RANGE, "iters must lie in [0, 1000]");
  if (!aligned16(L) || !aligned16(q0) || !aligned16(U)) TAP_FAIL(QC_ERR_ALIGN, "L, q0 and U must be 16-byte aligned");
  TAP_RC(check_work(work, work_bytes, EmbedWork(nullptr, N, n, k, kb).bytes));
  return embed_impl(L, N, n, n, k, kb, iters, q0, U, sigma, 0, work, Group{1, 0}, static_cast<hipStream_t>(stream));
}

int qc_tap_kmeans(const float *U, int N, int d, int k, const int *init_idx, int max_iter, int *labels, float *centres,
                  int *passes_out, void *work, size_t work_bytes, void *stream) {
  if (!U || !init_idx || !labels || !centres) TAP_FAIL(QC_ERR_NULL, "a required pointer is NULL");
  if (N < 1 || d < 1 || k < 1) TAP_FAIL(QC_ERR_SHAPE, "N, d, k must be positive");
  if (d > KB_MAX || k > KB_MAX) TAP_FAIL(QC_ERR_UNSUPPORTED, "d and k must be at most %d", KB_MAX);
  if ((long long)N * d >= (1ll << 31)) TAP_FAIL(QC_ERR_UNSUPPORTED, "N * d must be below 2^31");
  if (max_iter < 1) TAP_FAIL(QC_ERR_RANGE, "max_iter must be at least 1");
  TAP_RC(check_work(work, work_bytes, SmallWork(nullptr, N, d, k).bytes));
  return kmeans_impl(U, N, d, k, init_idx, max_iter, labels, centres, passes_out, work, static_cast<hipStream_t>(stream));
}

int qc_tap_aggregate(const int *labels, int m, int N, int k, int *out, int *perm_out, void *work, size_t work_bytes,
                     void *stream) {
  if (!labels || !out) TAP_FAIL(QC_ERR_NULL, "a required pointer is NULL");
  if (m < 1 || N < 1 || k < 1) TAP_FAIL(QC_ERR_SHAPE, "m, N, k must be positive");
  if (m > M_MAX) TAP_FAIL(QC_ERR_UNSUPPORTED, "at most %d label vectors", M_MAX);
  if (k > KB_MAX) TAP_FAIL(QC_ERR_UNSUPPORTED, "k must be at most %d", KB_MAX);
  if ((long long)m * N >= (1ll << 31)) TAP_FAIL(QC_ERR_UNSUPPORTED, "m * N must be below 2^31");
  TAP_RC(check_work(work, work_bytes, SmallWork(nullptr, 1, 1, k).bytes));
  return aggregate_impl(labels, m, N, k, out, perm_out, work, static_cast<hipStream_t>(stream));
}

int qc_tap_cluster(const float *X, const float *t, int N, int F, const int *subsamples, int m, int n, float alpha,
                   int k, int kb, int iters, const float *q0, const int *init_idx, int max_iter, int *labels_out,
                   int *per_labels, void *work, size_t work_bytes, void *stream) {
  if (!X || !t || !subsamples || !q0 || !init_idx || !labels_out || !per_labels)
    TAP_FAIL(QC_ERR_NULL, "a required pointer is NULL");
  TAP_RC(check_dims(N, F, n, k, kb));
  if (m < 1 || m > M_MAX) TAP_FAIL(QC_ERR_UNSUPPORTED, "m must lie in [1, %d]", M_MAX);
  if (!(alpha >= 0.f && alpha <= 1.f)) TAP_FAIL(QC_ERR_RANGE, "alpha must lie in [0, 1]");
  if (iters < 0 || iters > 1000) TAP_FAIL(QC_ERR_RANGE, "iters must lie in [0, 1000]");
  if (max_iter < 1) TAP_FAIL(QC_ERR_RANGE, "max_iter must be at least 1");
  if (!aligned16(X) || !aligned16(q0)) TAP_FAIL(QC_ERR_ALIGN, "X and q0 must be 16-byte aligned");
  const size_t per = (ClusterWork(nullptr, N, F, n, k, kb).bytes + 255) & ~size_t(255);
  TAP_RC(check_work(work, work_bytes, per));
  hipStream_t st = static_cast<hipStream_t>(stream);
  // As many subsamples at a time as the workspace holds (at most MAX_SLOTS), one launch a kernel for all of them.  (Three streams whose
  // large products were chained by events, so that one subsample's small kernels ran beside another's products: the same time at
  // 32768 samples, where they slowed each other down, and three times the launches, which bound small pools.)
  int slots = (int)(work_bytes / per);
  if (slots > MAX_SLOTS) slots = MAX_SLOTS;
  if (slots > m) slots = m;
  for (int i0 = 0; i0 < m; i0 += slots) {
    const Group gr{m - i0 < slots ? m - i0 : slots, (long long)per};
    ClusterWork w(work, N, F, n, k, kb);
    hipLaunchKernelGGL(fill_int_kernel, dim3(1), dim3(256), 0, st, w.flags, 64, 0, 0ll);
    const int ld = padded(n);
    TAP_RC(similarity_impl(X, t, N, F, subsamples + (size_t)i0 * n, n, alpha, w.A, ld, w.dr, w.dc, w.sub, gr, st, w.flags + 0));
    TAP_RC(normalise_impl(w.A, w.dr, w.dc, N, n, ld, w.sub, gr, st, w.flags + 1));
    TAP_RC(embed_impl(w.A, N, ld, n, k, kb, iters, q0, w.U, w.sigma, gr.zw, w.sub, gr, st, w.flags + 2));
    // the first pass of the k-means below runs on whatever the earlier stages left; the flags tell afterwards
    // whether that was meaningful (every kernel stays inside its buffers on any input)
    int words[MAX_SLOTS * SLOT_WORDS];
    TAP_RC(kmeans_group(w.U, gr.zw, N, k, k, init_idx + (size_t)i0 * k, max_iter, per_labels + (size_t)i0 * N, w.centres, w.sub, gr, st,
                        w.flags, words));
    for (int z = 0; z < gr.nz; ++z) {
      const int *fl = words + z * SLOT_WORDS;
      if (fl[0]) TAP_FAIL(QC_ERR_RANGE, "a subsample index lies outside [0, %d)", N);
      if (fl[1]) TAP_FAIL(QC_ERR_RANGE, "a degree of the similarity matrix is not positive and finite");
      if (fl[2]) TAP_FAIL(QC_ERR_RANGE, "the iteration block has no full rank (a zero start vector, or fewer than kb independent directions)");
      if (fl[3]) TAP_FAIL(QC_ERR_RANGE, "an initial-centre index lies outside [0, %d)", N);
    }
  }
  TAP_RC(aggregate_impl(per_labels, m, N, k, labels_out, nullptr, work, st));
  TAP_HIP(hipStreamSynchronize(st));
  return QC_OK;
}

}  // extern "C"
