// A tile of a float32 product on the matrix cores, C(m, n) = sum_k A(m, k) B(n, k), both operands contiguous along k (run) or both
// along their own index (run_tn): every output one chain of float32 fused multiply-adds in ascending k.
//
// v_mfma_f32_32x32x2_f32 adds its two products one after the other, each with the rounding of a fused multiply-add, in
// ascending k (checked bit by bit against fmaf), so the result is that of a plain loop over k, whatever the tile; K is never split.
// The 32 x 32 form because the 16 x 16 x 4 one does not reach its rate: loops of nothing else, one / two wavefronts a SIMD,
// 153 / 154 against 118 / 135 TFLOP/s.
//
// A workgroup of WM x WN wavefronts owns a tile of 32 WM TM x 32 WN TN outputs, a wavefront TM x TN blocks of 32 x 32.  K is
// walked in slabs of BK that go from memory straight to LDS (NS buffers, chunks swizzled by the thread that fetches them); the
// fragments of the next slab are read into registers while one is multiplied.  Every LDS and memory instruction is issued
// behind a product.
#pragma once
#include "qc_internal.h"

namespace qc {

typedef float f32x16 __attribute__((ext_vector_type(16)));

// all but the last N loads of this wavefront and all its LDS reads done, then the workgroup barrier
template <int N>
__device__ __forceinline__ void slab_barrier() {
  asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"(N) : "memory");
}

template <int WM, int WN, int TM, int TN, int BK, int NS>
struct F32Tile {
  static_assert(BK == 16, "the swizzle is that of rows of four chunks");
  static constexpr int NT = 64 * WM * WN, RM = 32 * WM * TM, RN = 32 * WN * TN;      // threads, rows of either operand
  static constexpr int CH = BK / 4, RP = NT / CH;                                     // 16-byte chunks of a slab row, rows per pass
  static constexpr int LM = (RM + RP - 1) / RP, LN = (RN + RP - 1) / RP, NL = LM + LN;      // passes
  static constexpr int SLAB = (LM + LN) * RP * BK;                                    // floats of a slab, both operands
  static_assert(NS % 2 == 0 && NS >= 4, "the fragment set of a slab is its parity");

  f32x16 acc[TM][TN];
  int wm, wn;             // first row and column of the wavefront in the tile

  // rows of this tile from m0, n0 (rows beyond M, N re-read the last one and give values that the caller does not store); slabs: NS *
  // SLAB floats of LDS; K a multiple of 4
  __device__ __forceinline__ void run(const float *__restrict__ A, size_t lda, const float *__restrict__ B, size_t ldb, int M, int N, int K,
                                      int m0, int n0, float *slabs) {
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    // Pass i of the loads covers rows RP i .. of a slab, 16 bytes per thread, and goes straight to LDS, thread after thread.  Chunk
    // c of row r lies at chunk c ^ swz(r) (so that the rows of a fragment read spread over the banks): the thread of a place
    // fetches the chunk that belongs there.
    const auto swz = [](int r) { return (r >> 2) & (CH - 1); };
    const int lr = tid / CH;
    const int ns = (K + BK - 1) / BK;
    unsigned ao[LM], bo[LN];                             // byte offsets of this thread's chunk in slab 0
#pragma unroll
    for (int i = 0; i < LM; ++i) ao[i] = ((unsigned)(min(m0 + lr + RP * i, M - 1) - m0) * (unsigned)lda + ((tid % CH) ^ swz(lr + RP * i)) * 4) * 4;
#pragma unroll
    for (int i = 0; i < LN; ++i) bo[i] = ((unsigned)(min(n0 + lr + RP * i, N - 1) - n0) * (unsigned)ldb + ((tid % CH) ^ swz(lr + RP * i)) * 4) * 4;
    const float *ab = A + (size_t)m0 * lda, *bb = B + (size_t)n0 * ldb;
    const unsigned lds0 = (unsigned)(size_t)(__attribute__((address_space(3))) float *)slabs + wave * 1024;
    // (m0 is a reserved register, which a clobber list cannot name: nothing else in these kernels uses it, tests/test_codegen_cpu.py)
    auto load = [&](int s, int b, int i) {               // slabs past the end re-read the last one (never used)
      const bool of_a = i < LM;
      const int row = of_a ? lr + RP * i : lr + RP * (i - LM);
      // chunks of the last slab beyond K re-read its end
      const int over = (ns - 1) * BK + ((tid % CH) ^ swz(row)) * 4 + 4 - K;
      const unsigned off = (of_a ? ao[of_a ? i : 0] : bo[of_a ? 0 : i - LM]) - (s >= ns - 1 && over > 0 ? (unsigned)over * 4 : 0u);
      asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" ::"s"(lds0 + (b * SLAB + i * RP * BK) * 4), "v"(off),
                   "s"((of_a ? ab : bb) + (size_t)min(s, ns - 1) * BK)
                   : "memory");
    };
    wm = (wave / WN) * 32 * TM;
    wn = (wave % WN) * 32 * TN;
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;
    // lane l supplies row l % 32, k = l / 32 of either operand: of a chunk of four k it reads floats l / 32 and l / 32 + 2
    const int row = lane & 31, h = lane >> 5;
    float fa[2][CH][TM][2], fb[2][CH][TN][2];
    // fragment read n of a slab, in the order of use: chunk, operand, block
    auto read = [&](int f, int b, int n) {
      const int q = n / (TM + TN), i = n % (TM + TN);
      if (i < TM) {
        const int r = wm + 32 * i + row;
        const float *p = slabs + b * SLAB + r * BK + ((q ^ swz(r)) << 2) + h;
        fa[f][q][i < TM ? i : 0][0] = p[0];
        fa[f][q][i < TM ? i : 0][1] = p[2];
      } else {
        const int r = wn + 32 * (i - TM) + row;
        const float *p = slabs + b * SLAB + LM * RP * BK + r * BK + ((q ^ swz(r)) << 2) + h;
        fb[f][q][i < TM ? 0 : i - TM][0] = p[0];
        fb[f][q][i < TM ? 0 : i - TM][1] = p[2];
      }
    };
    auto mul = [&](int f, int n) {
      const int e = n / (TM * TN), i = n / TN % TM, j = n % TN;      // e: pair of k
      acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(fa[f][e >> 1][i][e & 1], fb[f][e >> 1][j][e & 1], acc[i][j], 0, 0, 0);
    };
    constexpr int NM = 2 * CH * TM * TN, NR = CH * (TM + TN);       // products and fragment reads of a slab
    constexpr int RB = (NR + NM - 3) / (NM - 2);                    // reads behind a product
    static_assert((NM - 2) * RB >= NR, "the barrier stands behind every read");
    constexpr int LB = (NL + NM - 3) / (NM - 2);                    // loads behind a product
    // Step s: fragment set s % 2 holds slab s, buffer (s + 1) % NS slab s + 1; slabs s + 2 .. are on their way.  Buffer s % NS was
    // read in step s - 1, before its barrier, and takes slab s + NS.  The wait before the barrier is for slab s + 2: the loads of
    // the NS - 2 youngest steps may be outstanding.
    auto step = [&](int s, int u) {                      // u = s mod NS
      const int f = u & 1;
#pragma unroll
      for (int n = 0; n < NM; ++n) {
        __builtin_amdgcn_sched_barrier(0);
        mul(f, n);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int r = n * RB; r < min(n * RB + RB, NR); ++r) read(f ^ 1, (u + 1) % NS, r);
#pragma unroll
        for (int l = n * LB; l < min(n * LB + LB, NL); ++l) load(s + NS, u, l);
        if (n == NM - 2) slab_barrier<(NS - 2) * NL>();
      }
    };
#pragma unroll
    for (int b = 0; b < NS; ++b)
#pragma unroll
      for (int i = 0; i < NL; ++i) load(b, b, i);
    slab_barrier<(NS - 2) * NL>();                       // slabs 0 and 1
#pragma unroll
    for (int r = 0; r < NR; ++r) read(0, 0, r);
    slab_barrier<(NS - 2) * NL>();
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
        const int nm = (K - (s + u) * BK) / 2 * TM * TN;
#pragma unroll
        for (int n = 0; n < NM; ++n)
          if (n < nm) mul(u & 1, n);
      }
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");     // nothing lands in LDS after the workgroup's end
  }

  // The same with A(m, k) = A[k * lda + m], B(n, k) = B[k * ldb + n]; M, N, lda, ldb multiples of 4.  A slab keeps k rows of RM (RN)
  // floats; the 32-float halves of every odd row change places, so that the two k of a fragment read lie in different banks.
  __device__ __forceinline__ void run_tn(const float *__restrict__ A, size_t lda, const float *__restrict__ B, size_t ldb, int M, int N,
                                         int K, int m0, int n0, float *slabs) {
    static_assert(RM % 64 == 0 && RN % 64 == 0 && NT % (RM / 4) == 0 && NT % (RN / 4) == 0, "");
    constexpr int PA = NT / (RM / 4), PB = NT / (RN / 4);              // k rows per pass
    constexpr int XA = BK / PA, XB = BK / PB, XL = XA + XB, XSLAB = BK * (RM + RN);
    static_assert(XA * PA == BK && XB * PB == BK && XSLAB <= SLAB && PA % 2 == 0 && PB % 2 == 0, "");
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int ka = tid / (RM / 4), ca = ((tid % (RM / 4)) ^ ((ka & 1) << 3)) * 4, kb = tid / (RN / 4), cb = ((tid % (RN / 4)) ^ ((kb & 1) << 3)) * 4;
    const int ns = (K + BK - 1) / BK, nk = K - (ns - 1) * BK;          // k of the last slab
    const unsigned am = (unsigned)min(m0 + ca, M - 4) * 4, bn = (unsigned)min(n0 + cb, N - 4) * 4;
    const unsigned lds0 = (unsigned)(size_t)(__attribute__((address_space(3))) float *)slabs + wave * 1024;
    auto load = [&](int s, int b, int i) {               // slabs past the end re-read the last one, rows past K the last row
      const bool of_a = i < XA;
      const int k = of_a ? ka + PA * i : kb + PB * (i - XA);
      const int kc = s >= ns - 1 ? min(k, nk - 1) : k;
      const unsigned off = (unsigned)kc * (unsigned)((of_a ? lda : ldb) * 4) + (of_a ? am : bn);
      asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" ::"s"(lds0 + (b * XSLAB + (of_a ? i * PA * RM : BK * RM + (i - XA) * PB * RN)) * 4),
                   "v"(off), "s"((of_a ? A : B) + (size_t)min(s, ns - 1) * BK * (of_a ? lda : ldb))
                   : "memory");
    };
    wm = (wave / WN) * 32 * TM;
    wn = (wave % WN) * 32 * TN;
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;
    const int row = lane & 31, h = lane >> 5;
    float fa[2][BK / 2][TM], fb[2][BK / 2][TN];
    auto read = [&](int f, int b, int n) {
      const int e = n / (TM + TN), i = n % (TM + TN);
      if (i < TM) {
        const int x = wm + 32 * i + row;
        fa[f][e][i < TM ? i : 0] = slabs[b * XSLAB + (2 * e + h) * RM + (((x >> 2) ^ (h << 3)) << 2) + (x & 3)];
      } else {
        const int x = wn + 32 * (i - TM) + row;
        fb[f][e][i < TM ? 0 : i - TM] = slabs[b * XSLAB + BK * RM + (2 * e + h) * RN + (((x >> 2) ^ (h << 3)) << 2) + (x & 3)];
      }
    };
    auto mul = [&](int f, int n) {
      const int e = n / (TM * TN), i = n / TN % TM, j = n % TN;
      acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(fa[f][e][i], fb[f][e][j], acc[i][j], 0, 0, 0);
    };
    constexpr int NM = BK / 2 * TM * TN, NR = BK / 2 * (TM + TN);
    constexpr int RB = (NR + NM - 3) / (NM - 2), LB = (XL + NM - 3) / (NM - 2);
    auto step = [&](int s, int u) {                      // as in run
      const int f = u & 1;
#pragma unroll
      for (int n = 0; n < NM; ++n) {
        __builtin_amdgcn_sched_barrier(0);
        mul(f, n);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int r = n * RB; r < min(n * RB + RB, NR); ++r) read(f ^ 1, (u + 1) % NS, r);
#pragma unroll
        for (int l = n * LB; l < min(n * LB + LB, XL); ++l) load(s + NS, u, l);
        if (n == NM - 2) slab_barrier<(NS - 2) * XL>();
      }
    };
#pragma unroll
    for (int b = 0; b < NS; ++b)
#pragma unroll
      for (int i = 0; i < XL; ++i) load(b, b, i);
    slab_barrier<(NS - 2) * XL>();
#pragma unroll
    for (int r = 0; r < NR; ++r) read(0, 0, r);
    slab_barrier<(NS - 2) * XL>();
    int s = 0;
    for (; s + NS < ns; s += NS) {
#pragma unroll
      for (int u = 0; u < NS; ++u) step(s + u, u);
    }
#pragma unroll
    for (int u = 0; u < NS; ++u) {
      if (s + u + 1 < ns) {
        step(s + u, u);
      } else if (s + u < ns) {                           // no slab follows; an odd K leaves half a pair
        const int f = u & 1;
#pragma unroll
        for (int e = 0; e < BK / 2; ++e) {
          if (2 * e >= nk) break;
          const bool in = 2 * e + h < nk;
#pragma unroll
          for (int i = 0; i < TM; ++i) fa[f][e][i] = in ? fa[f][e][i] : 0.f;
#pragma unroll
          for (int j = 0; j < TN; ++j) fb[f][e][j] = in ? fb[f][e][j] : 0.f;
#pragma unroll
          for (int n = 0; n < TM * TN; ++n) mul(f, e * TM * TN + n);
        }
      }
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  }
};

}  // namespace qc
