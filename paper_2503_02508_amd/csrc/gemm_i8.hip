// int8 x int8 -> int32 GEMM on the gfx950 matrix cores (v_mfma_i32_32x32x32_i8)
// with the dequantise / GELU+requantise / cache-store+gated-residual epilogues
// of the quantised linears of a DiT block.
//
//   acc[m, n] = sum_k A[m, k] * W[n, k]          A: activation codes, W: weight codes
//   v[m, n]   = a_s * w_s[n] * (acc - a_z * wsum[n]) + bias[n]
//
// Tiling: a workgroup of 4 or 8 wavefronts owns a BM x BN tile of the
// output and walks K in slabs of 128 bytes.  Both operands are K-contiguous, so
// a slab row is 8 sixteen-byte chunks.  Slabs are staged in LDS (rows padded by
// 16 bytes so the 128-bit fragment reads of 8 neighbouring rows fall in 8
// different bank groups), two LDS buffers.  Global loads run PF slabs ahead of
// the MFMAs through a rotating set of registers: memory latency on this part
// is a few slab-times, so one slab of prefetch leaves the matrix cores idle.
//
// MFMA operand layout (32x32x32 i8): lane l supplies 16 bytes of row (l % 32)
// of either operand for k-group (l / 32); the products pair byte j of group g
// of both operands, so any k order works as long as both use the same one.
// Result layout: register r of lane l is row (r/4)*8 + (l/32)*4 + r%4 of the
// first operand, column l % 32 of the second.  The fp32 epilogues put the
// activations first (a lane owns one output column n, 32 lanes write 128
// contiguous bytes of a row); the int8 epilogue puts the weights first (a lane
// owns one row m and four consecutive n per register group, packed to a dword,
// staged through LDS and written out as 16-byte chunks).
//
// Workgroup -> tile mapping is XCD-aware: hardware deals workgroups round-robin
// to the 8 XCDs, each with its own L2; the mapping gives every XCD a contiguous
// range of weight panels so that a panel is fetched into one L2 only.
#include "gemm_i8_epilogue.h"

namespace qc {

template <int BM, int BN, int WM, int WN, int EPI, int TAG, bool W4, int PF, int BK, bool RBF>
__global__ __launch_bounds__(64 * WM * WN, (WM * WN == 4 && BM * BN <= 128 * 128) ? 2 : 1) void gemm_i8_kernel(GemmArgs p) {
  constexpr int WTM = BM / WM, WTN = BN / WN;
  constexpr int TM = WTM / 32, TN = WTN / 32;
  constexpr int NT = 64 * WM * WN;            // threads per workgroup
  constexpr int LDS_ROW = BK + 16;            // padded slab row in LDS
  constexpr int CPR = BK / 16;                // 16-byte chunks per slab row
  constexpr int RP = NT / CPR;                // slab rows covered by one pass of the workgroup
  constexpr int PA = BM / RP, PB = BN / RP;   // 16-byte chunks per thread per slab
  static_assert(TM >= 1 && TN >= 1 && PA >= 1 && PB >= 1, "tile too small for the workgroup");
  extern __shared__ __align__(16) unsigned char smem[];
  unsigned char *sA = smem;
  unsigned char *sB = smem + 2 * BM * LDS_ROW;

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int z = blockIdx.z;
  const int ncover = p.sel_D ? 2 * p.sel_D : p.N;
  const int tiles_m = (p.M + BM - 1) / BM;
  // XCD-aware order: workgroup b runs on XCD b % 8.  The 8 XCDs form an xm x xn
  // grid over the tile grid; each XCD owns a contiguous block of cm x cn tiles,
  // so an activation panel is fetched by xn L2s and a weight panel by xm L2s.
  const int tiles_n = (ncover + BN - 1) / BN;
  const int xm = p.xcd_m, xn = NUM_XCD / xm;
  const int cm = (tiles_m + xm - 1) / xm, cn = (tiles_n + xn - 1) / xn;
  const int xcd = blockIdx.x % NUM_XCD, local = blockIdx.x / NUM_XCD;
  const int tm = (xcd % xm) * cm + local % cm, tn = (xcd / xm) * cn + local / cm;
  if (tm >= tiles_m || tn >= tiles_n) return;
  const int m0 = tm * BM;
  const int n0 = tn * BN;
  const int wm0 = (wave / WN) * WTM, wn0 = (wave % WN) * WTN;

  const int8_t *A = p.A + (long long)z * p.zs_A;
  const unsigned char *W = (const unsigned char *)p.W + (long long)z * p.zs_W;   // byte stride
  const int w_row_bytes = W4 ? (p.K >> 1) : p.K;

  // Loads never branch: rows outside the matrix are clamped to the last row
  // (their products land in accumulators that are never stored) and the
  // chunks of a ragged last slab are clamped in k and zeroed by a select.
  const int lr = tid / CPR, lc = tid % CPR;   // slab row (per pass of RP rows) and chunk of this thread
  unsigned oa[PA], ob[PB];                  // byte offsets of this thread's chunk rows
#pragma unroll
  for (int i = 0; i < PA; ++i) oa[i] = (unsigned)min(m0 + lr + RP * i, p.M - 1) * (unsigned)p.lda;
#pragma unroll
  for (int i = 0; i < PB; ++i) ob[i] = (unsigned)map_col(min(n0 + lr + RP * i, ncover - 1), p.sel_D) * (unsigned)w_row_bytes;
  typedef typename std::conditional<W4, v2i, v4i>::type wload_t;
  v4i ra[PF][PA];
  wload_t rb[PF][PB];

  // The loaded values are not touched until store_slab, so that nothing waits
  // on a load right after issuing it.
  auto load_slab = [&](int s, int k0, bool ragged) {
    int k = k0 + lc * 16;
    if (ragged) k = min(k, p.K - 16);
#pragma unroll
    for (int i = 0; i < PA; ++i) ra[s][i] = *(const v4i *)(A + oa[i] + k);
#pragma unroll
    for (int i = 0; i < PB; ++i) {
      if (W4) *(v2i *)&rb[s][i] = *(const v2i *)(W + ob[i] + (k >> 1));
      else *(v4i *)&rb[s][i] = *(const v4i *)(W + ob[i] + k);
    }
  };
  auto store_slab = [&](int s, int buf, bool zero) {   // zero: this thread's chunk lies beyond K
#pragma unroll
    for (int i = 0; i < PA; ++i)
      *(v4i *)(sA + (buf * BM + lr + RP * i) * LDS_ROW + lc * 16) = zero ? (v4i){0, 0, 0, 0} : ra[s][i];
#pragma unroll
    for (int i = 0; i < PB; ++i) {
      v4i v;
      if (W4) v = unpack_w4(*(v2i *)&rb[s][i]);
      else v = *(v4i *)&rb[s][i];
      *(v4i *)(sB + (buf * BN + lr + RP * i) * LDS_ROW + lc * 16) = zero ? (v4i){0, 0, 0, 0} : v;
    }
  };

  // the same, one quarter at a time (chunk c of the PA + PB chunks belongs to part c % NPART): lets the
  // steady-state step spread its memory instructions between the MFMA groups
  constexpr int NPART = BK / 32;
  auto load_part = [&](int s, int k0, int part) {
    const int k = k0 + lc * 16;
#pragma unroll
    for (int i = 0; i < PA; ++i)
      if (i % NPART == part) ra[s][i] = *(const v4i *)(A + oa[i] + k);
#pragma unroll
    for (int i = 0; i < PB; ++i)
      if ((PA + i) % NPART == part) {
        if (W4) *(v2i *)&rb[s][i] = *(const v2i *)(W + ob[i] + (k >> 1));
        else *(v4i *)&rb[s][i] = *(const v4i *)(W + ob[i] + k);
      }
  };
  auto store_part = [&](int s, int buf, int part) {
#pragma unroll
    for (int i = 0; i < PA; ++i)
      if (i % NPART == part) *(v4i *)(sA + (buf * BM + lr + RP * i) * LDS_ROW + lc * 16) = ra[s][i];
#pragma unroll
    for (int i = 0; i < PB; ++i)
      if ((PA + i) % NPART == part) {
        v4i v;
        if (W4) v = unpack_w4(*(v2i *)&rb[s][i]);
        else v = *(v4i *)&rb[s][i];
        *(v4i *)(sB + (buf * BN + lr + RP * i) * LDS_ROW + lc * 16) = v;
      }
  };

  v16i acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][j][r] = 0;

  const int nk = (p.K + BK - 1) / BK;
  const bool k_ragged = (p.K % BK) != 0;
  const int frow = lane & 31, fk = (lane >> 5) * 16;

  auto compute = [&](int cur) {
    const unsigned char *a_base = sA + (cur * BM + wm0 + frow) * LDS_ROW + fk;
    const unsigned char *b_base = sB + (cur * BN + wn0 + frow) * LDS_ROW + fk;
#pragma unroll
    for (int kk = 0; kk < BK / 32; ++kk) {
      v4i fa[TM], fb[TN];
#pragma unroll
      for (int i = 0; i < TM; ++i) fa[i] = *(const v4i *)(a_base + i * 32 * LDS_ROW + kk * 32);
#pragma unroll
      for (int j = 0; j < TN; ++j) fb[j] = *(const v4i *)(b_base + j * 32 * LDS_ROW + kk * 32);
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) {
          if (EPI == EPI_GELU_Q)
            acc[i][j] = __builtin_amdgcn_mfma_i32_32x32x32_i8(fb[j], fa[i], acc[i][j], 0, 0, 0);
          else
            acc[i][j] = __builtin_amdgcn_mfma_i32_32x32x32_i8(fa[i], fb[j], acc[i][j], 0, 0, 0);
        }
    }
  };

  // One steady-state step, software-pipelined inside the wavefront.  LDS reads have a latency of a few
  // hundred cycles and a wavefront is alone on its SIMD when the launch has few workgroups, so a whole
  // slab of fragments (all NPART k-groups) is in flight at once: the reads of the next slab are issued
  // right after the barrier that publishes it, in front of the last MFMA group of the current slab, and a
  // quarter of the next slab's LDS stores and of the global loads PF slabs ahead is issued behind each
  // MFMA group, so that LDS and memory instructions execute under the matrix-core time.
  constexpr bool DEEP = TM * TN <= 4;          // a slab of fragments fits beside the accumulators
  v4i fa[DEEP ? NPART : 1][TM], fb[DEEP ? NPART : 1][TN];
  auto read_group = [&](int buf, int kk) {
    const unsigned char *a_base = sA + (buf * BM + wm0 + frow) * LDS_ROW + fk + kk * 32;
    const unsigned char *b_base = sB + (buf * BN + wn0 + frow) * LDS_ROW + fk + kk * 32;
#pragma unroll
    for (int i = 0; i < TM; ++i) fa[DEEP ? kk : 0][i] = *(const v4i *)(a_base + i * 32 * LDS_ROW);
#pragma unroll
    for (int j = 0; j < TN; ++j) fb[DEEP ? kk : 0][j] = *(const v4i *)(b_base + j * 32 * LDS_ROW);
  };
  auto mfma_group = [&](int kk) {
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j) {
        const int g = DEEP ? kk : 0;
        if (EPI == EPI_GELU_Q)
          acc[i][j] = __builtin_amdgcn_mfma_i32_32x32x32_i8(fb[g][j], fa[g][i], acc[i][j], 0, 0, 0);
        else
          acc[i][j] = __builtin_amdgcn_mfma_i32_32x32x32_i8(fa[g][i], fb[g][j], acc[i][j], 0, 0, 0);
      }
  };
  // precondition: the fragment reads of slab kt (buffer kt & 1) have been issued
  auto step = [&](int s, int kt) {
    const int cur = kt & 1;
#pragma unroll
    for (int kk = 0; kk < NPART; ++kk) {
      if (kk + 1 < NPART) {
        __builtin_amdgcn_sched_barrier(0);
        mfma_group(kk);
      }
      __builtin_amdgcn_sched_barrier(0);
      store_part((s + 1) % PF, cur ^ 1, kk);
      load_part(s, (kt + PF) * BK, kk);
    }
    __builtin_amdgcn_sched_barrier(0);
    __syncthreads();
#pragma unroll
    for (int kk = 0; kk + 1 < NPART; ++kk) read_group(cur ^ 1, kk);
    __builtin_amdgcn_sched_barrier(0);
    mfma_group(NPART - 1);
    __builtin_amdgcn_sched_barrier(0);
    read_group(cur ^ 1, NPART - 1);
    __builtin_amdgcn_sched_barrier(0);
  };

  // Shallow variant for tiles whose accumulators leave no room for a slab of fragments: the fragments of
  // k-group kk+1 are read while the MFMAs of group kk run.
  auto step_shallow = [&](int s, int kt) {
    const int cur = kt & 1;
    const unsigned char *a_base = sA + (cur * BM + wm0 + frow) * LDS_ROW + fk;
    const unsigned char *b_base = sB + (cur * BN + wn0 + frow) * LDS_ROW + fk;
    v4i ga[2][TM], gb[2][TN];
#pragma unroll
    for (int i = 0; i < TM; ++i) ga[0][i] = *(const v4i *)(a_base + i * 32 * LDS_ROW);
#pragma unroll
    for (int j = 0; j < TN; ++j) gb[0][j] = *(const v4i *)(b_base + j * 32 * LDS_ROW);
#pragma unroll
    for (int kk = 0; kk < NPART; ++kk) {
      if (kk + 1 < NPART) {
#pragma unroll
        for (int i = 0; i < TM; ++i) ga[(kk + 1) & 1][i] = *(const v4i *)(a_base + i * 32 * LDS_ROW + (kk + 1) * 32);
#pragma unroll
        for (int j = 0; j < TN; ++j) gb[(kk + 1) & 1][j] = *(const v4i *)(b_base + j * 32 * LDS_ROW + (kk + 1) * 32);
      }
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) {
          if (EPI == EPI_GELU_Q)
            acc[i][j] = __builtin_amdgcn_mfma_i32_32x32x32_i8(gb[kk & 1][j], ga[kk & 1][i], acc[i][j], 0, 0, 0);
          else
            acc[i][j] = __builtin_amdgcn_mfma_i32_32x32x32_i8(ga[kk & 1][i], gb[kk & 1][j], acc[i][j], 0, 0, 0);
        }
      __builtin_amdgcn_sched_barrier(0);
      store_part((s + 1) % PF, cur ^ 1, kk);
      load_part(s, (kt + PF) * BK, kk);
      __builtin_amdgcn_sched_barrier(0);
    }
    __syncthreads();
  };

  // prologue: PF slabs in flight, slab 0 into LDS
#pragma unroll
  for (int s = 0; s < PF; ++s)
    if (s < nk) load_slab(s, s * BK, k_ragged && s == nk - 1);
  store_slab(0, 0, k_ragged && nk == 1 && lc * 16 >= p.K);
  __syncthreads();
  // main loop, unrolled by PF so that the register sets rotate with static indices:
  // at step kt LDS[kt & 1] holds slab kt, registers hold slabs kt+1 .. kt+PF-1.
  // Steady state is straight-line code (every step loads, computes, stores) so
  // that the wait before a store only covers the one slab it needs; the last
  // few steps run in a conditional tail.
  int kb = 0;
  const int nk_steady = k_ragged ? nk - 1 : nk;      // the ragged last slab is loaded by the tail (clamped, zero-filled)
  if (DEEP && 2 * PF - 1 < nk_steady) {
#pragma unroll
    for (int kk = 0; kk < NPART; ++kk) read_group(0, kk);
  }
  for (; kb + 2 * PF - 1 < nk_steady; kb += PF) {
#pragma unroll
    for (int s = 0; s < PF; ++s) {
      if (DEEP) step(s, kb + s);
      else step_shallow(s, kb + s);
    }
  }
  for (; kb < nk; kb += PF) {
#pragma unroll
    for (int s = 0; s < PF; ++s) {
      const int kt = kb + s;
      if (kt < nk) {
        if (kt + PF < nk) load_slab(s, (kt + PF) * BK, k_ragged && kt + PF == nk - 1);
        if (kt + 1 < nk) store_slab((s + 1) % PF, (kt + 1) & 1, k_ragged && kt + 2 == nk && (kt + 1) * BK + lc * 16 >= p.K);
        compute(kt & 1);
        __syncthreads();
      }
    }
  }

  gemm_epilogue<BM, BN, WM, WN, EPI, RBF>(p, acc, smem, m0, n0, z);
}

template <int BM, int BN, int WM, int WN, int EPI, int TAG, bool W4, int PF, int BK = 128, bool RBF = false>
static hipError_t launch_cfg(const GemmArgs &a, int nz, hipStream_t st) {
  // the residual epilogue is compiled for float32 stream and cache, and once more for the bfloat16 variants of either
  if constexpr (EPI == EPI_RESID && !RBF) {
    if (a.x_bf16 || a.cache_bf16) return launch_cfg<BM, BN, WM, WN, EPI, TAG, W4, PF, BK, true>(a, nz, st);
  }
  constexpr int smem_loop = 2 * (BM + BN) * (BK + 16);
  constexpr int smem_epi = BN * 12 + BM * (BN + 16) + 16 + GELU_FIX_CAP * 16;
  constexpr int smem = smem_loop > smem_epi ? smem_loop : smem_epi;
  static std::atomic<unsigned long long> lds{0};
  auto kern = gemm_i8_kernel<BM, BN, WM, WN, EPI, TAG, W4, PF, BK, RBF>;
  if (const hipError_t e = allow_lds((const void *)kern, smem, lds)) return e;
  const int ncover = a.sel_D ? 2 * a.sel_D : a.N;
  const int tiles_m = (a.M + BM - 1) / BM, tiles_n = (ncover + BN - 1) / BN;
  const int best_xm = xcd_rows(tiles_m, tiles_n, (double)a.M * a.K, (double)ncover * a.K * (W4 ? 0.5 : 1.0));
  GemmArgs b = a;
  b.xcd_m = best_xm;
  const int cm = (tiles_m + best_xm - 1) / best_xm, cn = (tiles_n + NUM_XCD / best_xm - 1) / (NUM_XCD / best_xm);
  const int grid = NUM_XCD * cm * cn;
  hipLaunchKernelGGL(kern, dim3(grid, 1, nz), dim3(64 * WM * WN), smem, st, b);
  return hipGetLastError();
}

template <int EPI, int TAG, bool W4>
static hipError_t launch_shape(const GemmArgs &a, int nz, hipStream_t st) {
  if (gemm_split_pays(a, EPI, nz)) return launch_gemm_split(a, EPI, st);
  if (a.M <= 32) return launch_cfg<32, 128, 1, 4, EPI, TAG, W4, 3>(a, nz, st);
  if (a.M <= 64) return launch_cfg<64, 128, 2, 2, EPI, TAG, W4, 3>(a, nz, st);
  // Fewer tiles than compute units: a workgroup is alone on its CU and a single wavefront per SIMD cannot
  // keep the LDS and memory pipes busy (they are issue-bound per wavefront), so the tile is shared by 8.
  // The residual epilogue keeps a tile of x in registers, which would leave the 4-wavefront variant one
  // workgroup per CU: it always runs on 8.
  // Inside a block the QKV product runs beside the other sub-batch's kernels: beyond half a chip of tiles it takes
  // the 4-wavefront variant, whose workgroups share a compute unit with the other stream's instead of queueing for a
  // free one (measured on the benchmark's sub-batches, 216 tiles: +1.8 % on the whole pass although the launch itself
  // takes 5 % longer).
  const int n_tiles = ((a.M + 127) / 128) * (((a.sel_D ? 2 * a.sel_D : a.N) + 127) / 128);
  if (EPI == EPI_RESID || n_tiles <= (EPI == EPI_QKV ? 128 : 256))
    return launch_cfg<128, 128, 2, 4, EPI, TAG, W4, 3>(a, nz, st);
  // Otherwise 4 wavefronts per tile and two workgroups per compute unit.
  return launch_cfg<128, 128, 2, 2, EPI, TAG, W4, 3>(a, nz, st);
}

template <int EPI, int TAG>
static hipError_t launch_epi(const GemmArgs &a, int nz, hipStream_t st) {
  return a.w4 ? launch_shape<EPI, TAG, true>(a, nz, st) : launch_shape<EPI, TAG, false>(a, nz, st);
}

// `site` only names the instantiation (so that profiles tell the linears apart).
hipError_t launch_gemm(const GemmArgs &a, int epi, int nz, hipStream_t st, int site) {
  if (gemm_big_pays(a, epi, nz)) return launch_gemm_big(a, epi, st, site);
  if (epi == EPI_GELU_Q) return launch_epi<EPI_GELU_Q, QC_SITE_FC1>(a, nz, st);
  if (epi == EPI_RESID)
    return site == QC_SITE_FC2 ? launch_epi<EPI_RESID, QC_SITE_FC2>(a, nz, st) : launch_epi<EPI_RESID, QC_SITE_PROJ>(a, nz, st);
  if (epi == EPI_QKV) return launch_epi<EPI_QKV, QC_SITE_QKV>(a, nz, st);
  return site == QC_SITE_ADA ? launch_epi<EPI_F32, QC_SITE_ADA>(a, nz, st) : launch_epi<EPI_F32, QC_SITE_QKV>(a, nz, st);
}

}  // namespace qc

