// Split-K kernel for launches that leave the chip idle.  With a few hundred rows a 128 x 128 tile grid has fewer tiles than
// compute units and every workgroup walks the whole of K through barriers, 0.5 us per 128 bytes of K whatever the matrix
// rate.  Here the tile is small (32 TM x 32 TN, about one per compute unit) and the NW wavefronts of a workgroup share its
// K: wavefront w takes the 128-byte chunks w, w + NW, ... of K and accumulates the whole tile over them, alone and without
// barriers; the partial sums (exact integers) meet in LDS at the end, wavefront b finishing block b.
//   * activations: a wavefront loads 8 rows x 128 bytes per instruction (whole cache lines: 32 rows x 32 bytes, the fragment
//     shape, was measured at 18 instead of 60 bytes per clock and compute unit), writes them to a private LDS area (LDS
//     operations of one wavefront complete in order: no barrier, one buffer) and reads fragments back.  Rows are 128 bytes,
//     16-byte chunks swizzled with the row's low three bits (conflict-free writes and reads).
//   * weights in fragment order go straight to registers; row-major ones (WROW: the caller's matrix of qc_w8a8_linear) take
//     the activations' way.
//   * the first chunks (split_depth) are requested at once; from then on the activations of that many chunks are ahead of the one that is
//     multiplied, the weights of one less: their registers are free only behind the products.
// What bounds it: with few rows the round trips to weights that lie in HBM and the fixed costs around them (launch, reduction,
// epilogue).  With 1024 rows no unit: fc2 of 1024 x 1152 x 4608 (64 x 96 tiles, 18.3 us) has 192 of 256 compute units at work, each
// drawing 737 KB, 17 bytes a clock of the 60 its L2 gives, with 9 % of the matrix pipes busy; what it waits for there is not shown.
#include "gemm_i8_epilogue.h"

namespace qc {

// Columns of the wavefront grid that finishes a tile of tm x tn blocks: as many wavefronts as divide the blocks evenly
constexpr int split_em(int tm, int tn, int nw) {
  int best = 1, em_best = 1;
  for (int em = 1; em <= tm; ++em)
    for (int en = 1; en <= tn; ++en)
      if (tm % em == 0 && tn % en == 0 && em * en <= nw && em * en > best) { best = em * en; em_best = em; }
  return em_best;
}
constexpr int split_en(int tm, int tn, int nw) {
  int best = 1;
  const int em = split_em(tm, tn, nw);
  for (int en = 1; en <= tn; ++en)
    if (tn % en == 0 && em * en <= nw) best = en;
  return best;
}

// Chunks of a wavefront that are requested before it multiplies the first, and register sets.  What a launch of few tiles waits for are round
// trips to weights that lie in HBM, one after the other; K = 1152 is three chunks a wavefront.  32 x 64 tiles of which a compute unit has
// several keep to one: 112 registers, four workgroups a unit (two chunks, 160 and three, against that: QKV of 425 x 1152 x 1152 11.6 -> 9.9 us, fc2
// of 512 x 8192 x 2048 25.0 -> 23.9; 425 tokens of width 1152, 24 blocks, 7718 -> 7431 us, 8 latents 10235 -> 10081; three chunks were another 10 - 18 %
// slower).  32 x 32 tiles have one or two chunks a wavefront up to K = 2048, 64 x 64 ones no registers for a third, a 64 x 96 tile's third gained
// nothing.  Row-major weights go through LDS, one.
// One latent of 256 tokens, 50 steps, one chunk everywhere | this: 39.4 | 38.4 ms (proj and fc2 together 17.0 | 16.4 us).
constexpr int split_depth(int tm, int tn, bool few, bool wrow) { return wrow ? 1 : tm * tn == 2 ? (few ? 3 : 1) : 2; }

// whether a kernel differs with FEW
constexpr bool split_few(int tm, int tn, bool wrow) { return !wrow && tm * tn <= 2; }

// FEW: no more tiles than compute units (32 x 32 tiles are never more than 126; false for the kernels that are the same either way).
template <int TM, int TN, int NW, int EPI, bool W4, bool WROW, bool RBF, bool FEW>
__global__ __launch_bounds__(64 * NW, (NW <= 4 && TM * TN <= 4) ? 2 : 1) void gemm_i8_split_kernel(GemmArgs p) {
  constexpr int BM = 32 * TM, BN = 32 * TN, NB = TM * TN, CK = 128;
  constexpr int EM = split_em(TM, TN, NW), EN = split_en(TM, TN, NW);   // wavefront grid of the epilogue
  static_assert(EM * EN <= NW && TM % EM == 0 && TN % EN == 0, "every block needs a wavefront that finishes it");
  constexpr int PF = split_depth(TM, TN, FEW, WROW);
  constexpr int WREG = (BM + (WROW ? BN : 0)) * CK;                // private LDS bytes of a wavefront
  extern __shared__ __align__(16) unsigned char smem[];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int tiles_m = (p.M + BM - 1) / BM, tiles_n = (p.N + BN - 1) / BN;
  const int xm = p.xcd_m, xn = NUM_XCD / xm;                       // XCD grid over the tile grid, as in the tile kernel
  const int cm = (tiles_m + xm - 1) / xm, cn = (tiles_n + xn - 1) / xn;
  const int xcd = blockIdx.x % NUM_XCD, local = blockIdx.x / NUM_XCD;
  const int tm = (xcd % xm) * cm + local % cm, tn = (xcd / xm) * cn + local / cm;
  if (tm >= tiles_m || tn >= tiles_n) return;
  const int m0 = __builtin_amdgcn_readfirstlane(tm * BM), n0 = __builtin_amdgcn_readfirstlane(tn * BN);

  const int nc = (p.K + CK - 1) / CK;
  const int mine = (nc - wave + NW - 1) / NW;                      // chunks of this wavefront (may be 0)
  const int lrow = lane >> 3, lc = lane & 7;                       // row within a pass of 8 rows, 16-byte chunk
  unsigned aoff[TM * 4], boff[WROW ? TN * 4 : 1];
#pragma unroll
  for (int i = 0; i < TM * 4; ++i) aoff[i] = (unsigned)(min(m0 + 8 * i + lrow, p.M - 1) - m0) * (unsigned)p.lda + (WROW ? 0 : lc * 16);
  if constexpr (WROW) {
#pragma unroll
    for (int i = 0; i < TN * 4; ++i) boff[i] = (unsigned)(min(n0 + 8 * i + lrow, p.N - 1) - n0) * (unsigned)(W4 ? p.K >> 1 : p.K);
  }
  const int8_t *abase = p.A + (size_t)m0 * p.lda;
  constexpr int FRAG = W4 ? 512 : 1024;                            // bytes per weight fragment
  typedef typename std::conditional<W4, v2i, v4i>::type wload_t;
  const int ng = p.K / 32, nblocks = p.N / 32;
  const int bl0 = n0 / 32;                                         // (n0 < N: the tile's first block of columns exists)
  const unsigned char *wbase = WROW ? (const unsigned char *)p.W + (size_t)n0 * (W4 ? p.K >> 1 : p.K)
                                    : (const unsigned char *)p.Wt + (size_t)bl0 * ng * FRAG;
  // buffer loads: a lane's offset in one register, the chunk's in a scalar one, no 64-bit address a load
  const auto abuf = __builtin_amdgcn_make_buffer_rsrc((void *)abase, 0, -1, 0x00027000);
  const auto wbuf = __builtin_amdgcn_make_buffer_rsrc((void *)wbase, 0, -1, 0x00027000);
  int woff[TN];
#pragma unroll
  for (int j = 0; j < TN; ++j) woff[j] = (min(bl0 + j, nblocks - 1) - bl0) * ng * FRAG;
  unsigned char *sA = smem + wave * WREG, *sB = sA + BM * CK;
  v4i ra[PF][TM * 4];
  wload_t rb[PF][TN * 4];                                          // WROW: used until the chunk is in LDS
  auto load_a = [&](int set, int c) {
    if constexpr (WROW) {
      const unsigned k = (unsigned)min(c * CK + lc * 16, p.K - 16);  // beyond K: re-read the end, zeroed in store_a
#pragma unroll
      for (int i = 0; i < TM * 4; ++i) ra[set][i] = *(const v4i *)(abase + aoff[i] + k);
    } else {                                                       // K is whole chunks
#pragma unroll
      for (int i = 0; i < TM * 4; ++i) ra[set][i] = __builtin_bit_cast(v4i, __builtin_amdgcn_raw_buffer_load_b128(abuf, aoff[i], c * CK, 0));
    }
  };
  auto load_b = [&](int set, int c) {
    if constexpr (WROW) {
      const unsigned k = (unsigned)min(c * CK + lc * 16, p.K - 16);
#pragma unroll
      for (int i = 0; i < TN * 4; ++i) rb[set][i] = *(const wload_t *)(wbase + boff[i] + (W4 ? k >> 1 : k));
    } else {
#pragma unroll
      for (int j = 0; j < TN; ++j)
#pragma unroll
        for (int g = 0; g < 4; ++g) {
          const int so = woff[j] + (c * 4 + g) * FRAG;
          if constexpr (W4) rb[set][j * 4 + g] = __builtin_bit_cast(v2i, __builtin_amdgcn_raw_buffer_load_b64(wbuf, lane * 8, so, 0));
          else rb[set][j * 4 + g] = __builtin_bit_cast(v4i, __builtin_amdgcn_raw_buffer_load_b128(wbuf, lane * 16, so, 0));
        }
    }
  };
  auto store_a = [&](int set, int c) {
    const bool zero = WROW && c * CK + lc * 16 >= p.K;
#pragma unroll
    for (int i = 0; i < TM * 4; ++i) *(v4i *)(sA + (8 * i + lrow) * CK + ((lc ^ lrow) * 16)) = zero ? (v4i){0, 0, 0, 0} : ra[set][i];
    if constexpr (WROW) {
#pragma unroll
      for (int i = 0; i < TN * 4; ++i) {
        v4i v;
        if constexpr (W4) v = unpack_w4(rb[set][i]);
        else v = rb[set][i];
        *(v4i *)(sB + (8 * i + lrow) * CK + ((lc ^ lrow) * 16)) = v;
      }
    }
  };
  v16i acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][j][r] = 0;
  const int frow = lane & 31, fh = lane >> 5;
  auto compute = [&](int set) {
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      v4i fa[TM], fb[TN];
#pragma unroll
      for (int i = 0; i < TM; ++i) fa[i] = *(const v4i *)(sA + (32 * i + frow) * CK + (((2 * g + fh) ^ (frow & 7)) * 16));
#pragma unroll
      for (int j = 0; j < TN; ++j) {
        if constexpr (WROW) fb[j] = *(const v4i *)(sB + (32 * j + frow) * CK + (((2 * g + fh) ^ (frow & 7)) * 16));
        else if constexpr (W4) fb[j] = unpack_w4(rb[set][j * 4 + g]);
        else fb[j] = rb[set][j * 4 + g];
      }
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) {
          if (EPI == EPI_GELU_Q) acc[i][j] = __builtin_amdgcn_mfma_i32_32x32x32_i8(fb[j], fa[i], acc[i][j], 0, 0, 0);
          else acc[i][j] = __builtin_amdgcn_mfma_i32_32x32x32_i8(fa[i], fb[j], acc[i][j], 0, 0, 0);
        }
    }
  };
  // straight-line steps: chunk c is in registers (set); they are requested anew for chunk c + PF NW as they become free, the activations'
  // once they are in LDS, the weights' once they are multiplied (WROW: with the activations')
  auto step = [&](int set, int c) {
    const int next = WROW ? c + NW : min(c + PF * NW, nc - 1);     // (beyond the last chunk: not used; WROW: there is one)
    store_a(set, c);
    load_a(set, next);
    if constexpr (WROW) load_b(set, next);
    __builtin_amdgcn_sched_barrier(0);
    compute(set);
    if constexpr (!WROW) {
      __builtin_amdgcn_sched_barrier(0);
      load_b(set, next);
    }
  };
  auto last = [&](int set, int c) {
    store_a(set, c);
    compute(set);
  };
  auto request = [&](int d) {
    load_a(d, wave + d * NW);
    load_b(d, wave + d * NW);
  };
  // Nothing covers a round trip to memory behind the sums of a lone workgroup: what the epilogue reads comes in behind the first
  // chunk.  (Not for the larger tiles, which have no registers left for it; the residual stream's elements only where a unit has one
  // workgroup, and not where they may be bfloat16: converting would wait for them.)  One latent of 256 tokens, 50 steps: 40.5 ->
  // 39.3 ms; with 64 x 64 tiles and the stream's elements on every launch 39.5, and 8 latents 81.3 -> 83.0.
  constexpr bool PRE = !WROW && TM * TN <= 2, PREX = PRE && FEW && EPI == EPI_RESID && !RBF;
  EpiPre<EPI, TM / EM, TN / EN, PREX> pre;
  if constexpr (WROW) {
    // one chunk in flight, two steps a turn of the loop.  As the others (below; one step a turn, the epilogue's loads in front), float32 linears
    // of 1 to 2048 rows took 3 % longer on average, 4-bit ones up to 11 %: 500 x 1152 x 4608 13.1 -> 14.6 us
    if (mine > 0) {
      load_a(0, wave);
      load_b(0, wave);
      int c = wave, left = mine;
      for (; left > 2; left -= 2, c += 2 * NW) {
        step(0, c);
        step(0, c + NW);
      }
      if (left == 2) {
        step(0, c);
        last(0, c + NW);
      } else {
        last(0, c);
      }
    }
  } else {
    load_a(0, min(wave, nc - 1));                                    // (a wavefront without a chunk makes no use of it)
    load_b(0, min(wave, nc - 1));
    if constexpr (PRE) {
      __builtin_amdgcn_sched_barrier(0);
      epilogue_request<BM, BN, EM, EN, EPI, PREX>(p, pre, min(wave, EM * EN - 1), m0, n0);
      __builtin_amdgcn_sched_barrier(0);
    }
    // a path of its own for fewer than PF chunks: where paths with different numbers of loads in flight meet, the compiler waits for more
    // than it has to
    if (mine >= PF) {
#pragma unroll
      for (int d = 1; d < PF; ++d) request(d);
      __builtin_amdgcn_sched_barrier(0);
      int c = wave, left = mine;
      for (; left > PF; left -= PF, c += PF * NW) {
#pragma unroll
        for (int d = 0; d < PF; ++d) step(d, c + d * NW);
      }
      last(0, c);
      if constexpr (PF > 1) {
        if (left > 1) {
          last(1, c + NW);
          if constexpr (PF > 2) {
            if (left > 2) last(2, c + 2 * NW);
          }
        }
      }
    } else if (PF > 2 && mine == 2) {
      if constexpr (PF > 2) {
        request(1);
        __builtin_amdgcn_sched_barrier(0);
        last(0, wave);
        last(1, wave + NW);
      }
    } else if (mine == 1) {
      last(0, wave);
    }
  }

  // ---- the partial sums meet.  A block is 64 lanes x 16 integers, stored as 4 x [64 lanes][4].
  int *red = (int *)smem;
  auto put = [&](int slot, const v16i &v) {
#pragma unroll
    for (int q = 0; q < 4; ++q) *(v4i *)(red + ((slot * 4 + q) * 64 + lane) * 4) = (v4i){v[4 * q], v[4 * q + 1], v[4 * q + 2], v[4 * q + 3]};
  };
  auto add = [&](int slot, v16i &v) {
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const v4i t = *(const v4i *)(red + ((slot * 4 + q) * 64 + lane) * 4);
#pragma unroll
      for (int e = 0; e < 4; ++e) v[4 * q + e] += t[e];
    }
  };
  constexpr bool HALVE = NB * NW > 16;                             // more than 64 KB of partial sums: fold the upper half first
  constexpr int NS = HALVE ? NW / 2 : NW;                          // wavefronts that hold partial sums after that
  static_assert(!HALVE || NW % 2 == 0, "the upper half folds onto the lower one");
  __syncthreads();                                                 // every wavefront is past its fragments
  if constexpr (HALVE) {
    if (wave >= NS) {
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) put((wave - NS) * NB + i * TN + j, acc[i][j]);
    }
    __syncthreads();
    if (wave < NS) {
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) add(wave * NB + i * TN + j, acc[i][j]);
    }
    __syncthreads();
  }
  if (wave < NS) {
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j) put(wave * NB + i * TN + j, acc[i][j]);
  }
  __syncthreads();
  constexpr int FM = TM / EM, FN = TN / EN;                        // blocks a finishing wavefront owns
  v16i fin[FM][FN];
  if (wave < EM * EN) {
#pragma unroll
    for (int i = 0; i < FM; ++i)
#pragma unroll
      for (int j = 0; j < FN; ++j) {
        const int b = ((wave / EN) * FM + i) * TN + (wave % EN) * FN + j;
#pragma unroll
        for (int r = 0; r < 16; ++r) fin[i][j][r] = 0;
#pragma unroll
        for (int s = 0; s < NS; ++s) add(s * NB + b, fin[i][j]);
      }
  }
  __syncthreads();                                                 // the sums are read: LDS is free for the epilogue
  if (wave >= EM * EN) return;                                     // (ended wavefronts do not count at its barriers)
  gemm_epilogue<BM, BN, EM, EN, EPI, RBF, PRE, PREX>(p, fin, smem, m0, n0, 0, &pre);
}

template <int TM, int TN, int NW, int EPI, bool W4, bool WROW, bool RBF = false>
static hipError_t launch_split(const GemmArgs &a, hipStream_t st) {
  if constexpr (EPI == EPI_RESID && !RBF) {
    if (a.x_bf16 || a.cache_bf16) return launch_split<TM, TN, NW, EPI, W4, WROW, true>(a, st);
  }
  constexpr int BM = 32 * TM, BN = 32 * TN, NB = TM * TN;
  constexpr int s_loop = NW * (BM + (WROW ? BN : 0)) * 128, s_red = (NB * NW > 16 ? NW / 2 : NW) * NB * 4096;
  constexpr int s_epi = EPI == EPI_GELU_Q ? BN * 12 + BM * (BN + 16) + 16 + GELU_FIX_CAP * 16 : 0;
  constexpr int smem = s_loop > s_red ? (s_loop > s_epi ? s_loop : s_epi) : (s_red > s_epi ? s_red : s_epi);
  static_assert(smem <= 160 * 1024, "LDS of a compute unit");
  static std::atomic<unsigned long long> lds[2];
  GemmArgs b = a;
  const int tiles_m = (a.M + BM - 1) / BM, tiles_n = (a.N + BN - 1) / BN;
  const bool few = split_few(TM, TN, WROW) && (TM * TN == 1 || (long long)tiles_m * tiles_n <= 256);
  auto kern = gemm_i8_split_kernel<TM, TN, NW, EPI, W4, WROW, RBF, split_few(TM, TN, WROW)>;
  if constexpr (split_few(TM, TN, WROW) && TM * TN > 1)
    if (!few) kern = gemm_i8_split_kernel<TM, TN, NW, EPI, W4, WROW, RBF, false>;
  if (const hipError_t e = allow_lds((const void *)kern, smem, lds[few])) return e;
  b.xcd_m = xcd_rows(tiles_m, tiles_n, (double)a.M * a.K, (double)a.N * a.K * (W4 ? 0.5 : 1.0));
  const int cm = (tiles_m + b.xcd_m - 1) / b.xcd_m, xn = NUM_XCD / b.xcd_m, cn = (tiles_n + xn - 1) / xn;
  hipLaunchKernelGGL(kern, dim3(NUM_XCD * cm * cn), dim3(64 * NW), smem, st, b);
  return hipGetLastError();
}

// The rule, from launches alone on the chip with weights read from memory (DiT-XL/2 linears, us, this kernel against the tile
// kernel): M = 256: QKV 8.3 / 11.6, proj 5.1 / 10.1, fc1 8.8 / 11.7, fc2 9.8 / 25.5; M = 512: 10.9 / 12.0, 6.5 / 11.4,
// 13.0 / 11.9, 12.1 / 25.2; M = 1024: 18.3 / 14.9, 8.5 / 10.9, 19.1 / 18.2, 16.4 / 25.6; M = 2048: 31 / 20, 12.3 / 11.8,
// 31 / 24, 26.9 / 26.4.  In tiles of 64 x 64 (M / 64 x N / 64) it wins up to about 450; beyond, a compute unit gets several
// tiles one after the other and their fixed costs add up.
bool gemm_split_pays(const GemmArgs &a, int epi, int nz) {
  if (nz != 1 || a.sel_D || a.K % 16 || a.lda % 16) return false;
  if (epi == EPI_F32 ? a.Wt != nullptr : (!a.Wt || a.K % 128 || a.N % 32)) return false;
  return (long long)((a.M + 63) / 64) * ((a.N + 63) / 64) <= 450;
}

template <int EPI, bool W4>
static hipError_t launch_tile(const GemmArgs &a, hipStream_t st) {
  constexpr bool WROW = EPI == EPI_F32;
  const long long t64 = (long long)((a.M + 63) / 64) * ((a.N + 63) / 64);
  const long long t32 = (long long)((a.M + 31) / 32) * ((a.N + 63) / 64);
  // the smallest tile that still leaves a workgroup for every few compute units: 64 rows, 32 rows, 32 x 32 with the K of a
  // tile cut eight ways
  if (t32 < 64) return launch_split<1, 1, 8, EPI, W4, WROW>(a, st);
  if (t64 < 128) return launch_split<1, 2, 4, EPI, W4, WROW>(a, st);
  if constexpr (EPI == EPI_RESID) {
    // slightly more 64 x 64 tiles than compute units and a long K: 64 x 96 tiles take one turn instead of two (fc2 at
    // M = 1024: 16.4 against 19.1 us)
    const long long t96 = (long long)((a.M + 63) / 64) * ((a.N + 95) / 96);
    if (t64 > 256 && t96 <= 256 && a.K >= 2048) return launch_split<2, 3, 4, EPI, W4, WROW>(a, st);
  }
  // about as many 64 x 64 tiles as compute units and more: some unit gets two, one after the other, where several 32 x 64 tiles share it
  // (64 x 64 | 32 x 64, us between events: 252 tiles, M = 850: proj 14.5 | 12.6, fc2 23.7 | 20.9; 288: fc1 at M = 256 12.2 | 11.5, 4-bit 13.2 |
  // 12.8, QKV of width 384 at M = 1024 10.8 | 10.2; 384: fc1 there 10.5 | 10.0; but 216: fc2 at M = 768 16.3 | 18.0, QKV at M = 256 10.8 | 11.2)
  if (EPI != EPI_F32 && t64 > 232) return launch_split<1, 2, 4, EPI, W4, WROW>(a, st);
  return launch_split<2, 2, 4, EPI, W4, WROW>(a, st);
}

template <int EPI>
static hipError_t launch_bits(const GemmArgs &a, hipStream_t st) {
  return a.w4 ? launch_tile<EPI, true>(a, st) : launch_tile<EPI, false>(a, st);
}

hipError_t launch_gemm_split(const GemmArgs &a, int epi, hipStream_t st) {
  switch (epi) {
    case EPI_GELU_Q: return launch_bits<EPI_GELU_Q>(a, st);
    case EPI_RESID: return launch_bits<EPI_RESID>(a, st);
    case EPI_QKV: return launch_bits<EPI_QKV>(a, st);
    default: return launch_bits<EPI_F32>(a, st);
  }
}

}  // namespace qc
