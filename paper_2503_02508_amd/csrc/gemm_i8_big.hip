// Large-M int8 GEMM: the quantised linears of a block at several thousand rows.
//
// Two things bound it.  A compute unit can pull 64 bytes a clock through its vector memory path and LDS writes run at a
// quarter of the read rate; and the chip is held at its power limit throughout (the four linears at M = 32768 run at 1.5 -
// 2.0 GHz), so that bytes moved and registers toggled cost time even where they hide behind the matrix cores.  Hence:
//   * v_mfma_i32_16x16x64_i8, not 32x32x32: half the accumulator bytes per operation; with random operands and nothing else to do
//     the chip sustains 4.1 against 3.4 Pop/s.  Consecutive products share one operand (the row blocks are walked forth and
//     back), which is worth another 2 %;
//   * tile 128 (M) x 256 (N), four wavefronts side by side along N, each 128 x 64 (8 x 4 blocks of 16 x 16), two workgroups
//     per compute unit so that one tile's prologue and epilogue run under the other's main loop.  A launch with too few of those
//     for the chip takes tiles of 64 rows (4 x 4 blocks a wavefront), which ask for their operands a slab earlier since a slab
//     lasts half as long (the rule and both sides' times stand at big_rows);
//   * weights never touch LDS: they are stored a second time in MFMA fragment order (fragment (n / 32, k / 32) = 64 lanes x
//     16 bytes, lane l = row n % 32 = l % 32, bytes 16 (l / 32) .. of the 32 k values; packed nibbles: 8 bytes per lane) and
//     each wavefront streams the fragments of its own 64 columns straight into registers, 128 k ahead;
//   * activations go global -> registers -> LDS in slabs of 128 bytes of K, so that a load instruction covers 8 whole
//     128-byte lines (slabs of 64 bytes, half lines, were 2 % slower over all), one slab in flight in registers, two slab
//     buffers in LDS.  The eight 16-byte chunks of a slab row are XOR-swizzled with bits 1..3 of the row: 16 rows of one
//     chunk then lie in 16 different slots of 256 bytes, free of bank conflicts;
//   * one barrier per slab; every memory instruction is issued behind an MFMA (pinned with scheduling barriers);
//   * memory is written 256 contiguous bytes at a time: a lane's accumulators are four adjacent columns of one row, so that 16
//     adjacent lanes cover 16 rows, and stores straight from them write every sector in four pieces (QKV / fc2 at M = 32768: 258
//     / 262 us; 4-byte stores of 16 adjacent columns with the operands swapped 193 / 222).  Each wavefront turns its blocks
//     through its own part of LDS instead, without barriers;
//   * per-column constants are fetched before the K loop (an epilogue that starts with two dependent round trips to memory
//     costs a tile about 2 of its 12 us) and the accumulators start at minus the zero-point term.
// Every global load of the loop is an ordinary register load issued through inline assembly (the compiler neither sees nor
// counts them); register loads complete in the order they were issued, so each wait on the vector memory counter below
// is the number of loads issued after the one it is for.
// (A variant that sent the activations straight to LDS (global_load_lds_dwordx4) was measured first and gave wrong fragments on
// some machines with counted waits; draining the counter before every barrier cost 8 % against this version.  That the two kinds
// of load complete out of order with respect to each other was taken for the cause and not shown.)
#include <algorithm>

#include "gemm_i8_epilogue.h"

namespace qc {

// a wait, tied to the registers that become valid with it: their uses cannot be moved above it
#define QC_WAIT_VM_FOR2(n, r0, r1) asm volatile("s_waitcnt vmcnt(" #n ")" : "+v"(r0), "+v"(r1)::"memory")
#define QC_WAIT_VM_FOR4(n, r0, r1, r2, r3) asm volatile("s_waitcnt vmcnt(" #n ")" : "+v"(r0), "+v"(r1), "+v"(r2), "+v"(r3)::"memory")
// all LDS writes of this wavefront done, then the workgroup barrier
#define QC_LDS_DONE_BARRIER asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory")
#define QC_SB __builtin_amdgcn_sched_barrier(0)

constexpr int BIG_BN = 256, BIG_BK = 128;
constexpr int BIG_TN = 4;                                                // 16 x 16 blocks of a wavefront: TM (8 or 4) x BIG_TN
constexpr int BIG_CST = 4 * BIG_BN;                                      // floats: per-column constants of the epilogue
template <int TM>
constexpr int big_smem_loop = 2 * 16 * TM * BIG_BK;                      // two activation slabs
constexpr int BIG_VR = 64 + 4;                                           // floats per staged V^T row (64 tokens)
constexpr int BIG_SMEM_QKV = 4 * 64 * BIG_VR * 4;                        // 64 features of each wavefront
constexpr int BIG_SROW = BIG_BN + 16;                                    // bytes per staged row of codes
constexpr int BIG_SMEM_RESID = 4 * 32 * (64 + 4) * 4;                    // 32 rows of each wavefront
constexpr int BIG_FIX_CAP = 1024;                                        // groups of four fc1 outputs decided again in float64, per tile
template <int TM>
constexpr int big_smem_gelu = 16 * TM * BIG_SROW + 16 + BIG_FIX_CAP * 32;

template <int TM>
using BigAcc = v4i[TM][BIG_TN];

// Epilogues.  acc[i][j] is the 16 x 16 block of rows m0 + 16 i .. and columns n0 + wn0 + 16 j ..; the weights are the first
// MFMA operand, so a lane holds row lane % 16 and the columns 4 (lane / 16) + e of a block.  cst: per-column constants in LDS,
// BIG_BN each of w_scale, bias and, for the residual, the gates of the first and of the next batch element.  RAG: the tile may
// end beyond the last row and may span two batch elements (which have at least as many rows as a tile); otherwise it is whole and
// inside one.

// Stores 16 bytes a lane at `off` bytes (a vector register) from the buffer's start.  The whole offset goes through the vector
// register on purpose.  A store reads its data registers a little after it has issued, so a vector instruction must not rewrite
// them in the next two issue slots; the compiler keeps that distance, except behind stores whose offset comes from a scalar
// register, and there this chip needs it too: (float) conversions issued right behind such a store replaced the first word of a
// few lanes' data about once in 300 launches.  One vector addition per store instead; no kernel's time changed measurably.
__device__ __forceinline__ void big_store16(v4u v, __amdgpu_buffer_rsrc_t buf, int off, bool nt) {
  if (nt) __builtin_amdgcn_raw_buffer_store_b128(v, buf, off, 0, 2);
  else __builtin_amdgcn_raw_buffer_store_b128(v, buf, off, 0, 0);
}

// dequantised values of a lane's four columns
struct BigCols {
  double sc[4], bs[4];
  __device__ __forceinline__ BigCols(const float *cst, int nl, float a_s) {
    const v4f s = *(const v4f *)(cst + nl), b = *(const v4f *)(cst + BIG_BN + nl);
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      sc[e] = (double)a_s * (double)s[e];
      bs[e] = (double)b[e];
    }
  }
  __device__ __forceinline__ v4f value(const v4i &a) const {
    v4f v;
#pragma unroll
    for (int e = 0; e < 4; ++e) v[e] = dequant_f32(sc[e], a[e], bs[e]);
    return v;
  }
};

// 32 rows (row blocks ip, ip + 1) of a wavefront's 64 columns to its part of LDS, dequantised, rows of BIG_SR floats; afterwards
// lane l reads columns 4 (l % 16) .. + 3 of the rows l / 16, l / 16 + 4, ...
constexpr int BIG_SR = 64 + 4;
template <int TM>
__device__ __forceinline__ void big_stage_rows(const BigAcc<TM> &acc, float *stage, const float *cst, int wn0, float a_s, int ip) {
  const int lane = threadIdx.x & 63, row = lane & 15, g = lane >> 4;
  int nl = wn0 + g * 4;
  asm volatile("" : "+v"(nl));                                // the constants are read again by the next pass, not kept
#pragma unroll
  for (int j = 0; j < BIG_TN; ++j) {
    const BigCols c(cst, nl + j * 16, a_s);
#pragma unroll
    for (int ii = 0; ii < 2; ++ii) {
      *(v4f *)(stage + (ii * 16 + row) * BIG_SR + j * 16 + g * 4) = c.value(acc[ip + ii][j]);
      QC_SB;                                                  // few dequantised values live at a time
    }
  }
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");      // (LDS operations of a wavefront are in order)
}

template <int TM>
__device__ __forceinline__ void big_gelu(const GemmArgs &p, BigAcc<TM> &acc, unsigned char *smem, const float *cst, int m0, int n0, float a_s) {
  const int tid = threadIdx.x, lane = tid & 63, wn0 = (tid >> 6) * 64, row = lane & 15, g = lane >> 4;
  unsigned char *stage = smem;                         // [16 TM][BIG_SROW] codes
  // Elements whose fast evaluation lands too close to a rounding boundary of Eq. 1 to be trusted are queued here and
  // decided again in float64 (gelu_code_exact): the codes are then those of exact arithmetic on the accumulators.
  int *fix_cnt = (int *)(stage + 16 * TM * BIG_SROW);
  int *fix_ent = fix_cnt + 4;                          // [BIG_FIX_CAP][8]: a lane's four accumulators, row and first column
  if (tid == 0) *fix_cnt = 0;
  __syncthreads();
  const QParam oq = *p.o_qp;
  const GeluQuant gq(oq);
#pragma unroll
  for (int j = 0; j < BIG_TN; ++j) {
    const int nl = wn0 + j * 16 + g * 4;
    v4f sc = *(const v4f *)(cst + nl);
    const v4f bs = *(const v4f *)(cst + BIG_BN + nl);
#pragma unroll
    for (int e = 0; e < 4; ++e) sc[e] *= a_s;
#pragma unroll
    for (int i = 0; i < TM; i += 2) {
      float clear[2][4];
#pragma unroll
      for (int u = 0; u < 2; ++u) *(unsigned *)(stage + ((i + u) * 16 + row) * BIG_SROW + nl) = gq.codes(acc[i + u][j], sc, bs, clear[u]);
      // one comparison and one branch per eight outputs; the branch is short (this code is unrolled 16 times: with a queue entry
      // per output it outgrew the instruction cache)
      if (gq.doubt(clear[0]) || gq.doubt(clear[1])) {
#pragma unroll
        for (int u = 0; u < 2; ++u)
          if (gq.doubt(clear[u])) {
            const int slot = atomicAdd(fix_cnt, 1);
            if (slot < BIG_FIX_CAP) {
              *(v4i *)(fix_ent + slot * 8) = acc[i + u][j];
              fix_ent[slot * 8 + 4] = ((i + u) * 16 + row) * BIG_SROW + nl;
            }
          }
      }
    }
  }
  __syncthreads();
  const int nfix = min(*fix_cnt, BIG_FIX_CAP) * 4;
  for (int f = tid; f < nfix; f += 256) {
    const int pos = fix_ent[(f >> 2) * 8 + 4] + (f & 3), nl = pos % BIG_SROW;
    if (n0 + nl < p.N) stage[pos] = (unsigned char)gelu_code_exact(fix_ent[(f >> 2) * 8 + (f & 3)], a_s, cst[nl], cst[BIG_BN + nl], oq.s, oq.z);
  }
  if (nfix) __syncthreads();
  // coalesced write-out: 16 lanes cover 256 bytes of a row; streaming stores (the tensor is far larger than the L2 and would
  // only evict the operands)
  const int cc = (tid & 15) * 16;
  if (n0 + cc >= p.N) return;                          // N is a multiple of 32
#pragma unroll
  for (int q = 0; q < TM; ++q) {
    const int r = (tid >> 4) + q * 16;
    if (m0 + r < p.M) __builtin_nontemporal_store(*(const v4i *)(stage + r * BIG_SROW + cc), (v4i *)(p.q_out + (size_t)(m0 + r) * p.ldq + n0 + cc));
  }
}

// NT: streaming stores for Q and K.  A kernel of its own: with both ways in one, chosen by an argument (3890 instructions instead of 3044), 16 latents of
// 1024 tokens (28 blocks, 10 steps) took 0.1 - 0.4 % more than with a kernel that knew one way; now 99.6 | 99.7 ms.
template <int TM, bool RAG, bool NT>
__device__ __forceinline__ void big_qkv(const GemmArgs &p, BigAcc<TM> &acc, unsigned char *smem, const float *cst, int m0, int n0, float a_s) {
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), wn0 = wave * 64, row = lane & 15, g = lane >> 4;
  if (n0 + wn0 >= p.N) return;
  constexpr int BM = 16 * TM;
  const int T = p.rows_per_batch, D = p.N / 3;
  const int part = (n0 + wn0) / D, nn0 = n0 + wn0 - part * D;      // D is a multiple of 128: a wavefront's columns lie inside one of Q, K, V
  const int b = m0 / T, tb = m0 - b * T;                      // batch element and token of the tile's first row
  const int rows = RAG ? min(BM, p.M - m0) : BM;      // rows of the tile that exist
  const int bnd = RAG ? min(rows, T - tb) : BM;           // rows of the first batch element (the others: of the next)
  const float inv_hd = 1.0f / (float)p.hd;
  const auto head_of = [&](int nn) { return (int)(((float)nn + 0.5f) * inv_hd); };      // nn / hd, exactly (nn < 2^16)
  float *stage = (float *)smem + wave * (64 * BIG_VR);
  if (part < 2) {
    // a lane's four columns lie in one head (heads start at multiples of hd, a multiple of 4)
    const auto buf = __builtin_amdgcn_make_buffer_rsrc((part == 0 ? p.q32 : p.k32) + (size_t)b * T * D, 0, -1, 0x00027000);
    const int col = row * 4, nn = nn0 + col, h = head_of(nn), e = nn - h * p.hd;
    const int off = ((h * T + tb + g) * p.hd + e) * 4;
#pragma unroll
    for (int ip = 0; ip < TM; ip += 2) {
      big_stage_rows<TM>(acc, stage, cst, wn0, a_s, ip);
#pragma unroll
      for (int q = 0; q < 8; ++q) {
        const v4u v = *(const v4u *)(stage + (q * 4 + g) * BIG_SR + col);
        const int m = ip * 16 + q * 4;
        if (!RAG) {
          big_store16(v, buf, off + m * p.hd * 4, NT);
        } else {
          // row beyond the first batch element: its token 0 lies (heads - 1) * T tokens further than the next row would
          const int o = off + (m + (m + g >= bnd ? (p.heads - 1) * T : 0)) * p.hd * 4;
          if (m + g < rows) big_store16(v, buf, o, NT);
        }
      }
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    }
    return;
  }
  // V^T: 64 tokens of the wavefront's 64 features at a time
  const bool edge = RAG && (bnd < BM || (tb & 31) != 0);
#pragma unroll
  for (int rh = 0; rh < TM / 4; ++rh) {
    int nl = wn0 + g * 4;
    asm volatile("" : "+v"(nl));                              // the constants are read again in the next pass, not kept
#pragma unroll
    for (int j = 0; j < BIG_TN; ++j) {
      const BigCols c(cst, nl + j * 16, a_s);
#pragma unroll
      for (int ii = 0; ii < 4; ++ii) {
        const int ml = ii * 16 + row, pos = edge ? ml : vt_pos(ml);
        const v4f v = c.value(acc[rh * 4 + ii][j]);
#pragma unroll
        for (int e = 0; e < 4; ++e) stage[(j * 16 + g * 4 + e) * BIG_VR + pos] = v[e];
        QC_SB;
      }
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    // lane -> four consecutive token positions ch of the features fc, fc + 4, ...
    const int fc = lane >> 4, ch = (lane & 15) * 4, r0 = rh * 64 + ch;
    if (RAG && edge) {
      // the tile's rows do not start at a group of 32 keys: natural order in LDS, permuted on the way out.  Units of
      // four tokens stay whole when T is a multiple of 4 (then so is every tile's first token)
      if ((T & 3) == 0) {
        const bool second = r0 >= bnd;
        const int t0 = tb + r0 - (second ? T : 0), bb = b + (second ? 1 : 0);
#pragma unroll 4
        for (int q = 0; q < 16; ++q) {
          const int f = fc + q * 4, nn = nn0 + f, h = head_of(nn), e = nn - h * p.hd;
          if (r0 < rows) *(v4f *)(p.vt32 + ((size_t)(bb * p.heads + h) * p.DP + e) * p.Tp + vt_pos(t0)) = *(const v4f *)(stage + f * BIG_VR + ch);
        }
      } else {
        // Any T: the lanes go by the whole units of four tokens of V^T, not of the tile: 16 lanes a feature (64 tokens of one batch element
        // or two hold at most 16 whole units), and the up to three tokens at either end of the run of each batch element
        // follow, a feature a lane.  (Units of the tile, token by token: 5 x 425 tokens 21.8 us, 10 x 425 35.4.)
        const int nt = min(64, rows - rh * 64), na = max(min(bnd - rh * 64, nt), 0);      // tokens of the pass, of the first element among them
        const int ta = tb + rh * 64, tb2 = rh * 64 + na - bnd;  // first token of either run
        const int ha = min(-ta & 3, na), hb = nt > na ? min(-tb2 & 3, nt - na) : 0;       // tokens in front of a run's first whole unit
        const int ua = (na - ha) >> 2, ub = nt > na ? (nt - na - hb) >> 2 : 0;           // whole units
        const int u = lane & 15;
        const bool second = u >= ua;
        const int j0 = second ? na + hb + 4 * (u - ua) : ha + 4 * u;                      // the unit's place in the pass
        float *const dst = p.vt32 + (size_t)(b + (second ? 1 : 0)) * p.heads * p.DP * p.Tp + vt_pos(second ? tb2 + hb + 4 * (u - ua) : ta + ha + 4 * u);
        if (u < ua + ub) {
#pragma unroll 4
          for (int q = 0; q < 16; ++q) {
            const int f = fc + q * 4, nn = nn0 + f, h = head_of(nn), e = nn - h * p.hd;
            const float *const src = stage + f * BIG_VR + j0;
            *(v4f *)(dst + (size_t)(h * p.DP + e) * p.Tp) = (v4f){src[0], src[1], src[2], src[3]};
          }
        }
        const int nn = nn0 + lane, h = head_of(nn), e = nn - h * p.hd;
        const auto ends = [&](int bb, int j, int n, int t) {    // n tokens from t on, at place j of the pass
          float *const d = p.vt32 + ((size_t)(bb * p.heads + h) * p.DP + e) * p.Tp;
          for (int k = 0; k < n; ++k) d[vt_pos(t + k)] = stage[lane * BIG_VR + j + k];
        };
        ends(b, 0, ha, ta);
        ends(b, ha + 4 * ua, na - ha - 4 * ua, ta + ha + 4 * ua);
        if (nt > na) {
          ends(b + 1, na, hb, tb2);
          ends(b + 1, na + hb + 4 * ub, nt - na - hb - 4 * ub, tb2 + hb + 4 * ub);
        }
      }
    } else {
      const auto buf = __builtin_amdgcn_make_buffer_rsrc(p.vt32 + (size_t)b * p.heads * p.DP * p.Tp, 0, -1, 0x00027000);
#pragma unroll
      for (int q = 0; q < 16; ++q) {
        const int f = fc + q * 4, nn = nn0 + f, h = head_of(nn), e = nn - h * p.hd;
        big_store16(*(const v4u *)(stage + f * BIG_VR + ch), buf, ((h * p.DP + e) * p.Tp + tb + rh * 64 + ch) * 4, true);
      }
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  }
}

template <int TM, bool RBF, bool RAG>
__device__ __forceinline__ void big_resid(const GemmArgs &p, BigAcc<TM> &acc, unsigned char *smem, const float *cst, int m0, int n0, float a_s) {
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), wn0 = wave * 64, row = lane & 15, g = lane >> 4;
  const int left = p.N - n0 - wn0;                            // columns from this wavefront's first to the matrix's end (a multiple of 32)
  if (left <= 0) return;
  constexpr int BM = 16 * TM;
  const int b0 = m0 / p.rows_per_batch;
  const int rows = RAG ? min(BM, p.M - m0) : BM;      // rows of the tile that exist
  const int bnd = RAG ? min(rows, (b0 + 1) * p.rows_per_batch - m0) : BM;      // rows of the first batch element
  // element sizes: float32, or (RBF) either tensor may be bfloat16
  const int xb = RBF ? p.x_bf16 : 0, cb = RBF ? p.cache_bf16 : 0;
  const size_t tile0 = (size_t)m0 * p.N + n0 + wn0;           // first element of this wavefront's columns
  const auto xbuf = __builtin_amdgcn_make_buffer_rsrc((char *)p.x + tile0 * (xb ? 2 : 4), 0, -1, 0x00027000);
  const auto cbuf = __builtin_amdgcn_make_buffer_rsrc((char *)p.cache_out + tile0 * (cb ? 2 : 4), 0, -1, 0x00027000);
  float *stage = (float *)smem + wave * (32 * BIG_SR);
  const int col = row * 4, lc = min(col, left - 4);
  const auto pack = [](const v4f &v) {
    return (v2u){(unsigned)bf16_bits(v[0]) | ((unsigned)bf16_bits(v[1]) << 16), (unsigned)bf16_bits(v[2]) | ((unsigned)bf16_bits(v[3]) << 16)};
  };
  // buffer instructions (tile base, row and lane offset in 32 bits) need next to no address arithmetic
  const auto lane_off = [&](int m) { return (RAG ? min(m + g, rows - 1) : g) * p.N + lc; };      // m: first row of a group of four
  const auto row_off = [&](int m) { return RAG ? 0 : m * p.N; };
  // x is requested XD passes ahead of its use
  constexpr int XD = 2;
  v4u xv[XD][8];
  const auto load_x = [&](int ip) {
#pragma unroll
    for (int q = 0; q < 8; ++q) {
      const int m = ip * 16 + q * 4;
      v4u &x = xv[(ip >> 1) % XD][q];
      if (RBF && xb) {
        const auto t = __builtin_amdgcn_raw_buffer_load_b64(xbuf, lane_off(m) * 2, row_off(m) * 2, 0);
        x = (v4u){t[0], t[1], 0u, 0u};                        // converted when it is used
      } else {
        x = __builtin_amdgcn_raw_buffer_load_b128(xbuf, lane_off(m) * 4, row_off(m) * 4, 0);
      }
    }
  };
#pragma unroll
  for (int k = 0; k < XD; ++k) load_x(2 * k);
#pragma unroll
  for (int ip = 0; ip < TM; ip += 2) {
    QC_SB;
    big_stage_rows<TM>(acc, stage, cst, wn0, a_s, ip);
#pragma unroll
    for (int q = 0; q < 8; ++q) {
      const int m = ip * 16 + q * 4;
      const v4f v = *(const v4f *)(stage + (q * 4 + g) * BIG_SR + col);
      const v4f gate = *(const v4f *)(cst + (RAG && m + g >= bnd ? 3 : 2) * BIG_BN + wn0 + col);
      const v4u xr = xv[(ip >> 1) % XD][q];
      const v4f xo = __builtin_bit_cast(v4f, RBF && xb ? (v4u){xr[0] << 16, xr[0] & 0xFFFF0000u, xr[1] << 16, xr[1] & 0xFFFF0000u} : xr);
      v4f xn;
#pragma unroll
      for (int e = 0; e < 4; ++e) xn[e] = fmaf(gate[e], v[e], xo[e]);
      if (col < left && (!RAG || m + g < rows)) {
        // the cached tensor is written once and read a step later: a streaming store keeps it out of the L2's way
        const int lo = lane_off(m), so = row_off(m);
        if (RBF && cb) __builtin_amdgcn_raw_buffer_store_b64(pack(v), cbuf, lo * 2, so * 2, 2);
        else big_store16(__builtin_bit_cast(v4u, v), cbuf, (lo + so) * 4, true);
        if (RBF && xb) __builtin_amdgcn_raw_buffer_store_b64(pack(xn), xbuf, lo * 2, so * 2, 0);
        else big_store16(__builtin_bit_cast(v4u, xn), xbuf, (lo + so) * 4, false);
      }
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    QC_SB;
    if (ip + 2 * XD < TM) load_x(ip + 2 * XD);
  }
}

// float32 rows [M, ldy], any N and M.  NT: streaming stores
template <int TM, bool NT>
__device__ __forceinline__ void big_f32_rows(const GemmArgs &p, BigAcc<TM> &acc, unsigned char *smem, const float *cst, int m0, int n0, float a_s) {
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), wn0 = wave * 64, row = lane & 15, g = lane >> 4;
  const int left = p.N - n0 - wn0, rows = min(16 * TM, p.M - m0);
  if (left <= 0) return;
  float *stage = (float *)smem + wave * (32 * BIG_SR);
  const auto buf = __builtin_amdgcn_make_buffer_rsrc(p.y + (size_t)m0 * p.ldy + n0 + wn0, 0, -1, 0x00027000);
  const int col = row * 4;
#pragma unroll
  for (int ip = 0; ip < TM; ip += 2) {
    QC_SB;
    big_stage_rows<TM>(acc, stage, cst, wn0, a_s, ip);
    if ((p.N & 3) == 0) {                                     // whole groups of four columns
#pragma unroll
      for (int q = 0; q < 8; ++q) {
        const int m = ip * 16 + q * 4;
        const v4u v = *(const v4u *)(stage + (q * 4 + g) * BIG_SR + col);
        if (col < left && m + g < rows) big_store16(v, buf, ((m + g) * p.ldy + col) * 4, NT);
      }
    } else {                                                  // a row of 64 columns at a time
#pragma unroll 8
      for (int r = 0; r < 32; ++r) {
        const int m = ip * 16 + r;
        const unsigned v = *(const unsigned *)(stage + r * BIG_SR + lane);
        if (lane < left && m < rows) __builtin_amdgcn_raw_buffer_store_b32(v, buf, lane * 4, m * p.ldy * 4, NT ? 2 : 0);
      }
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    QC_SB;
  }
}
template <int TM>
__device__ __forceinline__ void big_f32(const GemmArgs &p, BigAcc<TM> &acc, unsigned char *smem, const float *cst, int m0, int n0, float a_s) {
  if (p.stream_out) big_f32_rows<TM, true>(p, acc, smem, cst, m0, n0, a_s);
  else big_f32_rows<TM, false>(p, acc, smem, cst, m0, n0, a_s);
}

// RBF: the residual epilogue's bfloat16 tensors; for Q | K | V streaming stores
template <int TM, int EPI, int TAG, bool W4, bool RBF, bool RAG>
__global__ __launch_bounds__(256, 2) void gemm_i8_big_kernel(GemmArgs p) {
  static_assert(TM == 8 || TM == 4, "");
  constexpr int BM = 16 * TM, BN = BIG_BN, BK = BIG_BK, TN = BIG_TN;
  constexpr int PA = BM / 32;                     // 16-byte activation chunks per thread per slab
  constexpr int AHEAD = TM == 8 ? 1 : 2;          // slabs that the operands are requested ahead of the one multiplied
  constexpr int SLAB = BM * BK;
  extern __shared__ __align__(16) unsigned char smem_base[];
  float *cst = (float *)smem_base;
  unsigned char *smem = smem_base + BIG_CST * 4;

  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  // Tile order: XCD x (= workgroup id mod 8) owns a contiguous range of the order "GM tile rows at a time, column by
  // column", GM chosen by the launcher so that the column tiles of a group of rows are resident on the XCD at the same
  // time, walk K in step and share the group's activation slabs through the XCD's L2.
  const int tiles_m = (p.M + BM - 1) / BM, tiles_n = (p.N + BN - 1) / BN;
  const int per_xcd = (gridDim.x + 7) >> 3;
  const int t = (blockIdx.x & 7) * per_xcd + (blockIdx.x >> 3);
  if (t >= tiles_m * tiles_n) return;
  const int GM = p.group_m;
  const int grp = t / (GM * tiles_n), gm0 = grp * GM, gsz = min(GM, tiles_m - gm0), rr = t - grp * GM * tiles_n;
  const int tn = rr / gsz, tm = gm0 + rr % gsz;
  const int m0 = __builtin_amdgcn_readfirstlane(tm * BM), n0 = __builtin_amdgcn_readfirstlane(tn * BN);   // the divisions above run on the vector ALU
  const int wn0 = wave * (TN * 16);
  float a_s = p.a_scale;
  int a_z = p.a_zp;
  if (p.a_qp) {
    a_s = p.a_qp[0].s;
    a_z = p.a_qp[0].z;
  }

  // Epilogue constants of column n0 + tid and the zero-point sums of this wavefront's columns (lane: 4 (lane / 16) .. + 3 of
  // every block): requested first, so that the prologue's wait for the first slab covers them.  They are loads of inline assembly
  // like all others: for loads that it sees the compiler places waits of its own, which count only those and so either stood in
  // front of the first operand load (fc1, packed weights) or drained the operand loads behind the first barrier (the others).
  // 16384 x 4608 x 1152 1.2 % faster, sampling runs 0.1 - 0.4 %.
  // Columns past N re-read the last one (never stored).
  const auto load_const = [](auto &r, const void *base, unsigned off) {
    if constexpr (sizeof(r) == 16) asm volatile("global_load_dwordx4 %0, %1, %2" : "=v"(r) : "v"(off), "s"(base) : "memory");
    else asm volatile("global_load_dword %0, %1, %2" : "=v"(r) : "v"(off), "s"(base) : "memory");
  };
  float c_sc, c_bs, c_g0 = 0.0f, c_g1 = 0.0f;
  const unsigned ccol = (unsigned)min(n0 + tid, p.N - 1) * 4u;
  load_const(c_sc, p.w_scale, ccol);
  load_const(c_bs, p.bias ? p.bias : p.w_scale, ccol);        // without a bias it is zeroed below
  if constexpr (EPI == EPI_RESID) {
    const int b = m0 / p.rows_per_batch, b1 = RAG && (b + 1) * p.rows_per_batch < min(m0 + BM, p.M) ? b + 1 : b;
    load_const(c_g0, p.gate + (size_t)b * p.ld_gate, ccol);
    if constexpr (RAG) load_const(c_g1, p.gate + (size_t)b1 * p.ld_gate, ccol);
  }
  v4i ws[TN];
  int w1[EPI == EPI_F32 ? TN * 4 : 1];
#pragma unroll
  for (int j = 0; j < TN; ++j) {
    const int n = n0 + wn0 + j * 16 + (lane >> 4) * 4;
    if constexpr (EPI == EPI_F32) {
#pragma unroll
      for (int e = 0; e < 4; ++e) load_const(w1[j * 4 + e], p.wsum, (unsigned)min(n + e, p.N - 1) * 4u);
    } else {
      load_const(ws[j], p.wsum, (unsigned)min(n, p.N - 4) * 4u);
    }
  }

  // activations: load i of thread tid covers row 32 i + tid / 8, 16-byte chunk tid % 8 of a slab and is written to
  // LDS at the swizzled position of that chunk.  Rows beyond M re-read row M - 1.
  unsigned aoff[PA];
  const int arow = tid >> 3, ac = tid & 7;
#pragma unroll
  for (int i = 0; i < PA; ++i) aoff[i] = (unsigned)(min(m0 + 32 * i + arow, p.M - 1) - m0) * (unsigned)p.lda + ac * 16;
  const unsigned lpos = arow * BK + ((ac ^ ((arow >> 1) & 7)) * 16);          // + 32 i rows: the same swizzle
  const int8_t *abase = p.A + (size_t)m0 * p.lda;
  // K: a multiple of 128, or (EPI_F32) of 16: the stored weights are zero from K to the end of the last slab, and chunks of it
  // beyond K re-read the row's last one
  const int nk = EPI == EPI_F32 ? (p.K + BK - 1) / BK : p.K / BK, ng = nk * (BK / 64);
  const unsigned kback = EPI == EPI_F32 ? (unsigned)max((nk - 1) * BK + ac * 16 + 16 - p.K, 0) : 0u;
  v4i ra[AHEAD][PA];                              // slab kt in set kt % AHEAD
  auto load_a = [&](v4i &r, int kt, int i) {      // slabs past the end re-read the last one (never used)
    // (kback of the last slab may exceed aoff of row 0: the sum of base and offset is what counts, so the base gives it up front)
    if constexpr (EPI == EPI_F32) {
      const int8_t *src = abase + min(kt, nk - 1) * BK - BK;
      asm volatile("global_load_dwordx4 %0, %1, %2" : "=v"(r) : "v"(aoff[i] + (BK - (kt >= nk - 1 ? kback : 0u))), "s"(src) : "memory");
    } else {
      asm volatile("global_load_dwordx4 %0, %1, %2" : "=v"(r) : "v"(aoff[i]), "s"(abase + min(kt, nk - 1) * BK) : "memory");
    }
  };
  auto write_a = [&](const v4i &r, int buf, int i) { *(v4i *)(smem + buf * SLAB + lpos + i * 32 * BK) = r; };

  if (EPI != EPI_GELU_Q && !W4 && n0 + wn0 >= p.N) {
    // A wavefront whose columns all lie beyond N (half of a last tile when N = 1152) only moves its share of the activations: at
    // the power limit the products it leaves out are time for the others (measured with M = 8192 and more: 0.3 - 0.7 % of a
    // whole run; with packed weights, which fewer bytes and more vector work bound, it lost 1 %).  It has registers and loads of its
    // own from the start: where it shared them with the loop below, the compiler copied registers that loads were on their way to.
    v4i sa[2][PA];                                // slab kt in set kt % 2
#pragma unroll
    for (int u = 0; u < 2; ++u)
#pragma unroll
      for (int i = 0; i < PA; ++i) load_a(sa[u][i], u, i);
    auto move = [&](int kt, int u) {              // slab kt (set u = kt % 2) to LDS, slab kt + 2 requested
      if constexpr (PA == 4) QC_WAIT_VM_FOR4(4, sa[u][0], sa[u][1], sa[u][2], sa[u][3]);
      else QC_WAIT_VM_FOR2(2, sa[u][0], sa[u][1]);
#pragma unroll
      for (int i = 0; i < PA; ++i) write_a(sa[u][i], u, i);
      QC_SB;
#pragma unroll
      for (int i = 0; i < PA; ++i) load_a(sa[u][i], kt + 2, i);
      QC_LDS_DONE_BARRIER;
    };
    // the barriers of the other wavefronts: one behind slab 0, one per slab of the loop (behind slab kt + 1), one at its end
    int kt = 0;
    for (; kt + 2 <= nk + 1; kt += 2) {
      move(kt, 0);
      move(kt + 1, 1);
    }
    if (kt < nk + 1) move(kt, 0);
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
#pragma unroll
    for (int u = 0; u < 2; ++u)
#pragma unroll
      for (int i = 0; i < PA; ++i) asm volatile("" : "+v"(sa[u][i]));
    __syncthreads();
    return;
  }

  // weight fragments of this wavefront: column block j (16 columns) is half j % 2 of the stored n-block (n0 + wn0) / 32 + j / 2
  // (blocks past N re-read the last one), group g (64 k) the two stored fragments 2 g and 2 g + 1 of it: lane l takes chunk l / 16 of
  // the 64 k, row l % 16 of the half
  constexpr int FRAG = W4 ? 512 : 1024;           // bytes per stored fragment
  typedef typename std::conditional<W4, v2i, v4i>::type wfrag_t;
  const int nblocks = (p.N + 31) / 32;
  const int8_t *sb[TN / 2];
#pragma unroll
  for (int j = 0; j < TN / 2; ++j) sb[j] = (const int8_t *)p.Wt + (size_t)min((n0 + wn0) / 32 + j, nblocks - 1) * (2 * ng) * FRAG;
  const unsigned woff = (lane >> 5) * FRAG + ((lane >> 4) & 1) * (FRAG / 2) + (lane & 15) * (FRAG / 64);
  wfrag_t bq[2 * AHEAD][TN];                      // group g (64 k, of all of K) in set g % (2 AHEAD)
  auto load_w = [&](int g, int kg, int j) {       // groups past the end re-read the last one (never used)
    const int8_t *src = sb[j >> 1] + (size_t)min(kg, ng - 1) * (2 * FRAG);
    if constexpr (W4) {
      if (j & 1) asm volatile("global_load_dwordx2 %0, %1, %2 offset:128" : "=v"(bq[g][j]) : "v"(woff), "s"(src) : "memory");
      else asm volatile("global_load_dwordx2 %0, %1, %2" : "=v"(bq[g][j]) : "v"(woff), "s"(src) : "memory");
    } else {
      if (j & 1) asm volatile("global_load_dwordx4 %0, %1, %2 offset:256" : "=v"(bq[g][j]) : "v"(woff), "s"(src) : "memory");
      else asm volatile("global_load_dwordx4 %0, %1, %2" : "=v"(bq[g][j]) : "v"(woff), "s"(src) : "memory");
    }
  };

  unsigned fbase[2];                              // LDS position of this lane's chunk of group g in row block 0
#pragma unroll
  for (int g = 0; g < 2; ++g) fbase[g] = (lane & 15) * BK + (((g * 4 + (lane >> 4)) ^ ((lane >> 1) & 7)) * 16);
  v4i fa[2][4];
  auto read_frag = [&](int f, int buf, int g, int half, int i) {
    fa[f][i] = *(const v4i *)(smem + buf * SLAB + fbase[g] + (half * 4 + i) * 16 * BK);
  };

  // prologue: slab 0 -> LDS (through registers of the fragments), slabs 1 .. AHEAD -> registers, the weights of slabs 0 .. AHEAD - 1
#pragma unroll
  for (int i = 0; i < PA; ++i) load_a(fa[1][i], 0, i);
#pragma unroll
  for (int u = 0; u < AHEAD; ++u) {
#pragma unroll
    for (int i = 0; i < PA; ++i) load_a(ra[(u + 1) % AHEAD][i], u + 1, i);
#pragma unroll
    for (int g = 0; g < 2; ++g)
#pragma unroll
      for (int j = 0; j < TN; ++j) load_w(2 * u + g, 2 * u + g, j);
  }
  QC_SB;
  if constexpr (TM == 8) QC_WAIT_VM_FOR4(12, fa[1][0], fa[1][1], fa[1][2], fa[1][3]);
  else QC_WAIT_VM_FOR2(20, fa[1][0], fa[1][1]);
  asm volatile("" : "+v"(c_sc), "+v"(c_bs));                  // (valid with the same wait)
  if constexpr (EPI == EPI_RESID) asm volatile("" : "+v"(c_g0));
  if constexpr (EPI == EPI_RESID && RAG) asm volatile("" : "+v"(c_g1));
  if constexpr (EPI == EPI_F32) {
#pragma unroll
    for (int i = 0; i < TN * 4; ++i) {
      asm volatile("" : "+v"(w1[i]));
      ws[i >> 2][i & 3] = w1[i];
    }
  } else {
    asm volatile("" : "+v"(ws[0]), "+v"(ws[1]), "+v"(ws[2]), "+v"(ws[3]));
  }
  // the accumulators start at minus the zero-point term a_z * wsum[n] of their column, so the epilogue finds acc - a_z * wsum[n] ready
  BigAcc<TM> acc;
#pragma unroll
  for (int j = 0; j < TN; ++j) {
    v4i c0;
#pragma unroll
    for (int e = 0; e < 4; ++e) c0[e] = -(a_z * ws[j][e]);
#pragma unroll
    for (int i = 0; i < TM; ++i) acc[i][j] = c0;
  }
#pragma unroll
  for (int i = 0; i < PA; ++i) write_a(fa[1][i], 0, i);
  cst[tid] = c_sc;
  cst[BN + tid] = p.bias ? c_bs : 0.0f;
  if (EPI == EPI_RESID) {
    cst[2 * BN + tid] = c_g0;
    if (RAG) cst[3 * BN + tid] = c_g1;
  }
  QC_LDS_DONE_BARRIER;
#pragma unroll
  for (int i = 0; i < 4; ++i) read_frag(0, 0, 0, 0, i);
  QC_SB;

  // Slab kt = two groups of 64 k, each in two steps of 64 rows (four row blocks, 16 products): step s = 2 g + half.  On entry:
  // slab kt is in LDS buffer kt % 2 and published; fa[0] holds (or awaits) the fragments of step 0; the weights of both groups and
  // activation slab kt + 1 are requested.
  //   step 0: activation slab kt + 1 registers -> LDS, slab kt + 2 requested (4 loads)
  //   steps 1 and 3: the weights of the group are free column block by column block, the next slab's are requested (4 loads each)
  //   every step reads the fragments of the next one; the barrier before step 3 publishes slab kt + 1, whose buffer was last
  //   read in step 2 of slab kt - 1, before that slab's barrier.
  // Loads issued after the one a wait is for:
  //   step 0, for the weights of group 0 (step 1 of slab kt - 1) and, older, the activations: the weights of group 1    = 4
  //   step 2, for the weights of group 1 (step 3 of slab kt - 1): the activations and weights of steps 0 and 1          = 8
  if constexpr (TM == 8) {
    v4i wf[TN];
    auto step = [&](int kt, int s, int buf) {
      const int g = s >> 1, half = s & 1, f = s & 1;
      if constexpr (W4) {
        if (half == 0) {
#pragma unroll
          for (int j = 0; j < TN; ++j) wf[j] = unpack_w4(bq[g][j]);
        }
      }
#pragma unroll
      for (int j = 0; j < TN; ++j) {
        v4i w;
        if constexpr (W4) w = wf[j];
        else w = bq[g][j];
#pragma unroll
        for (int ii = 0; ii < 4; ++ii) {
          const int i = (j & 1) ? 3 - ii : ii, k = j * 4 + ii;
          QC_SB;
          acc[half * 4 + i][j] = __builtin_amdgcn_mfma_i32_16x16x64_i8(w, fa[f][i], acc[half * 4 + i][j], 0, 0, 0);
          if (k < 4) read_frag(f ^ 1, s == 3 ? buf ^ 1 : buf, ((s + 1) >> 1) & 1, (s + 1) & 1, k);
          if (s == 0 && k >= 4 && k < 8) write_a(ra[0][k - 4], buf ^ 1, k - 4);
          if (s == 0 && k >= 12) load_a(ra[0][k - 12], kt + 2, k - 12);
        }
        if (half == 1) load_w(g, 2 * kt + g + 2, j);
      }
      QC_SB;
    };
    auto slab = [&](int kt, int buf) {
      QC_WAIT_VM_FOR4(4, ra[0][0], ra[0][1], ra[0][2], ra[0][3]);
      QC_WAIT_VM_FOR4(4, bq[0][0], bq[0][1], bq[0][2], bq[0][3]);
      step(kt, 0, buf);
      step(kt, 1, buf);
      QC_WAIT_VM_FOR4(8, bq[1][0], bq[1][1], bq[1][2], bq[1][3]);
      step(kt, 2, buf);
      QC_LDS_DONE_BARRIER;
      step(kt, 3, buf);
    };
    int kt = 0;
    for (; kt + 2 <= nk; kt += 2) {
      slab(kt, 0);
      slab(kt + 1, 1);
    }
    if (kt < nk) slab(kt, 0);
    // the loads that ran past the end (clamped addresses) must have landed before registers are reused (the waits name their
    // registers: a load whose result nobody uses would share its register with something live), and every wavefront must be past
    // its last fragment read before the epilogue reuses LDS
    QC_WAIT_VM_FOR4(0, ra[0][0], ra[0][1], ra[0][2], ra[0][3]);
#pragma unroll
    for (int g = 0; g < 2; ++g) QC_WAIT_VM_FOR4(0, bq[g][0], bq[g][1], bq[g][2], bq[g][3]);
  } else {
    // 64 rows: slab kt = two groups of 64 k, one step each (16 products).  A slab takes half as long, so its operands are requested
    // two slabs ahead: on entry slab kt is in LDS buffer kt % 2 and published; fa[0] holds (or awaits) the fragments of its group 0;
    // the weights of slabs kt, kt + 1 and the activations of slabs kt + 1, kt + 2 are requested.
    //   step 0: activation slab kt + 1 registers -> LDS, slab kt + 3 requested into the same registers (2 loads, in front of the
    //           weights of the last column block)
    //   both steps: the group's weights are free column block by column block, those of slab kt + 2 are requested (4 loads)
    //   the barrier before step 1 publishes slab kt + 1, whose buffer was last read in step 0 of slab kt - 1
    // Loads issued after the one a wait is for:
    //   step 0, for the weights of group 0 (step 0 of slab kt - 2) and, older, the activations: step 1 of slab kt - 2 (4), slab kt - 1 (10) = 14
    //   step 1, for the weights of group 1 (step 1 of slab kt - 2): slab kt - 1 (10), step 0 of this slab (6)                            = 16
    auto step = [&](int kt, int g, int u) {       // u = kt % 2
      constexpr bool w4 = W4;
      v4i wf[TN];
      if constexpr (w4) {
#pragma unroll
        for (int j = 0; j < TN; ++j) wf[j] = unpack_w4(bq[2 * u + g][j]);
      }
#pragma unroll
      for (int j = 0; j < TN; ++j) {
        v4i w;
        if constexpr (w4) w = wf[j];
        else w = bq[2 * u + g][j];
#pragma unroll
        for (int ii = 0; ii < 4; ++ii) {
          const int i = (j & 1) ? 3 - ii : ii, k = j * 4 + ii;
          QC_SB;
          acc[i][j] = __builtin_amdgcn_mfma_i32_16x16x64_i8(w, fa[g][i], acc[i][j], 0, 0, 0);
          if (k < 4) read_frag(g ^ 1, g == 1 ? u ^ 1 : u, g ^ 1, 0, k);
          if (g == 0 && k >= 4 && k < 6) write_a(ra[u ^ 1][k - 4], u ^ 1, k - 4);
          if (g == 0 && k >= 12 && k < 14) load_a(ra[u ^ 1][k - 12], kt + 3, k - 12);
        }
        load_w(2 * u + g, 2 * (kt + 2) + g, j);
      }
      QC_SB;
    };
    auto slab = [&](int kt, int u) {
      QC_WAIT_VM_FOR2(14, ra[u ^ 1][0], ra[u ^ 1][1]);
      QC_WAIT_VM_FOR4(14, bq[2 * u][0], bq[2 * u][1], bq[2 * u][2], bq[2 * u][3]);
      step(kt, 0, u);
      QC_LDS_DONE_BARRIER;
      QC_WAIT_VM_FOR4(16, bq[2 * u + 1][0], bq[2 * u + 1][1], bq[2 * u + 1][2], bq[2 * u + 1][3]);
      step(kt, 1, u);
    };
    auto drain = [&]() {
#pragma unroll
      for (int u = 0; u < AHEAD; ++u) {
        QC_WAIT_VM_FOR2(0, ra[u][0], ra[u][1]);
        QC_WAIT_VM_FOR4(0, bq[2 * u][0], bq[2 * u][1], bq[2 * u][2], bq[2 * u][3]);
        QC_WAIT_VM_FOR4(0, bq[2 * u + 1][0], bq[2 * u + 1][1], bq[2 * u + 1][2], bq[2 * u + 1][3]);
      }
    };
    int kt = 0;
    for (; kt + 2 <= nk; kt += 2) {
      slab(kt, 0);
      slab(kt + 1, 1);
    }
    if (kt < nk) slab(kt, 0);
    drain();
  }
  QC_SB;
  __syncthreads();
  if constexpr (EPI == EPI_GELU_Q) big_gelu<TM>(p, acc, smem, cst, m0, n0, a_s);
  else if constexpr (EPI == EPI_QKV) big_qkv<TM, RAG, RBF>(p, acc, smem, cst, m0, n0, a_s);
  else if constexpr (EPI == EPI_F32) big_f32<TM>(p, acc, smem, cst, m0, n0, a_s);
  else big_resid<TM, RBF, RAG>(p, acc, smem, cst, m0, n0, a_s);
}

template <int TM, int EPI, int TAG, bool W4, bool RBF, bool RAG = false>
static hipError_t launch_big_as(const GemmArgs &a, hipStream_t st) {
  constexpr int BM = 16 * TM;
  // launches whose tiles are not all whole and inside one batch element take the variant that handles the others
  if constexpr (!RAG && (EPI == EPI_RESID || EPI == EPI_QKV)) {
    if (a.M % BM || a.rows_per_batch % BM) return launch_big_as<TM, EPI, TAG, W4, RBF, true>(a, st);
  }
  constexpr int smem_epi = EPI == EPI_GELU_Q ? big_smem_gelu<TM> : (EPI == EPI_QKV ? BIG_SMEM_QKV : BIG_SMEM_RESID);
  constexpr int smem = BIG_CST * 4 + (smem_epi > big_smem_loop<TM> ? smem_epi : big_smem_loop<TM>);
  static_assert(2 * smem <= 160 * 1024, "two workgroups per compute unit");
  auto kern = gemm_i8_big_kernel<TM, EPI, TAG, W4, RBF, RAG>;
  static std::atomic<unsigned long long> lds{0};
  if (const hipError_t e = allow_lds((const void *)kern, smem, lds)) return e;
  const int tiles_n = (a.N + BIG_BN - 1) / BIG_BN, tiles = ((a.M + BM - 1) / BM) * tiles_n;
  GemmArgs b = a;
  // Tile rows per group.  Few columns: every column tile of a group resident on its XCD at once (64 workgroup slots), at most 4 rows of
  // 128 (5 column tiles, M = 16384: proj 48.3 us, with 8 rows 49.3, 16 51.7; fc2 95.4, 96.8, 98.0).  From 12 column tiles of 128 rows on, 8
  // rows where K is long: the 64 resident tiles are then 8 x 8, which pulls the least into the L2 (3 rows of fc1 stream all its weights, more
  // than the L2 holds, once for every 384 rows).  Fewer bytes of K a tile do not pay for the wider order: 16384 rows of qc_w8a8_linear, us, 4 | 8 rows:
  // 4608 columns, K = 512 92.2 | 95.9, 640 99.2 | 102.2, 768 106.7 | 108.2, 896 115.1 | 113.1, 1008 125.8 | 123.9, 1152 130.5 | 126.8, 1408 148.7 | 143.0;
  // 3456, K = 768 85.6 | 87.1, 896 91.6 | 92.0, 1008 102.1 | 101.8, 1152 105.1 | 104.4; packed weights, 4608, K = 768 105.4 | 106.1, 1152 136.8 |
  // 136.0, 2304 220.0 | 218.5.  In a block fc1 of width 768, 32768 rows, 99.6 | 102.3.
  // fc1 of networks of width 1152, one block by itself, us: 65536 rows 367 | 365, 32768 185.8 | 185.4, 16384 96.6 | 99.3, 8192 55.9 | 54.6; packed weights, 16384
  // rows 100.5 | 104.1, 4096 34.7 | 33.0.  What decides is the run, whose halves share the caches: 128 guided latents of 256 tokens (9 steps, 28
  // blocks, QKV too) 88.9 ms with 4 rows, 88.7 with 8; 12 blocks, 4 steps: 32 latents 6.85 | 6.81, 64 12.38 | 12.42, 96 18.28 | 18.18, 128 24.29 | 24.21.
  // QKV takes 4 there, which 8 do not beat in a run and are slower than where Q and K stream.  A block's launch, width 1152, us, 4 rows | 8, without
  // streaming: 8192 rows 43.8 | 43.2, 16384 79.4 | 81.4, 24576 142 | 145, 28672 166 | 163, 32768 184 | 186 (166 | 164 on a chip that holds its clocks), 65536
  // 339 | 329; streaming: 16384 90 | 98, 32768 181 | 190 (166 | 174), 65536 equal.  Runs of 12 blocks, 4 steps, fc1 with 8: 24 latents 5.71 | 5.71 ms, 32 6.94 | 6.96,
  // 64 12.73 | 12.82, 96 18.63 | 18.60, 128 24.72 | 24.79, 256 49.4 | 49.4, 32 of 1024 tokens 35.07 | 35.00, 76 of 425 28.64 | 28.59; wider networks, 3 (2) | 4 | 8: width 1536,
  // 6 blocks, 32 latents 5.32 | 5.25 | 5.25, 64 10.39 | 10.34 | 10.40, 128 20.44 | 20.39 | 20.37; 2048, 4 blocks, 32 5.79 | 5.71 | 5.73, 64 11.48 | 11.37 | 11.36, 128 22.20 |
  // 21.96 | 22.21.
  // Not where the last group is a good part of the rows (M = 4250 25.0 | 25.6), nor for float32 results whose rows are no whole lines, whose pieces
  // then meet later (16300 x 4600 x 1008 127 | 131, 32000 x 3300 x 400 151 | 159), or of fewer than some 1500 tiles (K = 1152, 4608 columns, 8192 rows
  // 80.9 | 81.3, 13000 106.9 | 107.9, 14336 117.7 | 117.2, 24576 186.8 | 182.9; 3456, 12288 90.2 | 91.2, 14336 94.7 | 94.5, 17000 113.7 | 111.8; 4096 columns
  // lose up to 1 % below 3000 tiles: 16384 118.0 | 119.0, 24576 164.7 | 163.8).  64-row tiles gain and lose 2 % by shape and stay.
  const int tiles_m = tiles / tiles_n;
  const bool wide = TM == 8 && tiles_n >= 12 && a.K >= 960 && (tiles_m % 8 == 0 || tiles_m >= 64) &&
                    (EPI != EPI_F32 || ((a.ldy & 31) == 0 && tiles >= 1500));
  b.group_m = wide ? (EPI == EPI_QKV ? 4 : 8) : std::min(std::max(64 / tiles_n, 1), 32 / TM);
  // Float32 rows of whole lines stream.  Others, cut into pieces, where the result, the codes and the float32 values that these were made from outgrow the
  // memory-side cache, the sooner the longer a tile multiplies and the pieces' writes hide behind it (one float a lane, N no multiple of 4, hides
  // them later).  16384 - 49152 rows, us with the quantiser, streaming | not (MB of all three, x K / 1000): N = 1160, 16384 rows, K = 1152 64.3 | 59.7 (170,
  // 196), 24576 81.6 | 76.3 (255, 294), 32768 99.8 | 104.3 (341, 393), K = 768 86.3 | 79.4 (278, 213), 1408 107.6 | 117.3 (383, 539); N = 2308, 16384, K = 1152
  // 92.9 | 84.5 (245, 282), 20480 111.4 | 110.3 (307, 354), 24576 127.4 | 131.0 (369, 425), 32768 158 | 172 (491, 566), 576 135.8 | 122.5 (397, 229), 12288, K =
  // 2304 114.1 | 109.2 (255, 588); N = 3460, 16384, 1152 126.0 | 127.4 (321, 370; other inputs each pass), 1408 129.7 | 134.3 (342, 482), 32768 211 | 241 (643, 741); N = 4100, 16384 133.4 |
  // 141.0 (363, 418), 24576, K = 704 168.3 | 169.7 (490, 376; the same), 768 164.0 | 166.3 (497, 382); N = 4600, 16384, 896 133.9 | 131.7 (375, 336), 1152 138.5 | 149.1 (396, 456);
  // N = 2309, 16384, 1152 104.8 | 93.3 (245, 282), 32768 179.5 | 179.4 (491, 566), 49152 256 | 288 (737, 849); N = 3333, 16384, 1152 134 | 127 (313, 360), 2304 179 |
  // 187 (407, 937), 32768, 768 204 | 200 (563, 432), 1152 237 | 247 (626, 721).  Rows of whole lines, 16384: 4608 115.5 | 121, 1152 41.4 | 42.9, 2304 68 | 68.5.
  if constexpr (EPI == EPI_F32) {
    const double all = (double)a.M * (4.0 * a.N + 5.0 * a.K);
    const int Kp = (a.K + BIG_BK - 1) / BIG_BK * BIG_BK;      // what a tile multiplies
    b.stream_out = (a.ldy & 31) == 0 || (all > 3.0e8 && all * Kp > ((a.N & 3) == 0 ? 3.65e11 : 5.6e11));
  }
  hipLaunchKernelGGL(kern, dim3(((tiles + 7) / 8) * 8), dim3(256), smem, st, b);
  return hipGetLastError();
}

// Rows of a tile for this launch; 0: the launch has too few tiles, the other kernels take it.  Measured alone on the chip
// (us; other kernels | 64 rows | 128 rows), by the number of 64-row tiles, at K = 1152 unless said otherwise:
//    48 - 80 tiles    11.6 | 12.9 | 17.0 (N = 1152, M = 1024), 10.4 | 11.2 | 15.1 (N = 3456, M = 256), K = 4608: 20.4 | 24.2 | 38.8
//   112 - 144 tiles   13.2 | 11.6 | 15.2 (N = 3456, M = 512), 14.2 | 13.3 | 17.3 (N = 1152, M = 1536), K = 4608: 27.1 | 24.0 | 39.7
//   160 - 252 tiles   18.4 | 12.6 | 15.5 (N = 3456, M = 1024), 24.6 | 14.5 | 18.4 (N = 4608, M = 850), K = 4608: 30.8 | 25.1 | 39.8
//   288 tiles         21.1 | 17.9 | 18.8 (N = 4608, M = 1024)
//   320 - 384 tiles   16.9 | 16.4 (64 | 128 rows; N = 3456, M = 1536), 21.8 | 20.0 (N = 1152, M = 4096), K = 4608: 42.2 | 43.0
//   from 576 tiles    the 128-row tile reads each weight for twice the rows and is 0 - 25 % faster
// One 64-row tile on each of the 256 compute units is what such a launch can use; two on a unit take as long as one of
// 128 rows.  The 4-bit codes lie the same way (288 tiles 22.7 | 20.1 | 20.7, 80 tiles 12.9 | 14.7 | 20.4).
// Refresh and cached steps of an eight-block network of width 1152, before and after: 6 latents of 256 tokens 2804 -> 2607 us,
// 8: 3116 -> 3061, 16: 4749 -> 4620, 5 of 425 tokens 4453 -> 3854; 1 and 24 latents unchanged.  (From 60 tiles on: 6 latents 2910.)
static int big_rows(const GemmArgs &a) {
  const long long tiles_n = (a.N + BIG_BN - 1) / BIG_BN;
  const long long t64 = (a.M + 63) / 64 * tiles_n, t128 = (a.M + 127) / 128 * tiles_n;
  if (t64 >= 100 && t64 < 300) return 64;
  return t128 >= 150 ? 128 : 0;
}

// The large-M kernel takes over when the weights exist in fragment order, the shape fits its loop (K a multiple of
// 128, N of 32, 16-byte aligned rows), a tile holds rows of at most two batch elements (its epilogues are compiled
// without the general paths) and the launch has enough tiles for it to pay.
bool gemm_big_pays(const GemmArgs &a, int epi, int nz) {
  if (epi == EPI_F32 || !a.Wt || nz != 1 || a.sel_D || a.acc_out) return false;
  if (a.K % 128 || a.N % 32 || a.lda % 16) return false;
  const int rows = big_rows(a);
  if (epi == EPI_RESID && a.rows_per_batch < rows) return false;
  if (epi == EPI_QKV && (a.y || a.rows_per_batch < rows || (a.N / 3) % 128 || a.hd % 4 || a.Tp % 8)) return false;
  return rows > 0;
}

template <int EPI, int TAG, bool RBF>
static hipError_t launch_big_w(const GemmArgs &a, hipStream_t st) {
  if (big_rows(a) == 64) return a.w4 ? launch_big_as<4, EPI, TAG, true, RBF>(a, st) : launch_big_as<4, EPI, TAG, false, RBF>(a, st);
  return a.w4 ? launch_big_as<8, EPI, TAG, true, RBF>(a, st) : launch_big_as<8, EPI, TAG, false, RBF>(a, st);
}

// Streaming stores for Q and K, by the results of all launches that run together.  Heads of whole 128-byte lines (a wavefront's 64 columns cut their
// rows into whole lines): above half of the memory-side cache, from which attention would read what fits.  Other heads (72 features: pieces of lines,
// which streaming stores send to memory one by one and others let meet in the L2): not before the results are 1.5 times that cache,
// and 1.75 times where halves run beside each other, which at less gain nothing by it or lose a little.
// Whole runs, 12 blocks, 4 steps, 256 tokens, two halves, ms, streaming | not (MB of all results): heads of 64, width 768: 32 latents (75) 4.48 | 4.47,
// 64 (151) 7.58 | 7.75, 96 10.86 | 11.00, 256 (604) 27.7 | 28.1, width 384: 64 (75) 3.76 | 3.73, 128 (151) 6.45 | 6.50, 512 (604) 24.0 | 24.7, width
// 1152: 64 (226) 12.72 | 12.76, 128 24.2 | 24.4; heads of 72, width 1152: 64 (226) 12.93 | 12.71, 96 (340) 18.79 | 18.65, 112 (396) 21.92 | 21.96,
// 128 (453) 24.83 | 24.87, 136 (481) 26.75 | 26.92, 192 (679) 37.40 | 37.47, 76 of 425 tokens (447) 28.56 | 28.65, 30 and 32 of 1024 (425, 453) 32.82 | 32.76, 34.80 | 34.67;
// 28 blocks, 6 steps, guided: 56 (396) 53.53 | 53.47, 60 (425) 57.54 | 57.59, 64 (453, 9 steps) 90.79 | 90.74, 72 (510) 68.69 | 68.91; heads of 80, width 640, 192 (377) 17.68 |
// 17.76, 256 (503) 23.22 | 23.44.
// Ragged tiles, 425 tokens: 72, 10 and 16 latents 5.07 | 5.05, 7.31 | 7.27; 64, width 768, 16 latents 4.62 | 4.58, 76 equal.
// One block alone, QKV and attention, us: 72, 16384 rows 90 + 114 | 79 + 114, 24576 145 + 189 | 142 + 191, 28672 166 + 216 | 166 + 216, 32768 181 + 241 | 184 + 242
// (on a chip that holds its clocks 166 + 229 | 166 + 230), 40960 226 + 291 | 224 + 292, 65536 338 + 440 | 339 + 449.
static bool qkv_streams(const GemmArgs &a) {
  const size_t limit = (a.hd & 31) == 0 ? 128 : a.beside > 1 ? 448 : 384;          // MiB
  return big_rows(a) == 128 && (size_t)std::max(a.beside, 1) * a.M * a.N * sizeof(float) > limit << 20;      // (64-row tiles: at most 300 of them, 20 MB)
}

// `site` only names the instantiation (so that profiles tell the linears apart); the residual epilogue is compiled twice,
// for float32 stream and cache and for the bfloat16 variants of either
hipError_t launch_gemm_big(const GemmArgs &a, int epi, hipStream_t st, int site) {
  if (epi == EPI_GELU_Q) return launch_big_w<EPI_GELU_Q, QC_SITE_FC1, false>(a, st);
  if (epi == EPI_QKV && qkv_streams(a))
    return a.w4 ? launch_big_as<8, EPI_QKV, QC_SITE_QKV, true, true>(a, st) : launch_big_as<8, EPI_QKV, QC_SITE_QKV, false, true>(a, st);
  if (epi == EPI_QKV) return launch_big_w<EPI_QKV, QC_SITE_QKV, false>(a, st);
  if (a.x_bf16 || a.cache_bf16)
    return site == QC_SITE_FC2 ? launch_big_w<EPI_RESID, QC_SITE_FC2, true>(a, st) : launch_big_w<EPI_RESID, QC_SITE_PROJ, true>(a, st);
  return site == QC_SITE_FC2 ? launch_big_w<EPI_RESID, QC_SITE_FC2, false>(a, st) : launch_big_w<EPI_RESID, QC_SITE_PROJ, false>(a, st);
}

// Row-major weights (qc_w8a8_linear).  The kernel wants them in fragment order and the library owns no memory for a second copy,
// so the copy (columns padded with zeros to 32, k to 128) goes where the last rows of the result will lie; those rows
// follow in a launch of their own from the row-major weights, which overwrites it.  (The kernel reading row-major weights
// itself was measured: adjacent lanes of a fragment are different rows, the address unit merges only adjacent lanes, and
// 32768 x 1152 x 4608 took 207 us instead of 151, more than the tile kernel at 8192 rows.)
static int big_copy_rows(const GemmArgs &a) {     // rows of the result that hold the copy, plus those that make the rest whole tiles
  const size_t bytes = (size_t)((a.N + 31) / 32 * 32) * ((a.K + BIG_BK - 1) / BIG_BK * BIG_BK) / (a.w4 ? 2 : 1) + 16;      // + alignment
  const size_t row = (size_t)a.N * sizeof(float), n = (bytes + row - 1) / row;
  return (size_t)a.M > n ? (int)(n + (a.M - n) % 128) : a.M;
}

bool gemm_big_rows_pays(const GemmArgs &a) {
  if (a.acc_out) return false;
  const double work = (double)a.M * a.N * a.K;
  const double padded = (double)((a.M + 127) / 128 * 128) * ((a.N + BIG_BN - 1) / BIG_BN * BIG_BN) * ((a.K + BIG_BK - 1) / BIG_BK * BIG_BK);
  // measured (us, tile kernel / copy, this kernel and the last rows): 16384 x 4608 x 1152 175 / 125, 32768 x 1152 x 4608 235 / 172,
  // 8192 x 3456 x 1152 68 / 62, 16384 x 1152 x 1152 49 / 43, 16384 x 1000 x 1168 46 / 42.  Below 1.5e10 products the two more
  // launches are not earned back (8192 x 2049 x 528 39 / 49), nor where the last rows are more than a sixteenth (8192 x 1152 x
  // 4608 69 / 78, 4096 x 4608 x 1152 51 / 52, 3000 x 4608 x 1152 38 / 40) or a third of the products are padding
  // (16384 x 2049 x 528 68 / 70)
  return work >= 1.55e10 && padded <= 1.34 * work && big_copy_rows(a) <= a.M / 16;
}

hipError_t launch_gemm_big_rows(const GemmArgs &a, hipStream_t st) {
  const int m1 = a.M - big_copy_rows(a), Kp = (a.K + BIG_BK - 1) / BIG_BK * BIG_BK;
  GemmArgs b = a, c = a;
  float *const y1 = a.y + (size_t)m1 * a.ldy;
  void *const wt = reinterpret_cast<void *>((reinterpret_cast<uintptr_t>(y1) + 15) & ~uintptr_t(15));
  b.M = m1;
  b.Wt = wt;
  c.M = a.M - m1;
  c.A = a.A + (size_t)m1 * a.lda;
  c.y = y1;
  hipError_t e = launch_tile_weight(a.W, wt, a.N, a.K, a.w4 ? 4 : 8, Kp, st);
  if (e == hipSuccess) e = a.w4 ? launch_big_as<8, EPI_F32, QC_SITE_QKV, true, false>(b, st) : launch_big_as<8, EPI_F32, QC_SITE_QKV, false, false>(b, st);
  return e == hipSuccess ? launch_gemm(c, EPI_F32, 1, st, QC_SITE_QKV) : e;
}

#undef QC_WAIT_VM_FOR2
#undef QC_WAIT_VM_FOR4
#undef QC_LDS_DONE_BARRIER
#undef QC_SB

}  // namespace qc
