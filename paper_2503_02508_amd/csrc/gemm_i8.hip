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

  gemm_epilogue<BM, BN, WM, WN, EPI, false, RBF>(p, acc, smem, m0, n0, z);
}

// ---------------------------------------------------------------------------------------------------------------
// Large-M kernel.  At M of several thousand rows the tile loop above is bound by LDS traffic (its writes run at a
// quarter of the read rate) and by the 64 bytes per clock a compute unit can pull through its vector memory path,
// so this kernel moves fewer bytes through both:
//   * tile 128 (M) x 256 (N), four wavefronts side by side along N, each 128 x 64 (4 x 2 blocks of 32 x 32: one LDS
//     fragment read feeds two MFMAs, one weight fragment four), two workgroups per compute unit so that one tile's
//     prologue and epilogue run under the other's main loop;
//   * weights never touch LDS: they are stored a second time in MFMA fragment order (fragment (n / 32, k / 32) =
//     64 lanes x 16 bytes, lane l = row n % 32 = l % 32, bytes 16 (l / 32) .. of the 32 k values; packed nibbles:
//     8 bytes per lane) and each wavefront streams the fragments of its own 64 columns straight into a ring of
//     registers, four k-groups deep (slots 2 par, 2 par + 1 for the two k-groups of a slab of parity par);
//   * activations go global -> registers -> LDS in slabs of 64 bytes of K (a thread moves two 16-byte chunks per
//     slab), two slabs in flight in registers, three slab buffers in LDS.  A slab row is 64 bytes, its four 16-byte
//     chunks XOR-swizzled with bits 2..3 of the row so that the fragment reads (32 consecutive rows, one chunk) are
//     free of bank conflicts;
//   * one barrier per slab, between its two k-groups: slab kt + 1 is written to LDS during the first k-group of slab
//     kt and read after that barrier; its buffer was last read in slab kt - 2, two barriers ago;
//   * one memory instruction is issued behind each MFMA (pinned with scheduling barriers), so a wavefront keeps its
//     matrix pipe fed while its loads, LDS writes and fragment reads are in flight.
// Every global load here is an ordinary register load issued through inline assembly (the compiler neither sees nor
// counts them); register loads complete in the order they were issued, so each wait on the vector memory counter below
// is the number of loads issued after the one it is for.  Per slab the order is: two activation loads (slab kt + 3),
// two ring loads (k-group 2 kt + 4), [barrier], two ring loads (k-group 2 kt + 5).
// (A variant that sent the activations straight to LDS (global_load_lds_dwordx4) was measured first: those loads and
// register loads share the counter but complete out of order with respect to each other, so counted waits gave wrong
// fragments on some boxes, and draining the counter before every barrier cost 8 % against this version.)
#define QC_WAIT_VM(n) asm volatile("s_waitcnt vmcnt(" #n ")" ::: "memory")
// the same, tied to registers that become valid with it: their uses cannot be moved above the wait
#define QC_WAIT_VM_FOR2(n, r0, r1) asm volatile("s_waitcnt vmcnt(" #n ")" : "+v"(r0), "+v"(r1)::"memory")
#define QC_WAIT_VM_FOR4(n, r0, r1, r2, r3) asm volatile("s_waitcnt vmcnt(" #n ")" : "+v"(r0), "+v"(r1), "+v"(r2), "+v"(r3)::"memory")
// all LDS writes of this wavefront done, then the workgroup barrier
#define QC_LDS_DONE_BARRIER asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory")

template <int EPI, int TAG, bool W4, bool RBF, bool RAG>
__global__ __launch_bounds__(256, 2) void gemm_i8_big_kernel(GemmArgs p) {
  constexpr int BM = 128, BN = 256, WM = 1, WN = 4, TM = 4, TN = 2, BK = 64;
  constexpr int RB = 4, NB = 3, NS = 2;           // ring depth (k-groups), LDS slab buffers, slabs in flight in registers
  constexpr int SLAB = BM * BK;
  extern __shared__ __align__(16) unsigned char smem[];

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
  const int wn0 = wave * (TN * 32);

  // activations: load i of thread tid covers row 64 i + tid / 4, 16-byte chunk tid % 4 of a slab and is written to
  // LDS at the swizzled position of that chunk.  Rows beyond M re-read row M - 1.
  unsigned aoff[2], lpos[2];
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const int row = i * 64 + (tid >> 2), c = tid & 3;
    aoff[i] = (unsigned)(min(m0 + row, p.M - 1) - m0) * (unsigned)p.lda + c * 16;
    lpos[i] = row * BK + ((c ^ ((row >> 2) & 3)) * 16);
  }
  const int8_t *abase = p.A + (size_t)m0 * p.lda;
  const int nk = p.K / BK, ng = p.K / 32;
  v4i ra[NS][2];
  auto load_a = [&](int q, int kt, int i) {       // slabs past the end re-read the last one (never used)
    asm volatile("global_load_dwordx4 %0, %1, %2" : "=v"(ra[q][i]) : "v"(aoff[i]), "s"(abase + min(kt, nk - 1) * BK) : "memory");
  };
  auto write_a = [&](int q, int kt, int i) { *(v4i *)(smem + (kt % NB) * SLAB + lpos[i]) = ra[q][i]; };

  // weight fragment streams of this wavefront: n-blocks (n0 + wn0) / 32 + j (blocks past N re-read the last block)
  constexpr int FRAG = W4 ? 512 : 1024;           // bytes per fragment
  typedef typename std::conditional<W4, v2i, v4i>::type wfrag_t;
  const int nblocks = p.N / 32;
  const int8_t *sb[TN];
#pragma unroll
  for (int j = 0; j < TN; ++j) sb[j] = (const int8_t *)p.Wt + (size_t)min((n0 + wn0) / 32 + j, nblocks - 1) * ng * FRAG;
  const unsigned lane_off = lane * (W4 ? 8 : 16);
  wfrag_t bq[RB][TN];
  auto load_ring = [&](int slot, int g) {         // groups past the end re-read the last one (never used)
    const size_t go = (size_t)min(g, ng - 1) * FRAG;
#pragma unroll
    for (int j = 0; j < TN; ++j) {
      if (W4) asm volatile("global_load_dwordx2 %0, %1, %2" : "=v"(bq[slot][j]) : "v"(lane_off), "s"(sb[j] + go) : "memory");
      else asm volatile("global_load_dwordx4 %0, %1, %2" : "=v"(bq[slot][j]) : "v"(lane_off), "s"(sb[j] + go) : "memory");
    }
  };

  v16i acc[TM][TN];
  if constexpr (EPI == EPI_GELU_Q) {
    // the accumulators start at minus the zero-point term a_z * wsum[n] of their column (the weights are the first
    // MFMA operand here: register 4 rg + e of block j is column 32 j + 8 rg + 4 (lane / 32) + e), so the epilogue
    // finds acc - a_z * wsum[n] ready; the loads complete under the prologue's wait for the first slabs
    const int a_z = p.a_qp ? p.a_qp[0].z : p.a_zp;
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int rg = 0; rg < 4; ++rg) {
        const v4i ws = *(const v4i *)(p.wsum + min(n0 + wn0 + j * 32 + rg * 8 + (lane >> 5) * 4, p.N - 4));
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
          for (int e = 0; e < 4; ++e) acc[i][j][rg * 4 + e] = -(a_z * ws[e]);
      }
  } else {
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j)
#pragma unroll
        for (int q = 0; q < 16; ++q) acc[i][j][q] = 0;
  }

  const int frow = lane & 31, fsw = (frow >> 2) & 3;
  v4i fa[2][TM];
  auto read_frag = [&](int f, int kt, int kg, int i) {
    fa[f][i] = *(const v4i *)(smem + (kt % NB) * SLAB + frow * BK + ((((lane >> 5) + 2 * kg) ^ fsw) * 16) + i * 32 * BK);
  };
  v4i wf[TN];
  auto unpack_ring = [&](int slot) {
#pragma unroll
    for (int j = 0; j < TN; ++j) {
      if constexpr (W4) wf[j] = unpack_w4(bq[slot][j]);
      else wf[j] = bq[slot][j];
    }
  };
  auto mfma = [&](int f, int i, int j) {
    if (EPI == EPI_GELU_Q) acc[i][j] = __builtin_amdgcn_mfma_i32_32x32x32_i8(wf[j], fa[f][i], acc[i][j], 0, 0, 0);
    else acc[i][j] = __builtin_amdgcn_mfma_i32_32x32x32_i8(fa[f][i], wf[j], acc[i][j], 0, 0, 0);
  };
#define QC_SB __builtin_amdgcn_sched_barrier(0)

  // prologue: slab 0 -> LDS, slabs 1 and 2 -> the two register sets, ring groups 0 .. 3
  load_a(0, 0, 0); load_a(0, 0, 1);
  load_a(1, 1, 0); load_a(1, 1, 1);
#pragma unroll
  for (int g = 0; g < RB; ++g) load_ring(g, g);
  QC_SB;
  QC_WAIT_VM_FOR4(0, ra[0][0], ra[0][1], ra[1][0], ra[1][1]);
  write_a(0, 0, 0); write_a(0, 0, 1);
  QC_SB;
  load_a(0, 2, 0); load_a(0, 2, 1);
  QC_LDS_DONE_BARRIER;
#pragma unroll
  for (int i = 0; i < TM; ++i) read_frag(0, 0, 0, i);
  QC_SB;

  // Slab kt = k-groups 2 kt and 2 kt + 1, ring slots 2 par and 2 par + 1 (par = kt % 2), register set q = (kt + 1) % 2
  // holds slab kt + 1.  On entry: slab kt is in LDS and published; fa[0] holds (or awaits) the fragments of (kt,
  // group 0); ring groups up to 2 kt + 3 and activation slabs up to kt + 2 are requested.
  // Loads issued after the one a wait is for:
  //   top of the slab, for ring group 2 kt and for slab kt + 1 in registers (both requested in the first half of slab
  //   kt - 2, the activations first): ring group 2 kt - 1 ... (2) and the six loads of slab kt - 1                 = 8
  //   (slab 1 needs the prologue's load of slab 2, which has only the six loads of slab 0 behind it:                 6)
  //   after the barrier, for ring group 2 kt + 1 (requested at the end of slab kt - 2): six loads of slab kt - 1 and
  //   the four of this slab's first half                                                                          = 10
  static_assert(RB == 4 && NB == 3 && NS == 2 && TM == 4 && TN == 2, "waits and slots below are written for this depth");
  auto slab = [&](int kt, int par, auto first) {
    const int q = (kt + 1) % NS;
    if constexpr (decltype(first)::value) QC_WAIT_VM_FOR4(6, bq[2 * par][0], bq[2 * par][1], ra[q][0], ra[q][1]);
    else QC_WAIT_VM_FOR4(8, bq[2 * par][0], bq[2 * par][1], ra[q][0], ra[q][1]);
    unpack_ring(2 * par);
    QC_SB;
    mfma(0, 0, 0); write_a(q, kt + 1, 0); QC_SB;
    mfma(0, 0, 1); write_a(q, kt + 1, 1); QC_SB;
    mfma(0, 1, 0); read_frag(1, kt, 1, 0); QC_SB;
    mfma(0, 1, 1); read_frag(1, kt, 1, 1); QC_SB;
    mfma(0, 2, 0); read_frag(1, kt, 1, 2); QC_SB;
    mfma(0, 2, 1); read_frag(1, kt, 1, 3); QC_SB;
    mfma(0, 3, 0); load_a(q, kt + 3, 0); QC_SB;
    mfma(0, 3, 1); load_a(q, kt + 3, 1); QC_SB;
    load_ring(2 * par, 2 * kt + 4);
    QC_SB;
    QC_LDS_DONE_BARRIER;
    QC_WAIT_VM_FOR2(10, bq[2 * par + 1][0], bq[2 * par + 1][1]);
    unpack_ring(2 * par + 1);
    QC_SB;
    mfma(1, 0, 0); QC_SB;
    mfma(1, 0, 1); QC_SB;
    mfma(1, 1, 0); QC_SB;
    mfma(1, 1, 1); QC_SB;
    mfma(1, 2, 0); read_frag(0, kt + 1, 0, 0); QC_SB;
    mfma(1, 2, 1); read_frag(0, kt + 1, 0, 1); QC_SB;
    mfma(1, 3, 0); read_frag(0, kt + 1, 0, 2); QC_SB;
    mfma(1, 3, 1); read_frag(0, kt + 1, 0, 3); QC_SB;
    load_ring(2 * par + 1, 2 * kt + 5);
    QC_SB;
  };
  // K is a multiple of 128 (checked by the launcher): an even number of slabs, at least two
  slab(0, 0, std::false_type());
  slab(1, 1, std::true_type());
  for (int kt = 2; kt + 2 <= nk; kt += 2) {
    slab(kt, 0, std::false_type());
    slab(kt + 1, 1, std::false_type());
  }
#undef QC_SB
  // the loads that ran past the end (clamped addresses) must have landed before registers are reused, and every
  // wavefront must be past its last fragment read before the epilogue reuses LDS
  QC_WAIT_VM(0);
  __builtin_amdgcn_sched_barrier(0);
  __syncthreads();
  gemm_epilogue<BM, BN, WM, WN, EPI, true, RBF, RAG>(p, acc, smem, m0, n0, 0);
}

constexpr int BIG_SMEM_LOOP = 3 * 128 * 64;
constexpr int BIG_SMEM_STAGE = 128 * (128 + 4) * 4;                      // one staged column half, float32 (QKV scatter, residual)
constexpr int BIG_SMEM_GELU = 256 * 12 + 128 * (256 + 16) + 16 + GELU_FIX_CAP * 16;

template <int EPI, int TAG, bool W4, bool RBF, bool RAG = false>
static hipError_t launch_big_fmt(const GemmArgs &a, hipStream_t st) {
  // launches whose tiles are not all whole and inside one batch element take the variant that handles the others
  if constexpr (!RAG && (EPI == EPI_RESID || EPI == EPI_QKV)) {
    if (a.M % 128 || a.rows_per_batch % 128) return launch_big_fmt<EPI, TAG, W4, RBF, true>(a, st);
  }
  constexpr int smem_epi = EPI == EPI_GELU_Q ? BIG_SMEM_GELU : BIG_SMEM_STAGE;
  constexpr int smem = smem_epi > BIG_SMEM_LOOP ? smem_epi : BIG_SMEM_LOOP;
  static_assert(2 * smem <= 160 * 1024, "two workgroups per compute unit");
  static bool attr_set = false;
  auto kern = gemm_i8_big_kernel<EPI, TAG, W4, RBF, RAG>;
  if (!attr_set) {
    hipError_t e = hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize, smem);
    if (e != hipSuccess) return e;
    attr_set = true;
  }
  const int tiles = ((a.M + 127) / 128) * ((a.N + 255) / 256);
  GemmArgs b = a;
  {
    // tile rows per group: every column tile of a group resident on its XCD at once (64 workgroup slots), at most 4
    // rows (measured on M = 32768: 4 rows beat 16 by 2 - 9 % on the four linears of DiT-XL/2, 1 - 2 rows lose again)
    const int tiles_n = (a.N + 255) / 256, fit = 64 / tiles_n;
    b.group_m = fit < 1 ? 1 : (fit > 4 ? 4 : fit);
  }
  hipLaunchKernelGGL(kern, dim3(((tiles + 7) / 8) * 8), dim3(256), smem, st, b);
  return hipGetLastError();
}

// the residual epilogue is compiled twice: for float32 stream and cache, and for the bfloat16 variants of either
template <int EPI, int TAG, bool W4>
static hipError_t launch_big(const GemmArgs &a, hipStream_t st) {
  if constexpr (EPI == EPI_RESID) {
    if (a.x_bf16 || a.cache_bf16) return launch_big_fmt<EPI, TAG, W4, true>(a, st);
  }
  return launch_big_fmt<EPI, TAG, W4, false>(a, st);
}

// The large-M kernel takes over when the weights exist in fragment order, the shape fits its loop (K a multiple of
// 128, N of 32, 16-byte aligned rows), a 128-row tile holds rows of at most two batch elements (its epilogues are
// compiled without the general paths) and the launch has enough 128 x 256 tiles for it to pay.
static bool use_big(const GemmArgs &a, int epi, int nz) {
  if (!a.Wt || nz != 1 || a.sel_D || a.acc_out) return false;
  if (a.K % 128 || a.N % 32 || a.lda % 16) return false;
  if (epi == EPI_RESID && a.rows_per_batch < 128) return false;
  if (epi == EPI_QKV && (a.y || a.rows_per_batch < 128 || (a.N / 3) % 128 || a.hd % 4 || a.Tp % 8)) return false;
  const long long tiles = (long long)((a.M + 127) / 128) * ((a.N + 255) / 256);
  // measured alone on the chip (DiT-XL/2 shapes): 160 tiles (proj / fc2 at M = 4096) run 20 % faster here than in the
  // tile kernel, 224 - 288 tiles (QKV / fc1 at M = 2048) 0 - 10 % faster, 112 - 144 tiles (M = 1024) 3 - 15 % slower,
  // 80 tiles (proj / fc2 at M = 2048) 15 - 25 % slower
  return tiles >= 150;
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
  static bool attr_set = false;
  auto kern = gemm_i8_kernel<BM, BN, WM, WN, EPI, TAG, W4, PF, BK, RBF>;
  if (!attr_set) {
    hipError_t e = hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize, smem);
    if (e != hipSuccess) return e;
    attr_set = true;
  }
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
  if constexpr (EPI != EPI_F32) {
    if (use_big(a, EPI, nz)) return launch_big<EPI, TAG, W4>(a, st);
  }
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
  if (epi == EPI_GELU_Q) return launch_epi<EPI_GELU_Q, QC_SITE_FC1>(a, nz, st);
  if (epi == EPI_RESID)
    return site == QC_SITE_FC2 ? launch_epi<EPI_RESID, QC_SITE_FC2>(a, nz, st) : launch_epi<EPI_RESID, QC_SITE_PROJ>(a, nz, st);
  if (epi == EPI_QKV) return launch_epi<EPI_QKV, QC_SITE_QKV>(a, nz, st);
  return site == QC_SITE_ADA ? launch_epi<EPI_F32, QC_SITE_ADA>(a, nz, st) : launch_epi<EPI_F32, QC_SITE_QKV>(a, nz, st);
}

}  // namespace qc

