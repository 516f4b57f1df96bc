// softmax(Q K^T / sqrt(d)) V per (batch, head) in fp32 on the matrix cores
// (v_mfma_f32_16x16x4_f32), keys streamed through LDS in tiles of 64 with an
// online softmax, so no T x T matrix ever exists.  The output is quantised with
// the attention-projection site's (s, z) on the way out (Eq. 1), or written as
// fp32 for calibration.
//
// Work split: one workgroup = 64 queries of one (batch, head); each of its four
// wavefronts owns 16 queries.  The products are formed transposed so that a
// lane always owns ONE query:
//   S^T = K Q^T : A operand = K rows (keys), B operand = Q^T (queries)
//   O^T = V^T P^T : A operand = V^T rows (features), B operand = P^T
// MFMA 16x16x4 layouts: lane l supplies A[row l%16][k l/16] and B[k l/16][col l%16];
// result register r of lane l is row 4*(l/16)+r, column l%16.  Hence the S^T
// result of lane (q = l%16, g = l/16) holds keys 4g..4g+3 of query q, which is
// exactly the B operand P^T[key][q] needs if the k index of the second product
// enumerates keys as 4g + r; the V^T operand is read with the same enumeration.
// The running max / sum of a query are per-lane scalars, shared across the four
// g groups with two shuffles.
//
// What bounds it: the float32 matrix rate of a wavefront that is alone on its SIMD (42 of 32 clocks a product) and, at a few
// hundred tokens, the first round trips.  So nothing stands in front of the products: the next tile of keys comes into registers
// while one is multiplied, the four blocks of keys alternate (a chain on one accumulator waits for itself), and the fragments
// are read from LDS a step ahead.  Us (16 heads of 72): 1 x 256 tokens 26.5 -> 18.1, 4 x 256 29.2 -> 22.1, 2 x 425 45.2 -> 31.8, 1 x 1024
// 98.6 -> 66.0, 1 x 4096 992 -> 874.  (Workgroups of 32 queries, twice as many: 1 x 256 21.2, 4 x 256 27.7, 1 x 4096 1200, against 20.1, 23.9
// and 926 without the fragments read ahead.)
#include <type_traits>

#include "qc_internal.h"

namespace qc {

typedef float v4f __attribute__((ext_vector_type(4)));

template <int DP>   // head dim padded to a multiple of 16
__global__ __launch_bounds__(256) void attention_kernel(const float *__restrict__ qkv, int T, int H, int hd,
                                                        const QParam *qp, int8_t *__restrict__ q_out,
                                                        float *__restrict__ f32_out, float scale_log2e) {
  constexpr int S = DP + 4;          // LDS row stride in floats: 8 consecutive rows hit 8 distinct 16-byte bank groups
  constexpr int NC = DP / 16;        // 16-wide feature chunks
  __shared__ __align__(16) float Ks[64 * S];
  __shared__ __align__(16) float Vs[64 * S];

  const int D = H * hd;
  const int bh = blockIdx.y, b = bh / H, h = bh % H;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int ql = lane & 15, g = lane >> 4;
  const int q_row = blockIdx.x * 64 + wave * 16 + ql;            // query of this lane
  const float *base = qkv + (size_t)b * T * 3 * D + (size_t)h * hd;

  // Q^T operand: features 16c + 4g + u of this lane's query, pre-scaled by log2(e)/sqrt(d)
  v4f qf[NC];
#pragma unroll
  for (int c = 0; c < NC; ++c) {
    const int e = 16 * c + 4 * g;
    v4f v = {0.f, 0.f, 0.f, 0.f};
    if (q_row < T && e < hd) v = *(const v4f *)(base + (size_t)q_row * 3 * D + e);
    qf[c] = v * scale_log2e;
  }

  v4f o[NC];
#pragma unroll
  for (int c = 0; c < NC; ++c) o[c] = (v4f){0.f, 0.f, 0.f, 0.f};
  float m_run = -INFINITY, l_run = 0.0f;

  // K and V tiles, zero padded in features and keys; the next tile's loads are in flight while a tile is multiplied
  constexpr int NL = NC;             // 64 rows x 4 NC chunks, 256 threads
  v4f kreg[NL], vreg[NL];
  auto load_tile = [&](int k0) {
#pragma unroll
    for (int u = 0; u < NL; ++u) {
      const int i = tid + 256 * u, r = i / (DP / 4), e = (i % (DP / 4)) * 4;
      kreg[u] = vreg[u] = (v4f){0.f, 0.f, 0.f, 0.f};
      if (k0 + r < T && e < hd) {
        const float *src = base + (size_t)(k0 + r) * 3 * D + e;
        kreg[u] = *(const v4f *)(src + D);
        vreg[u] = *(const v4f *)(src + 2 * D);
      }
    }
  };
  load_tile(0);
  for (int k0 = 0; k0 < T; k0 += 64) {
    __syncthreads();
#pragma unroll
    for (int u = 0; u < NL; ++u) {
      const int i = tid + 256 * u, r = i / (DP / 4), e = (i % (DP / 4)) * 4;
      *(v4f *)(Ks + r * S + e) = kreg[u];
      *(v4f *)(Vs + r * S + e) = vreg[u];
    }
    __syncthreads();
    if (k0 + 64 < T) load_tile(k0 + 64);

    // S^T tile: 4 blocks of 16 keys, whose chains of products alternate
    v4f s[4];
#pragma unroll
    for (int kt = 0; kt < 4; ++kt) s[kt] = (v4f){0.f, 0.f, 0.f, 0.f};
    v4f kf[2][4];
    auto load_k = [&](int c) {
#pragma unroll
      for (int kt = 0; kt < 4; ++kt) kf[c & 1][kt] = *(const v4f *)(Ks + (kt * 16 + ql) * S + 16 * c + 4 * g);
    };
    load_k(0);
#pragma unroll
    for (int c = 0; c < NC; ++c) {
      if (c + 1 < NC) load_k(c + 1);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int u = 0; u < 4; ++u)
#pragma unroll
        for (int kt = 0; kt < 4; ++kt) s[kt] = __builtin_amdgcn_mfma_f32_16x16x4f32(kf[c & 1][kt][u], qf[c][u], s[kt], 0, 0, 0);
      __builtin_amdgcn_sched_barrier(0);
    }
    // the first V fragments are requested before the softmax arithmetic
    float vf[2][4][NC];
    auto load_v = [&](int kt) {
#pragma unroll
      for (int r = 0; r < 4; ++r)
#pragma unroll
        for (int c = 0; c < NC; ++c) vf[kt & 1][r][c] = Vs[(kt * 16 + 4 * g + r) * S + ql + 16 * c];
    };
    load_v(0);
    // mask keys past the end, running max
    float mx = -INFINITY;
#pragma unroll
    for (int kt = 0; kt < 4; ++kt)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        if (k0 + kt * 16 + 4 * g + r >= T) s[kt][r] = -INFINITY;
        mx = fmaxf(mx, s[kt][r]);
      }
    mx = fmaxf(mx, __shfl_xor(mx, 16, 64));
    mx = fmaxf(mx, __shfl_xor(mx, 32, 64));
    const float m_new = fmaxf(m_run, mx);           // finite: every tile holds at least one valid key
    const float alpha = exp2f(m_run - m_new);
    m_run = m_new;
    l_run *= alpha;
#pragma unroll
    for (int c = 0; c < NC; ++c) o[c] *= alpha;
#pragma unroll
    for (int kt = 0; kt < 4; ++kt)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const float pv = exp2f(s[kt][r] - m_new);
        s[kt][r] = pv;
        l_run += pv;
      }
    // O^T += V^T P^T
#pragma unroll
    for (int kt = 0; kt < 4; ++kt) {
      if (kt < 3) load_v(kt + 1);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int r = 0; r < 4; ++r)
#pragma unroll
        for (int c = 0; c < NC; ++c) o[c] = __builtin_amdgcn_mfma_f32_16x16x4f32(vf[kt & 1][r][c], s[kt][r], o[c], 0, 0, 0);
      __builtin_amdgcn_sched_barrier(0);
    }
  }

  l_run += __shfl_xor(l_run, 16, 64);
  l_run += __shfl_xor(l_run, 32, 64);
  if (q_row >= T) return;
  const float inv = 1.0f / l_run;
  float qs = 1.0f;
  int qz = 0;
  if (qp) {
    QParam t = *qp;
    qs = t.s;
    qz = t.z;
  }
  const size_t out_row = ((size_t)b * T + q_row) * D + (size_t)h * hd;
#pragma unroll
  for (int c = 0; c < NC; ++c) {
    const int e = 16 * c + 4 * g;
    if (e >= hd) continue;
    const v4f v = o[c] * inv;
    if (q_out) {
      int c0, c1, c2, c3;
      float r;
      r = rintf(v[0] / qs) + (float)qz; c0 = (int)fminf(fmaxf(r, -128.f), 127.f);
      r = rintf(v[1] / qs) + (float)qz; c1 = (int)fminf(fmaxf(r, -128.f), 127.f);
      r = rintf(v[2] / qs) + (float)qz; c2 = (int)fminf(fmaxf(r, -128.f), 127.f);
      r = rintf(v[3] / qs) + (float)qz; c3 = (int)fminf(fmaxf(r, -128.f), 127.f);
      *(unsigned *)(q_out + out_row + e) = (unsigned)(c0 & 0xFF) | ((unsigned)(c1 & 0xFF) << 8) |
                                           ((unsigned)(c2 & 0xFF) << 16) | ((unsigned)(c3 & 0xFF) << 24);
    }
    if (f32_out) *(v4f *)(f32_out + out_row + e) = v;
  }
}

template <int DP>
static hipError_t launch_attention_dp(const float *qkv, int B, int T, int H, int hd, const QParam *qp, int8_t *q_out, float *f32_out, hipStream_t st) {
  const float sl2 = 1.4426950408889634f / sqrtf((float)hd);
  hipLaunchKernelGGL(attention_kernel<DP>, dim3((T + 63) / 64, B * H), dim3(256), 0, st, qkv, T, H, hd, qp, q_out, f32_out, sl2);
  return hipGetLastError();
}

hipError_t launch_attention(const float *qkv, int B, int T, int H, int hd, const QParam *qp, int8_t *q_out, float *f32_out,
                            hipStream_t st) {
  switch ((hd + 15) / 16) {
    case 1: return launch_attention_dp<16>(qkv, B, T, H, hd, qp, q_out, f32_out, st);
    case 2: return launch_attention_dp<32>(qkv, B, T, H, hd, qp, q_out, f32_out, st);
    case 3: return launch_attention_dp<48>(qkv, B, T, H, hd, qp, q_out, f32_out, st);
    case 4: return launch_attention_dp<64>(qkv, B, T, H, hd, qp, q_out, f32_out, st);
    case 5: return launch_attention_dp<80>(qkv, B, T, H, hd, qp, q_out, f32_out, st);
    case 6: return launch_attention_dp<96>(qkv, B, T, H, hd, qp, q_out, f32_out, st);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace qc

// ---------------------------------------------------------------------------
// Production kernel: the same online-softmax tiling on the fp16 matrix cores
// (v_mfma_f32_16x16x32_f16, 16x the fp32 MFMA rate).  Every operand is carried
// as an fp16 pair (high part + low part, ~22 significant bits, split when a tile
// is staged) and every product is formed as hi*hi + hi*lo + lo*hi with fp32
// accumulation, which keeps the result at fp32 accuracy so that the int8 codes
// quantised from it stay the oracle's.  The probabilities are split the same
// way after the exponential.
//
// Global layouts (float32, written by the QKV GEMM epilogue): Q and K
// [B, H, T, d]; V transposed [B, H, DPv, Tp] with the keys of each group of 32
// interleaved in units of 4 (vt_pos).
//
// Layout facts used (16x16x32 f16): lane l supplies A[row l%16][k 8(l/16)..+7]
// and B[k 8(l/16)..+7][col l%16] as 8 halves; result register r of lane l is
// row 4(l/16)+r, column l%16.  With S^T = K Q^T a lane owns one query and the
// keys 4g..4g+3 of each block of 16; two such blocks give the 8 k-values of the
// P^T operand of O^T = V^T P^T, whose key order (4g..4g+3, 16+4g..16+4g+3) is
// the order V^T was stored in.
//
// One workgroup = 128 queries of one (batch, head); each of the 4 wavefronts
// owns two blocks of 16 queries, so every K / V^T fragment read from LDS feeds
// two MFMAs.  Two key tiles lie in LDS: while one is multiplied, the next one is
// split from registers into the other behind the products of the scores, and the
// one after that comes into the registers from then on.  (One query block a
// wavefront, or no room for two: one tile, written between two barriers.)
namespace qc {

typedef _Float16 v8h __attribute__((ext_vector_type(8)));
typedef _Float16 v4h __attribute__((ext_vector_type(4)));
typedef unsigned v4u __attribute__((ext_vector_type(4)));
typedef unsigned v2u __attribute__((ext_vector_type(2)));

// Two float32 values -> their hi halves (the values rounded to fp16, packed) and lo halves (what the rounding left,
// again rounded to fp16): hi + lo carries about 22 significant bits.  Three instructions per pair: one packed conversion,
// then the mixed-precision multiply-add forms a - (float)hi (exact in float32) from the stored hi half and rounds it to
// fp16 in one go, into either half of the lo word.
typedef float v2f __attribute__((ext_vector_type(2)));
typedef _Float16 v2h __attribute__((ext_vector_type(2)));
__device__ __forceinline__ void split_pair(float a, float b, unsigned &hi, unsigned &lo) {
  hi = __builtin_bit_cast(unsigned, __builtin_convertvector((v2f){a, b}, v2h));
  asm("v_fma_mixlo_f16 %0, %1, -1.0, %2 op_sel_hi:[1,0,0]" : "=v"(lo) : "v"(hi), "v"(a));
  asm("v_fma_mixhi_f16 %0, %1, -1.0, %2 op_sel:[1,0,0] op_sel_hi:[1,0,0]" : "+v"(lo) : "v"(hi), "v"(b));
}
__device__ __forceinline__ void split_pairs(v4f v, v2u &hi, v2u &lo) {
  unsigned h0, l0, h1, l1;
  split_pair(v[0], v[1], h0, l0);
  split_pair(v[2], v[3], h1, l1);
  hi = (v2u){h0, h1};
  lo = (v2u){l0, l1};
}

// The same split of eight values into the two operands of a product that may follow at once.  v_fma_mixhi_f16 writes half a
// register, and a product that reads that register as the first half of an operand less than two issue slots later (the
// second half: one) gets its old upper half; the compiler does not see what the assembly holds, so the wait is part of it.
__device__ __forceinline__ void split_operand(v4f a, v4f b, v8h &hi, v8h &lo) {
  unsigned h0 = __builtin_bit_cast(unsigned, __builtin_convertvector((v2f){a[0], a[1]}, v2h));
  unsigned h1 = __builtin_bit_cast(unsigned, __builtin_convertvector((v2f){a[2], a[3]}, v2h));
  unsigned h2 = __builtin_bit_cast(unsigned, __builtin_convertvector((v2f){b[0], b[1]}, v2h));
  unsigned h3 = __builtin_bit_cast(unsigned, __builtin_convertvector((v2f){b[2], b[3]}, v2h));
  unsigned l0, l1, l2, l3;
  asm("v_fma_mixlo_f16 %0, %4, -1.0, %8 op_sel_hi:[1,0,0]\n\t"
      "v_fma_mixlo_f16 %1, %5, -1.0, %10 op_sel_hi:[1,0,0]\n\t"
      "v_fma_mixlo_f16 %2, %6, -1.0, %12 op_sel_hi:[1,0,0]\n\t"
      "v_fma_mixlo_f16 %3, %7, -1.0, %14 op_sel_hi:[1,0,0]\n\t"
      "v_fma_mixhi_f16 %0, %4, -1.0, %9 op_sel:[1,0,0] op_sel_hi:[1,0,0]\n\t"
      "v_fma_mixhi_f16 %1, %5, -1.0, %11 op_sel:[1,0,0] op_sel_hi:[1,0,0]\n\t"
      "v_fma_mixhi_f16 %2, %6, -1.0, %13 op_sel:[1,0,0] op_sel_hi:[1,0,0]\n\t"
      "v_fma_mixhi_f16 %3, %7, -1.0, %15 op_sel:[1,0,0] op_sel_hi:[1,0,0]\n\t"
      "s_nop 1"
      : "=&v"(l0), "=&v"(l1), "=&v"(l2), "=&v"(l3)
      : "v"(h0), "v"(h1), "v"(h2), "v"(h3), "v"(a[0]), "v"(a[1]), "v"(a[2]), "v"(a[3]), "v"(b[0]), "v"(b[1]), "v"(b[2]), "v"(b[3]));
  hi = __builtin_bit_cast(v8h, (v4u){h0, h1, h2, h3});
  lo = __builtin_bit_cast(v8h, (v4u){l0, l1, l2, l3});
}

// Second half of both kernels' epilogue, run by the whole workgroup once the codes of its NQ queries (the first of them q_first)
// are staged and the doubtful ones queued (FIX_CAP of them at most): the queued outputs are decided again in float64, then
// the rows go out.  qbase, kbase, vbase: float32 Q, K and V^T of the (batch, head); m_s: reference point of the exponentials
// per query; parts: FB * NW * 16 bytes of LDS, [output][wavefront][2]; q_out: the head's first byte in the batch element's
// first output row.
// ONE: at most 64 NW keys, so that a wavefront has one group of them, the same for all outputs: its rows are loaded once and no next group is
// requested.  A kernel of its own for each: with both ways in one, registers went to scratch memory, and a launch that has any, even if
// only this part uses it, is 10 - 20 % slower.  16 heads of 72, us, the general way | ONE: 128 x 256 tokens 179 | 177, 64 x 256 87 | 87, 16 x 256
// 29.3 | 28.8, 8 x 256 18.4 | 18.1, 4 x 256 13.8 | 13.3; runs of 8 latents of 256 tokens 0.4 % faster.
// What it costs: a decision takes about 4300 clocks at 256 keys and 10 500 at 1024.  The mean
// is 0.28 decisions a workgroup of 128 queries at 256 keys, 1.0 at 1024, 4.1 at 4096; but a launch of few rounds of workgroups ends with those that
// have several.  Us with decisions | with the queue left empty | with this part compiled out: 8 x 1024 tokens 150.5 | 120.2 | 120.1, 64 x 256
// 87 | 82 | 82, 2 x 4096 724 | 433 | 433, 4 x 256 13.3 | 11.0 | 10.5: all of it is the decisions themselves, nothing registers or code size.
constexpr int FIX_CAP = 192;
template <int NEB, int NQ, int NW, int FB, bool ONE>
__device__ __forceinline__ void decide_again_and_store(unsigned char *stage, const int *fix_cnt, const int *fix_ent, double *parts,
                                                       const float *m_s, const float *qbase, const float *kbase, const float *vbase,
                                                       int q_first, int T, int Tp, int hd, int D, float qs, float qz,
                                                       int8_t *__restrict__ q_out) {
  constexpr int SRB = 16 * NEB;                   // staged row: the head's features, padded
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  // softmax(q K^T / sqrt(d)) V[:, feature] in float64 for every queued output.  The reference point of the exponentials is
  // the running max of the fast path (any point near the maximum gives the same quotient), so the parts of a sum need no
  // common maximum: wavefront w takes the groups w, w + NW, ... of 64 keys of every output and the parts meet in LDS.  Four
  // lanes share a key row (lane h: 16-byte chunks h, h + 4, ...) and take four keys of a group, 16 apart; a row of the
  // next group is requested as soon as the current one is used, and after the exchange each lane has one key's score: one
  // exponential per lane and group.  About 250 float64-rate instructions per 64 keys are what bounds it.
  const int nfix = min(*fix_cnt, FIX_CAP);
  const double rs = 1.0 / sqrt((double)hd);
  const int h4 = lane & 3, kl = lane >> 2;
  for (int base = 0; base < nfix; base += FB) {
    const int nb = min(nfix - base, FB);
    if constexpr (ONE) {
      v4f kv[4][NEB];
      // this lane's chunks of a key row: h4, h4 + 4, ...; the last one is clamped into the row (its query operand is zero then)
      const auto load_row = [&](int key0, v4f (&dst)[NEB]) {
        int ln = lane;
        asm volatile("" : "+v"(ln));              // (the places are formed when they are needed, not kept)
        const int h4 = ln & 3, kl = ln >> 2;
        const unsigned r = (unsigned)(min(key0 + kl, T - 1) * hd), clast = (unsigned)min(16 * (NEB - 1) + 4 * h4, hd - 4);
#pragma unroll
        for (int c = 0; c < NEB - 1; ++c) dst[c] = *(const v4f *)(kbase + (r + 4 * h4) + 16 * c);
        dst[NEB - 1] = *(const v4f *)(kbase + (r + clast));
      };
      const auto load_group = [&]() {
#pragma unroll
        for (int u = 0; u < 4; ++u) load_row(64 * wave + 16 * u, kv[u]);
      };
      load_group();
#pragma unroll 1
      for (int fi = 0; fi < nb; ++fi) {
        const int qloc = __builtin_amdgcn_readfirstlane(fix_ent[2 * (base + fi)]);
        const int feat = __builtin_amdgcn_readfirstlane(fix_ent[2 * (base + fi) + 1]);
        int ln = lane;
        asm volatile("" : "+v"(ln));
        const int h4 = ln & 3, kl = ln >> 2;
        const float *qr = qbase + (size_t)(q_first + qloc) * hd;
        const float *vrow = vbase + (size_t)feat * Tp;          // V^T row of the feature, keys in vt_pos order
        const float v = vrow[(unsigned)vt_pos(min(64 * wave + 16 * h4 + kl, Tp - 1))];
        double qd[NEB][4];
#pragma unroll
        for (int c = 0; c < NEB; ++c) {
          const int f = 16 * c + 4 * h4;
          const v4f t4 = *(const v4f *)(qr + (unsigned)min(f, hd - 4));
#pragma unroll
          for (int e = 0; e < 4; ++e) qd[c][e] = f < hd ? (double)t4[e] : 0.0;
        }
        const double mref = (double)m_s[qloc] * 0.6931471805599453;     // base 2 -> natural
        double den = 0.0, num = 0.0;
        if (64 * wave < T) {
          double sc = 0.0;
#pragma unroll
          for (int u = 0; u < 4; ++u) {
            double a0 = 0.0, a1 = 0.0;
#pragma unroll
            for (int c = 0; c < NEB; ++c) {
              a0 = fma(qd[c][0], (double)kv[u][c][0], a0);
              a1 = fma(qd[c][1], (double)kv[u][c][1], a1);
              a0 = fma(qd[c][2], (double)kv[u][c][2], a0);
              a1 = fma(qd[c][3], (double)kv[u][c][3], a1);
            }
            a0 += a1;
            a0 += dpp_move_d<0xB1>(a0);                         // quad_perm [1, 0, 3, 2], then [2, 3, 0, 1]: the four lanes
            a0 += dpp_move_d<0x4E>(a0);                         // hold the whole dot product
            sc = h4 == u ? a0 : sc;
            __builtin_amdgcn_sched_barrier(0);                  // (the conversions of one row at a time: all of them would not fit)
          }
          const double pj = 64 * wave + 16 * h4 + kl < T ? exp(sc * rs - mref) : 0.0;
          den += pj;
          num = fma(pj, (double)v, num);
        }
        den = wave_sum_dpp(den);
        num = wave_sum_dpp(num);
        if (lane == 0) {
          parts[(fi * NW + wave) * 2] = den;
          parts[(fi * NW + wave) * 2 + 1] = num;
        }
      }
    } else {
      for (int fi = 0; fi < nb; ++fi) {
        const int qloc = fix_ent[2 * (base + fi)], feat = fix_ent[2 * (base + fi) + 1];
        const float *qr = qbase + (size_t)(q_first + qloc) * hd;
        const float *vrow = vbase + (size_t)feat * Tp;            // V^T row of the feature, keys in vt_pos order
        v4f kv[4][NEB];
        float va;
        auto load_row = [&](int key, v4f (&dst)[NEB]) {
          const float *r = kbase + (size_t)min(key, T - 1) * hd;
#pragma unroll
          for (int c = 0; c < NEB; ++c) dst[c] = *(const v4f *)(r + min(16 * c + 4 * h4, hd - 4));
        };
        int k0 = 64 * wave;
#pragma unroll
        for (int u = 0; u < 4; ++u) load_row(k0 + 16 * u + kl, kv[u]);
        va = vrow[vt_pos(min(k0 + 16 * h4 + kl, Tp - 1))];
        double qd[NEB][4];
#pragma unroll
        for (int c = 0; c < NEB; ++c) {
          const int f = 16 * c + 4 * h4;
          const v4f t4 = *(const v4f *)(qr + min(f, hd - 4));
#pragma unroll
          for (int e = 0; e < 4; ++e) qd[c][e] = f < hd ? (double)t4[e] : 0.0;
        }
        const double mref = (double)m_s[qloc] * 0.6931471805599453;       // base 2 -> natural
        double den = 0.0, num = 0.0;
        for (; k0 < T; k0 += 64 * NW) {
          const float v = va;
          double sc = 0.0;
#pragma unroll
          for (int u = 0; u < 4; ++u) {
            double a0 = 0.0, a1 = 0.0;
#pragma unroll
            for (int c = 0; c < NEB; ++c) {
              a0 = fma(qd[c][0], (double)kv[u][c][0], a0);
              a1 = fma(qd[c][1], (double)kv[u][c][1], a1);
              a0 = fma(qd[c][2], (double)kv[u][c][2], a0);
              a1 = fma(qd[c][3], (double)kv[u][c][3], a1);
            }
            load_row(k0 + 64 * NW + 16 * u + kl, kv[u]);          // beyond T: the last row again, never used
            a0 += a1;
            a0 += dpp_move_d<0xB1>(a0);                           // quad_perm [1, 0, 3, 2], then [2, 3, 0, 1]: the four lanes
            a0 += dpp_move_d<0x4E>(a0);                           // hold the whole dot product
            sc = h4 == u ? a0 : sc;
          }
          va = vrow[vt_pos(min(k0 + 64 * NW + 16 * h4 + kl, Tp - 1))];
          const double pj = k0 + 16 * h4 + kl < T ? exp(sc * rs - mref) : 0.0;
          den += pj;
          num = fma(pj, (double)v, num);
        }
        den = wave_sum_dpp(den);
        num = wave_sum_dpp(num);
        if (lane == 0) {
          parts[(fi * NW + wave) * 2] = den;
          parts[(fi * NW + wave) * 2 + 1] = num;
        }
      }
    }
    __syncthreads();
    if (tid < nb) {
      double den = 0.0, num = 0.0;
#pragma unroll
      for (int w = 0; w < NW; ++w) {
        den += parts[(tid * NW + w) * 2];
        num += parts[(tid * NW + w) * 2 + 1];
      }
      const float ov = (float)(num / den);
      stage[fix_ent[2 * (base + tid)] * SRB + fix_ent[2 * (base + tid) + 1]] =
          (unsigned char)(int)fminf(fmaxf(rintf(ov / qs) + qz, -128.f), 127.f);
    }
    __syncthreads();
  }
  // rows out: hd bytes per query (a multiple of 4), contiguous in the output row of the token.  The lanes go by the 32-bit words of all
  // rows, and every word is read before the first is stored (one after the other, each waited for LDS: 2400 clocks a workgroup)
  const int wpr = hd >> 2;                        // words per row (at most 4 NEB)
  const float inv_wpr = __builtin_amdgcn_rcpf((float)wpr);
  constexpr int NO = (NQ * 4 * NEB + 64 * NW - 1) / (64 * NW);
  unsigned word[NO];
  unsigned at[NO];
  const int n_out = min(NQ, T - q_first) * wpr;
#pragma unroll
  for (int k = 0; k < NO; ++k) {
    const int i = min(tid + 64 * NW * k, NQ * wpr - 1), r = (int)(((float)i + 0.5f) * inv_wpr), wd = i - r * wpr;      // i / wpr, exactly
    word[k] = *(const unsigned *)(stage + r * SRB + 4 * wd);
    at[k] = (unsigned)((q_first + r) * D + 4 * wd);
  }
#pragma unroll
  for (int k = 0; k < NO; ++k)
    if (tid + 64 * NW * k < n_out) *(unsigned *)(q_out + at[k]) = word[k];
}

// NCH feature chunks of 32 (operand width), NEB feature blocks of 16 that hold real features, QB query blocks of 16 per
// wavefront (a workgroup covers 64 * QB queries).  QB = 2 reads every K / V^T fragment once for two MFMAs; QB = 1 makes
// twice as many workgroups with half the MFMA chain each, for launches that would leave compute units idle.  The
// arithmetic per query is the same in both.
//
// TAIL: the last feature chunk holds at most 8 real features (d = 72: 64 + 8).  Its three products then share ONE
// instruction: of the 32 k positions of the K operand, 0..7 are the features' hi halves, 8..15 their lo halves, 16..23 (and 24..31)
// the hi halves again, and the query operand has hi, hi, lo (and zeros) there (7 instructions per key block instead of 9 at d = 72).
// The last block of V^T then has at most 8 real features as well, and its other 8 rows hold their lo halves: one fragment, two
// products instead of three (the lo x lo terms come with them), and one addition across lanes at the end.
// (16 heads of 72, 16 x 1024 tokens: 301.6 -> 298 us, and 0.1 - 1 % closer to float64 in the mean.)
//
// What bounds the key loop: vector issue.  Per tile of 64 keys a wavefront (QB = 2, d = 72) issues 112 MFMAs and about 300 other vector
// instructions, 32 of them exponentials.  On this chip an MFMA 16x16x32 takes 18 clocks of the matrix pipe and keeps the SIMD, for
// whichever of its wavefronts, from issuing for 10 of them (two FMAs behind each cost nothing, every further one 4 clocks), so the
// two kinds add up to 5000 of the 6170 clocks that a tile of both resident wavefronts takes.  Cycle counters, 8 x 1024 tokens, 16
// heads of 72, clocks a wavefront: first loads and first tile 9900; 16 tiles of 6170 (scores and staging 2690, softmax 1300, V^T products 1130,
// barrier and loads 1050); codes 4000; decisions and rows out 12 600: 125 000, twice a slot, of the launch's 290 000 - 340 000, in
// which 1.5 of a SIMD's two slots are taken in the mean: the rest is the last round, which waits for the workgroups with most decisions.  64 x 256
// tokens: 8300; 4 tiles of 5580; 3500; 3200.  With one tile in LDS, staged between two barriers, a tile took 6830: 64 x 256 tokens 92.8 -> 90.3 us,
// 8 x 1024 158 -> 154, 10 x 425 59.5 -> 56.2 (LDS active in 33 % of the cycles -> 28 %, conflicts in 13 % -> 8 %).  Units of K and V^T are dealt to
// threads such that their places are constants away from a few registers: the tables of places that stood here would not fit beside a tile in flight,
// and a single register in scratch memory costs more than the second tile gains.
// Not better: 32x32x16 products (half the issue slots, the same clocks a tile, and the chip, at its power limit, runs them 4 % slower),
// eight wavefronts on one tile (half the staging, 3 - 10 % slower), one branch for all outputs of a query.
// Vector work is what was cut before: the
// running max is only raised when a tile exceeds it by more than MAX_SLACK (a probability may reach 2^MAX_SLACK; hi + lo keep
// their relative precision), which leaves one test per tile instead of two shuffles, an exponential and the rescaling of every
// output register.
// The sum of the probabilities stays a float32 addition each: a row of ones in V^T gives it for free (2 - 4 % of a launch), but
// from the 22 bits of the halves and with the matrix cores' accumulation, 1.2 (256 keys) to 1.6 (4096) times as far from
// float64, and the outputs of a sharp softmax over 4096 keys 1.5 times.
template <int NCH, int NEB, int QB, bool TAIL, bool ONE>
__global__ __launch_bounds__(256, 2) void attention_f16_kernel(const float *__restrict__ Qp, const float *__restrict__ Kp,
                                                            const float *__restrict__ Vt, int BH, int T, int Tp, int H, int hd, int DPv,
                                                            float q_mul, const QParam *qp, int8_t *__restrict__ q_out) {
  constexpr int NM = TAIL ? NCH - 1 : NCH;        // feature chunks multiplied in three instructions
  constexpr int NI = NM + (TAIL ? 1 : 0);         // fragment steps per key block
  constexpr int NW = 4, NT = 64 * NW;             // wavefronts, threads
  constexpr int KCH = NEB;                        // 16-byte units of K per thread per tile: units p, p + 4, ... of row r (below)
  constexpr int VCH = (NEB + 1) / 2;              // 32-byte units of V^T: unit c of rows f, f + 32, ...
  constexpr int NQ = 16 * QB * NW;                // queries of this workgroup
  constexpr float MAX_SLACK = 8.0f;
  // A tile in LDS, in units of 16 bytes without padding, whose places are swapped so that 16 rows of one unit lie in 16 different
  // places of 256 bytes (free of conflicts when they are read).  K: one plane of 64 rows x 32 features per feature chunk, hi then
  // lo; the packed tail has 8 hi and 8 lo halves a row.  V^T: rows of 64 keys, hi then lo; the last block of TAIL holds both.
  constexpr int KPL = 64 * 32, KTL = TAIL ? 64 * 16 : 0;  // halves of a plane and of the tail
  constexpr int KSZ = 2 * NM * KPL + KTL, VSZ = 64 * (16 * NEB + 16 * (TAIL ? NEB - 1 : NEB));
  // Two tiles where two workgroups a compute unit have room for them (160 KB): not for 76 and 80 features, whose tiles take 45 KB.
  // Nor with one query block a wavefront, whose tile is multiplied in half the time: by itself 4 x 256 tokens 13.0 us with two tiles, 12.5 with one,
  // 8 x 256 17.5 | 16.9, 1 x 1024 42.1 | 40.9, and beside the other half's kernels, which need LDS too, more: 28 blocks of width 1152, 50 steps
  // of 8 x 256 tokens (two halves of 4) 78.6 ms | 76.7; 12 blocks, 4 steps: width 384, 40 x 256 tokens 2.90 | 2.80, width 768, 20 x 256 3.43 |
  // 3.37, width 1152, 4 x 1024 5.82 | 5.74, 6 x 425 3.78 | 3.75, 16 x 256 4.20 | 4.18; 6 x 256 equal.
  // Nor for heads of up to 32 features: their kernels fit three or four wavefronts a SIMD, with a tile in flight beside the loop one less.
  // A block's attention, two | one, us: 24 heads of 16, 32 x 1024 tokens 277 | 266, 64 x 256 50.2 | 46.0, 12 of 32, 32 x 1024 204 | 189,
  // 8 x 1024 69 | 62, 36 of 32, 16 x 1024 307 | 280, 24 of 20, 8 x 1024 91 | 86.  (A tile, of one buffer, stored behind the V^T products takes as
  // many registers: the compiler moves the conversions among them.)
  constexpr int NBUF = NCH > 1 && QB == 2 && 4 * (KSZ + VSZ) <= 78 * 1024 ? 2 : 1;
  __shared__ __align__(16) _Float16 kv_s[NBUF][KSZ + VSZ];
  __shared__ int fix_cnt_s;                       // outputs queued for the exact decision (epilogue)
  __shared__ float m_s[NQ];                       // running max of every query (reference point of the exact decision)

  const int D = H * hd;
  if (threadIdx.x == 0) fix_cnt_s = 0;            // published by the barriers of the key loop
  // Workgroups go round-robin over the 8 XCDs.  Workgroup id -> XCD id % 8, position id / 8 on that XCD; the query
  // blocks of one (batch, head) take consecutive positions of one XCD, so they run at the same time and the head's K
  // and V are fetched from HBM once, into that XCD's L2.
  const int n_qblk = gridDim.y;                   // query blocks per head (the grid is 1-D in effect: x * y workgroups)
  const int wg = blockIdx.y * gridDim.x + blockIdx.x;
  const int pos = wg >> 3, qblk = pos % n_qblk;
  const int bh = (pos / n_qblk) * 8 + (wg & 7);
  if (bh >= BH) return;                           // the grid is rounded up to whole groups of 8 heads
  const int b = bh / H, h = bh % H;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int ql = lane & 15, g = lane >> 4;
  const long long tok_base = (long long)bh * T * hd;
  const long long vt_base = (long long)bh * DPv * Tp;
  // what no tile writes, where a head has padding: the padded features of the K rows and the V^T rows beyond d (zeros)
  if (hd != 32 * NM + (TAIL ? 8 : 0) || hd != 16 * NEB - (TAIL ? 8 : 0)) {
    for (int i = tid; i < (int)(sizeof(kv_s) / 16); i += NT) ((v8h *)kv_s)[i] = (v8h){0, 0, 0, 0, 0, 0, 0, 0};
    __syncthreads();
  }

  // This thread's part of a tile: of K, the 16-byte units kp, kp + 4, ... of row kr; of V^T, the 32-byte unit vc of rows vf, vf + 32, ...
  // Its places in memory and in LDS are then constants away from a few registers.  Loads never branch: a unit or row beyond the
  // head's last reads the last one, a key beyond T key T - 1 (finite values that the ragged-tile mask or the store predicate
  // discards), so that all loads of a tile are issued back to back and nothing waits in between.
  const int hd4 = hd >> 2, kr = tid >> 2, kp = tid & 3, vf = tid >> 3, vc = tid & 7;
  const float *const kbase = Kp + tok_base, *const vbase = Vt + vt_base;
  const int klast = min(kp + 4 * (KCH - 1), hd4 - 1) * 4 - kp * 4;             // from a thread's first unit to its last, in floats
  const unsigned voff = (unsigned)(vf * Tp + vc * 8), vlast = (unsigned)(min(vf + 32 * (VCH - 1), hd - 1) * Tp + vc * 8);
  const bool k_has = kp + 4 * (KCH - 1) < hd4, v_has = vf + 32 * (VCH - 1) < hd;
  // places in LDS, in halves: K's even and odd units, the tail's hi and lo half, V^T's rows, the lo row of the shared block
  const int ksw = (kr >> 2) & 3, kat0 = kr * 32 + (((kp >> 1) ^ ksw) << 3) + (kp & 1) * 4, kat1 = kat0 ^ 16;
  const int ktl0 = 2 * NM * KPL + kr * 16 + (((kr >> 3) & 1) << 3) + (kp & 1) * 4, ktl1 = ktl0 ^ 8;
  const int vat0 = KSZ + vf * 64 + ((vc ^ ((vf >> 1) & 7)) << 3), vat1 = (vat0 ^ 32) + 8 * 64;
  auto load_tile = [&](int k0, v4f (&kreg)[KCH], v4f (&vreg)[2][VCH]) {
    const float *const kb = kbase + (size_t)k0 * hd, *vb = vbase + k0;
    const unsigned off = (unsigned)(min(kr, T - 1 - k0) * hd + kp * 4);
#pragma unroll
    for (int u = 0; u < KCH - 1; ++u) kreg[u] = *(const v4f *)(kb + off + 16 * u);
    kreg[KCH - 1] = *(const v4f *)(kb + (unsigned)(off + klast));
#pragma unroll
    for (int u = 0; u < VCH; ++u) {
      const float *const src = u < VCH - 1 ? vb + (size_t)(32 * u) * Tp + voff : vb + vlast;
      vreg[0][u] = *(const v4f *)src;
      vreg[1][u] = *(const v4f *)(src + 4);
    }
  };
  // unit u of a tile (K's, then V^T's) from registers to LDS
  auto store_unit = [&](int u, _Float16 *dst, const v4f (&kreg)[KCH], const v4f (&vreg)[2][VCH]) {
    if (u < KCH) {
      if (u < KCH - 1 || k_has) {
        v2u hi, lo;
        split_pairs(kreg[u], hi, lo);
        if (TAIL && u == KCH - 1) {
          *(v2u *)(dst + ktl0) = hi;
          *(v2u *)(dst + ktl1) = lo;
        } else {
          _Float16 *const at = dst + (u & 1 ? kat1 : kat0) + (u >> 1) * KPL;
          *(v2u *)at = hi;
          *(v2u *)(at + NM * KPL) = lo;
        }
      }
    } else {
      const int w = u - KCH;
      if (w < VCH - 1 || v_has) {
        v2u h0, l0, h1, l1;
        split_pairs(vreg[0][w], h0, l0);
        split_pairs(vreg[1][w], h1, l1);
        _Float16 *const at = dst + vat0 + w * 32 * 64;
        *(v4u *)at = (v4u){h0.x, h0.y, h1.x, h1.y};
        *(v4u *)(TAIL && w == VCH - 1 ? dst + vat1 + w * 32 * 64 : at + NEB * 16 * 64) = (v4u){l0.x, l0.y, l1.x, l1.y};
      }
    }
  };
  const auto lds_barrier = [] {                   // (loads from memory stay in flight)
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
  };

  v4f kreg[KCH], vreg[2][VCH];
  int q_row[QB];
  v8h qh[QB][NI], qlo[QB][NM > 0 ? NM : 1];       // with TAIL, qh[.][NM] is the packed tail operand
  {
    // the queries are in flight together with the first two key tiles, or the first one where LDS holds one
    v4f kfirst[KCH], vfirst[2][VCH];
    if constexpr (NBUF == 2) load_tile(0, kfirst, vfirst);
    else load_tile(0, kreg, vreg);
    // all query loads are issued before any is used; rows beyond T read row T-1 (their results are never
    // stored), features beyond d read the last chunk and are zeroed below
    v4f qraw[QB][NCH][2];
#pragma unroll
    for (int j = 0; j < QB; ++j) {
      q_row[j] = qblk * NQ + wave * (16 * QB) + j * 16 + ql;
      const float *src = Qp + tok_base + (long long)min(q_row[j], T - 1) * hd;
#pragma unroll
      for (int c = 0; c < NCH; ++c) {
        const int f = 32 * c + (c < NM ? 8 * g : 0);
        qraw[j][c][0] = *(const v4f *)(src + min(f, hd - 4));
        qraw[j][c][1] = *(const v4f *)(src + min(f + 4, hd - 4));
      }
    }
    if constexpr (NBUF == 2) {
      if (64 < T) load_tile(64, kreg, vreg);
#pragma unroll
      for (int u = 0; u < KCH + VCH; ++u) store_unit(u, kv_s[0], kfirst, vfirst);
    }
#pragma unroll
    for (int j = 0; j < QB; ++j)
#pragma unroll
      for (int c = 0; c < NCH; ++c) {
        const int f = 32 * c + (c < NM ? 8 * g : 0);
        v2u h0, l0, h1, l1;
        split_pairs(qraw[j][c][0] * q_mul, h0, l0);     // queries pre-scaled by log2(e) / sqrt(d): the softmax runs in base 2
        split_pairs(qraw[j][c][1] * q_mul, h1, l1);
        if (f >= hd) { h0 = (v2u){0, 0}; l0 = h0; }
        if (f + 4 >= hd) { h1 = (v2u){0, 0}; l1 = h1; }
        v4u hh = {h0.x, h0.y, h1.x, h1.y}, ll = {l0.x, l0.y, l1.x, l1.y};
        if (c < NM) {
          qh[j][c] = *(v8h *)&hh;
          qlo[j][c] = *(v8h *)&ll;
        } else {                                        // lane group g supplies k positions 8 g .. 8 g + 7
          v4u t = g == 2 ? ll : hh;
          if (g == 3) t = (v4u){0, 0, 0, 0};
          qh[j][c] = *(v8h *)&t;
        }
      }
  }
  v4f o[QB][NEB];
#pragma unroll
  for (int j = 0; j < QB; ++j)
#pragma unroll
    for (int e = 0; e < NEB; ++e) o[j][e] = (v4f){0.f, 0.f, 0.f, 0.f};
  float m_run[QB], l_run[QB];
#pragma unroll
  for (int j = 0; j < QB; ++j) {
    m_run[j] = -INFINITY;
    l_run[j] = 0.0f;
  }
  // this lane's fragments: row ql of a block, unit g of a K plane, units g and 4 + g of a V^T row; of the tail, the lane groups take
  // hi, lo, hi (and hi again, against zeros)
  const int kat = ql * 32 + ((g ^ (ql >> 2)) << 3), tat = ql * 16 + (((g == 1 ? 1 : 0) ^ (ql >> 3)) << 3);
  const int vat[2] = {ql * 64 + ((g ^ (ql >> 1)) << 3), ql * 64 + (((4 + g) ^ (ql >> 1)) << 3)};
  lds_barrier();          // (one tile: nothing to publish yet, but a run of 8 x 256 tokens takes 76.7 ms with it, 76.9 without)

  for (int k0 = 0; k0 < T; k0 += 64) {
    const bool more = k0 + 64 < T;
    if constexpr (NBUF == 1) {
      // at the head of the loop, not behind the V^T products (runs of width 768, 20 x 256 tokens, 3.40 ms there, 3.37 here; width 384, 40 x 256
      // 2.84 | 2.80)
      if (k0) lds_barrier();                      // everyone is done with the tile before
#pragma unroll
      for (int u = 0; u < KCH + VCH; ++u) store_unit(u, kv_s[0], kreg, vreg);
      if (more) load_tile(k0 + 64, kreg, vreg);
      lds_barrier();
    }
    const _Float16 *const cur = kv_s[NBUF == 2 ? (k0 >> 6) & 1 : 0], *const curv = cur + KSZ;
    _Float16 *const nxt = kv_s[NBUF == 2 ? ((k0 >> 6) & 1) ^ 1 : 0];        // (two tiles)

    // S^T = K Q^T: the K fragments run two iterations ahead of the MFMAs that use them (LDS latency is
    // several MFMA groups long and a wavefront is alone on its SIMD).  The next tile goes to the other buffer behind the products
    v4f s[QB][4];
    auto scores = [&](auto stage_next) {
      constexpr int NS = 4 * NI, NU = KCH + VCH;
      v8h kfh[3], kfl[3];
      auto load_k = [&](int it, int slot) {
        const int kt = it / NI, c = it % NI;
        if (c < NM) {
          kfh[slot] = *(const v8h *)(cur + c * KPL + kt * 16 * 32 + kat);
          kfl[slot] = *(const v8h *)(cur + (NM + c) * KPL + kt * 16 * 32 + kat);
        } else {
          kfh[slot] = *(const v8h *)(cur + 2 * NM * KPL + kt * 16 * 16 + tat);
        }
      };
      load_k(0, 0);
      load_k(1, 1);
      v4f acc[QB];
#pragma unroll
      for (int it = 0; it < NS; ++it) {
        const int kt = it / NI, c = it % NI, slot = it % 3;
        if (it + 2 < NS) load_k(it + 2, (it + 2) % 3);
        __builtin_amdgcn_sched_barrier(0);
        const v8h kh = kfh[slot], kl = kfl[slot];
        if (c == 0) {
#pragma unroll
          for (int j = 0; j < QB; ++j) acc[j] = (v4f){0.f, 0.f, 0.f, 0.f};
        }
        // the query blocks alternate so that consecutive MFMAs do not wait on each other's result
        if (c < NM) {
#pragma unroll
          for (int j = 0; j < QB; ++j) acc[j] = __builtin_amdgcn_mfma_f32_16x16x32_f16(kl, qh[j][c], acc[j], 0, 0, 0);
#pragma unroll
          for (int j = 0; j < QB; ++j) acc[j] = __builtin_amdgcn_mfma_f32_16x16x32_f16(kh, qlo[j][c < NM ? c : 0], acc[j], 0, 0, 0);
        }
#pragma unroll
        for (int j = 0; j < QB; ++j) acc[j] = __builtin_amdgcn_mfma_f32_16x16x32_f16(kh, qh[j][c], acc[j], 0, 0, 0);
        if constexpr (decltype(stage_next)::value) {
#pragma unroll
          for (int u = NU * it / NS; u < NU * (it + 1) / NS; ++u) store_unit(u, nxt, kreg, vreg);
        }
        __builtin_amdgcn_sched_barrier(0);
        if (c == NI - 1) {
#pragma unroll
          for (int j = 0; j < QB; ++j) s[j][kt] = acc[j];
        }
      }
    };
    if (NBUF == 2 && more) scores(std::true_type{});
    else scores(std::false_type{});
    if (NBUF == 2 && k0 + 128 < T) load_tile(k0 + 128, kreg, vreg);       // in flight until the next tile's products
    // the first V^T fragments are requested before the softmax arithmetic, which hides their latency
    constexpr int NP = 2 * NEB;
    v8h vfh[3], vfl[3];
    auto load_v = [&](int it, int slot) {
      const int a = it / NEB, e = it % NEB;
      vfh[slot] = *(const v8h *)(curv + e * 16 * 64 + vat[a]);
      if (!TAIL || e < NEB - 1) vfl[slot] = *(const v8h *)(curv + (NEB + e) * 16 * 64 + vat[a]);
    };
    load_v(0, 0);
    load_v(1, 1);
    v8h ph[QB][2], pl[QB][2];
    if (k0 + 64 > T) {                      // wavefront-uniform: whole tiles skip the masking
      asm volatile("");                     // (kept a branch: as selects it would cost every tile three instructions a key)
#pragma unroll
      for (int j = 0; j < QB; ++j)
#pragma unroll
        for (int kt = 0; kt < 4; ++kt)
#pragma unroll
          for (int r = 0; r < 4; ++r)
            if (k0 + kt * 16 + 4 * g + r >= T) s[j][kt][r] = -INFINITY;
    }
    float mx[QB];
    bool over = false;
#pragma unroll
    for (int j = 0; j < QB; ++j) {
      mx[j] = s[j][0][0];
#pragma unroll
      for (int kt = 0; kt < 4; ++kt)
#pragma unroll
        for (int r = 0; r < 4; ++r) mx[j] = fmaxf(mx[j], s[j][kt][r]);
      over = over || mx[j] > m_run[j] + MAX_SLACK;      // true on the first tile: m_run starts at minus infinity
    }
    if (__builtin_amdgcn_ballot_w64(over) != 0ull) {
      // raise the running max of every query of the wavefront to its true value so far and rescale what was summed
#pragma unroll
      for (int j = 0; j < QB; ++j) {
        mx[j] = fmaxf(mx[j], __shfl_xor(mx[j], 16, 64));
        mx[j] = fmaxf(mx[j], __shfl_xor(mx[j], 32, 64));
        const float m_new = fmaxf(m_run[j], mx[j]);
        const float alpha = __builtin_amdgcn_exp2f(m_run[j] - m_new);
        m_run[j] = m_new;
        l_run[j] *= alpha;
#pragma unroll
        for (int e = 0; e < NEB; ++e) o[j][e] *= alpha;
      }
    }
#pragma unroll
    for (int j = 0; j < QB; ++j) {
#pragma unroll
      for (int a = 0; a < 2; ++a) {
        v4u hw, lw;
#pragma unroll
        for (int w = 0; w < 4; ++w) {         // word w of the operand: keys (kt = 2 a + w / 2, r = 2 (w % 2) .. + 1)
          const int kt = 2 * a + (w >> 1), r = 2 * (w & 1);
          const float p0 = __builtin_amdgcn_exp2f(s[j][kt][r] - m_run[j]), p1 = __builtin_amdgcn_exp2f(s[j][kt][r + 1] - m_run[j]);
          l_run[j] += p0;
          l_run[j] += p1;
          unsigned h2, l2;
          split_pair(p0, p1, h2, l2);
          hw[w] = h2;
          lw[w] = l2;
        }
        ph[j][a] = __builtin_bit_cast(v8h, hw);
        pl[j][a] = __builtin_bit_cast(v8h, lw);
      }
    }
#pragma unroll
    for (int it = 0; it < NP; ++it) {
      const int a = it / NEB, e = it % NEB, slot = it % 3;
      if (it + 2 < NP) load_v(it + 2, (it + 2) % 3);
      __builtin_amdgcn_sched_barrier(0);
      const v8h vh = vfh[slot], vl = vfl[slot];
      if (!TAIL || e < NEB - 1) {
#pragma unroll
        for (int j = 0; j < QB; ++j) o[j][e] = __builtin_amdgcn_mfma_f32_16x16x32_f16(vl, ph[j][a], o[j][e], 0, 0, 0);
      }
#pragma unroll
      for (int j = 0; j < QB; ++j) o[j][e] = __builtin_amdgcn_mfma_f32_16x16x32_f16(vh, pl[j][a], o[j][e], 0, 0, 0);
#pragma unroll
      for (int j = 0; j < QB; ++j) o[j][e] = __builtin_amdgcn_mfma_f32_16x16x32_f16(vh, ph[j][a], o[j][e], 0, 0, 0);
      __builtin_amdgcn_sched_barrier(0);
    }
    if (NBUF == 2 && more) lds_barrier();
  }
  if constexpr (TAIL) {                           // the lo halves' rows to those of their features: 8 rows = 2 lane groups further
#pragma unroll
    for (int j = 0; j < QB; ++j)
#pragma unroll
      for (int r = 0; r < 4; ++r) o[j][NEB - 1][r] += __shfl_xor(o[j][NEB - 1][r], 32, 64);
  }

  // ---- epilogue.  The codes of the workgroup's queries are staged in LDS (the K tiles are no longer needed), the ones
  // whose value lies too close to a rounding boundary of Eq. 1 for the arithmetic above (fp16 pairs, fp32 sums and
  // exponentials) to be trusted are decided again in float64 from the float32 Q | K | V, then the rows go out.
  const QParam t = *qp;
  const float qs = t.s, qz = (float)t.z;
  constexpr int SRB = 16 * NEB;                   // staged row: the head's features, padded
  static_assert(NQ * SRB + FIX_CAP * 8 <= 2 * KSZ, "the epilogue's staging area must fit in the K tile");
  unsigned char *stage = (unsigned char *)kv_s;
  int *fix_cnt = &fix_cnt_s;
  int *fix_ent = (int *)(stage + NQ * SRB);       // [FIX_CAP][2]: query within the workgroup, feature
  __syncthreads();                                // every wavefront is past its last K / V^T fragment
  // |v / s - rint(v / s)| within tol of 1/2: 1.2e-5 steps + 4e-7 of the code's size at 256 keys.  Against float64 on the Q | K | V of
  // a DiT-XL/2 block (weights of standard deviation 0.02) the fast path is off by 3.9e-6 / 7.3e-6 / 1.4e-5 steps in the mean at
  // 256 / 1024 / 4096 keys and by at most 1.02 / 0.59 / 0.34 of the window.  The window is no bound: an error beyond it turns a
  // code only where the value lies between the two, and with weights of 0.05, whose scores are six times as large, the
  // largest error at 256 keys was 7.6 windows (mean 0.3) and still no code of a million differed.
  // The quotient of Eq. 1 is formed as v * (1 / s) here: that is within 2.5e-7 |v / s| of the correctly rounded
  // quotient, so the two can only round to different integers inside the window below (whose relative part is widened
  // by that much), where the float64 path, which divides, decides.
  const float tol_k = fmaxf(1.0f, (float)T * (1.0f / 256.0f));      // the sums grow with the number of keys and the bound with them
  const float tol_0 = 1.2e-5f * tol_k, tol_q = 4e-7f * tol_k + 2.5e-7f;
  const float doubt_at = 0.5f - tol_0;
  const float inv_qs = 1.0f / qs, zu = qz + 128.0f;
#pragma unroll
  for (int j = 0; j < QB; ++j) {
    float l = l_run[j];
    l += __shfl_xor(l, 16, 64);
    l += __shfl_xor(l, 32, 64);
    const float k = (1.0f / l) * inv_qs;            // value and quotient of Eq. 1 in one multiplication per output
    const int qloc = wave * (16 * QB) + j * 16 + ql;
    if (g == 0) m_s[qloc] = m_run[j];
#pragma unroll
    for (int e = 0; e < NEB; ++e) {
      const int f = 16 * e + 4 * g;
      unsigned w = 0;
      float dist[4];                                // distance from the rounding boundary plus the window's relative part
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const float qv = o[j][e][r] * k, rr = __builtin_rintf(qv);
        w = __builtin_amdgcn_cvt_pk_u8_f32(__builtin_amdgcn_fmed3f(rr + zu, 0.0f, 255.0f), r, w);
        dist[r] = fmaf(tol_q, fabsf(qv), fabsf(qv - rr));
      }
      // one comparison and one branch per four outputs
      if (fmaxf(fmaxf(dist[0], dist[1]), fmaxf(dist[2], dist[3])) > doubt_at) {
#pragma unroll
        for (int r = 0; r < 4; ++r)
          if (dist[r] > doubt_at && q_row[j] < T && f + r < hd) {
            const int slot = atomicAdd(fix_cnt, 1);
            if (slot < FIX_CAP) {
              fix_ent[2 * slot] = qloc;
              fix_ent[2 * slot + 1] = f + r;
            }
          }
      }
      *(unsigned *)(stage + qloc * SRB + f) = w ^ 0x80808080u;
    }
  }
  __syncthreads();
  constexpr int FB = 2 * VSZ / (NW * 16) < 64 ? 2 * VSZ / (NW * 16) : 64;       // outputs per batch of parts in LDS
  decide_again_and_store<NEB, NQ, NW, FB, ONE>(stage, &fix_cnt_s, fix_ent, (double *)(kv_s[0] + KSZ), m_s, Qp + tok_base, kbase, vbase, qblk * NQ, T,
                                          Tp, hd, D, qs, qz, q_out + (size_t)b * T * D + (size_t)h * hd);
}

// The same attention for launches that would leave the chip idle: one workgroup = 16 QB queries of one (batch, head), its four
// wavefronts share the KEYS (wavefront w takes the tiles w, w + 4, ... of 64), so the chain of key tiles a query waits for is a
// quarter as long and there are four times as many workgroups.  No K or V^T fragment is used by two wavefronts, so none
// goes through LDS: each lane loads its fragments from memory in operand layout (32 bytes at a time) and splits them in
// registers, all of a tile's loads in flight together, the next tile's K requested as soon as the scores are formed.  (Loads of
// whole lines turned through LDS: 11.7 against 9.3 us at 1 x 256 tokens.)  Every workgroup splits its head's whole K and V, so the
// kernel is for launches that fit the chip at once; what is left is memory latency, about 1100 vector instructions a wavefront
// and the exact decisions (2 us).  The running sums meet in LDS at the end: with M the largest running max of a query, each wavefront's sums are scaled by
// 2^(m - M) in float32, the arithmetic of the rescaling in the key loop.
template <int NCH, int NEB, int QB, bool TAIL, bool ONE>
__global__ __launch_bounds__(256, 1) void attention_f16_keys_kernel(const float *__restrict__ Qp, const float *__restrict__ Kp,
                                                                    const float *__restrict__ Vt, int BH, int T, int Tp, int H, int hd,
                                                                    int DPv, float q_mul, const QParam *qp, int8_t *__restrict__ q_out) {
  constexpr int NM = TAIL ? NCH - 1 : NCH;        // feature chunks multiplied in three instructions
  constexpr int NI = NM + (TAIL ? 1 : 0);
  constexpr int NW = 4, NT = 64 * NW, NQ = 16 * QB;
  constexpr int SRB = 16 * NEB;                   // staged row: the head's features, padded
  constexpr int FB = 64;                          // doubtful outputs per batch of parts in LDS
  constexpr float MAX_SLACK = 8.0f;
  // sums of the wavefronts, [wavefront][query block, feature block][lane]; later the parts of the exact decisions
  __shared__ __align__(16) v4f osum[NW * QB * NEB * 64];
  __shared__ float msum[NW][NQ], lsum[NW][NQ], m_s[NQ];
  __shared__ __align__(16) unsigned char stage[NQ * SRB];
  __shared__ int fix_ent[2 * FIX_CAP], fix_cnt_s;
  static_assert(FB * NW * 16 <= (int)sizeof(osum), "the parts of the exact decisions must fit in the sums' area");

  const int D = H * hd;
  if (threadIdx.x == 0) fix_cnt_s = 0;            // published by the barrier behind the sums
  // query blocks of one (batch, head) on one XCD, as above
  const int n_qblk = gridDim.y;
  const int wg = blockIdx.y * gridDim.x + blockIdx.x;
  const int pos = wg >> 3, qblk = pos % n_qblk;
  const int bh = (pos / n_qblk) * 8 + (wg & 7);
  if (bh >= BH) return;                           // the grid is rounded up to whole groups of 8 heads
  const int b = bh / H, h = bh % H;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int ql = lane & 15, g = lane >> 4;
  const float *const qbase = Qp + (long long)bh * T * hd, *const kbase = Kp + (long long)bh * T * hd;
  const float *const vbase = Vt + (long long)bh * DPv * Tp;

  // K fragment (key block kt, chunk c): features 32 c + 8 g .. + 7 of key 16 kt + ql; in the packed tail every lane group
  // needs the last eight features (hi, lo, hi, unused).  Keys beyond T read key T - 1 (masked below), features beyond d the last
  // chunk (their query operand is zero).
  v4f kraw[4][NCH][2], vraw[2][NEB][2];
  unsigned foff[NCH][2];                          // features of the fragment's halves
#pragma unroll
  for (int c = 0; c < NCH; ++c) {
    const int f = 32 * c + (c < NM ? 8 * g : 0);
    foff[c][0] = (unsigned)min(f, hd - 4);
    foff[c][1] = (unsigned)min(f + 4, hd - 4);
  }
  auto load_k = [&](int k0) {
#pragma unroll
    for (int kt = 0; kt < 4; ++kt) {
      const unsigned row = (unsigned)(min(k0 + 16 * kt + ql, T - 1) * hd);
#pragma unroll
      for (int c = 0; c < NCH; ++c)
#pragma unroll
        for (int i = 0; i < 2; ++i) kraw[kt][c][i] = *(const v4f *)(kbase + (row + foff[c][i]));
    }
  };
  // V^T fragment (32 keys a, feature block e): keys 8 g .. + 7 (in stored order) of row 16 e + ql; the rows and keys of the
  // padding are zeros in memory
  auto load_v = [&](int k0) {
#pragma unroll
    for (int e = 0; e < NEB; ++e) {
      const unsigned at = (unsigned)((16 * e + ql) * Tp + k0 + 8 * g);
#pragma unroll
      for (int a = 0; a < 2; ++a)
#pragma unroll
        for (int i = 0; i < 2; ++i) vraw[a][e][i] = *(const v4f *)(vbase + (at + 32 * a + 4 * i));
    }
  };

  const int k_first = 64 * wave;                  // wavefronts beyond the last tile load a valid one and use nothing of it
  load_k(min(k_first, Tp - 64));
  int q_row[QB];
  v8h qh[QB][NI], qlo[QB][NM > 0 ? NM : 1];       // with TAIL, qh[.][NM] is the packed tail operand
  {
    v4f qraw[QB][NCH][2];
#pragma unroll
    for (int j = 0; j < QB; ++j) {
      q_row[j] = qblk * NQ + j * 16 + ql;
      const unsigned row = (unsigned)(min(q_row[j], T - 1) * hd);
#pragma unroll
      for (int c = 0; c < NCH; ++c)
#pragma unroll
        for (int i = 0; i < 2; ++i) qraw[j][c][i] = *(const v4f *)(qbase + (row + foff[c][i]));
    }
    load_v(min(k_first, Tp - 64));
#pragma unroll
    for (int j = 0; j < QB; ++j)
#pragma unroll
      for (int c = 0; c < NCH; ++c) {
        const int f = 32 * c + (c < NM ? 8 * g : 0);
        v2u h0, l0, h1, l1;
        split_pairs(qraw[j][c][0] * q_mul, h0, l0);     // queries pre-scaled by log2(e) / sqrt(d): the softmax runs in base 2
        split_pairs(qraw[j][c][1] * q_mul, h1, l1);
        if (f >= hd) { h0 = (v2u){0, 0}; l0 = h0; }
        if (f + 4 >= hd) { h1 = (v2u){0, 0}; l1 = h1; }
        const v4u hh = {h0.x, h0.y, h1.x, h1.y}, ll = {l0.x, l0.y, l1.x, l1.y};
        if (c < NM) {
          qh[j][c] = __builtin_bit_cast(v8h, hh);
          qlo[j][c] = __builtin_bit_cast(v8h, ll);
        } else {                                        // lane group g supplies k positions 8 g .. 8 g + 7: hi, hi, lo, nothing
          v4u t = g == 2 ? ll : hh;
          if (g == 3) t = (v4u){0, 0, 0, 0};
          qh[j][c] = __builtin_bit_cast(v8h, t);
        }
      }
  }
  v4f o[QB][NEB];
  float m_run[QB], l_run[QB];
#pragma unroll
  for (int j = 0; j < QB; ++j) {
    m_run[j] = -INFINITY;
    l_run[j] = 0.0f;
#pragma unroll
    for (int e = 0; e < NEB; ++e) o[j][e] = (v4f){0.f, 0.f, 0.f, 0.f};
  }

  for (int k0 = k_first; k0 < T; k0 += 64 * NW) {
    const int k_next = k0 + 64 * NW;
    v4f s[QB][4];
#pragma unroll
    for (int kt = 0; kt < 4; ++kt) {
#pragma unroll
      for (int j = 0; j < QB; ++j) s[j][kt] = (v4f){0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int c = 0; c < NI; ++c) {
        v8h kh, kl;
        split_operand(kraw[kt][c][0], kraw[kt][c][1], kh, kl);
        if (c < NM) {
#pragma unroll
          for (int j = 0; j < QB; ++j) s[j][kt] = __builtin_amdgcn_mfma_f32_16x16x32_f16(kl, qh[j][c], s[j][kt], 0, 0, 0);
#pragma unroll
          for (int j = 0; j < QB; ++j) s[j][kt] = __builtin_amdgcn_mfma_f32_16x16x32_f16(kh, qlo[j][c < NM ? c : 0], s[j][kt], 0, 0, 0);
#pragma unroll
          for (int j = 0; j < QB; ++j) s[j][kt] = __builtin_amdgcn_mfma_f32_16x16x32_f16(kh, qh[j][c], s[j][kt], 0, 0, 0);
        } else {
          const v8h kt8 = g == 1 ? kl : kh;
#pragma unroll
          for (int j = 0; j < QB; ++j) s[j][kt] = __builtin_amdgcn_mfma_f32_16x16x32_f16(kt8, qh[j][c], s[j][kt], 0, 0, 0);
        }
      }
    }
    if (k_next < T) load_k(k_next);
    if (k0 + 64 > T) {
#pragma unroll
      for (int j = 0; j < QB; ++j)
#pragma unroll
        for (int kt = 0; kt < 4; ++kt)
#pragma unroll
          for (int r = 0; r < 4; ++r)
            if (k0 + kt * 16 + 4 * g + r >= T) s[j][kt][r] = -INFINITY;
    }
    float mx[QB];
    bool over = false;
#pragma unroll
    for (int j = 0; j < QB; ++j) {
      mx[j] = s[j][0][0];
#pragma unroll
      for (int kt = 0; kt < 4; ++kt)
#pragma unroll
        for (int r = 0; r < 4; ++r) mx[j] = fmaxf(mx[j], s[j][kt][r]);
      over = over || mx[j] > m_run[j] + MAX_SLACK;      // true on the first tile: m_run starts at minus infinity
    }
    if (__builtin_amdgcn_ballot_w64(over) != 0ull) {
#pragma unroll
      for (int j = 0; j < QB; ++j) {
        mx[j] = fmaxf(mx[j], __shfl_xor(mx[j], 16, 64));
        mx[j] = fmaxf(mx[j], __shfl_xor(mx[j], 32, 64));
        const float m_new = fmaxf(m_run[j], mx[j]);
        const float alpha = __builtin_amdgcn_exp2f(m_run[j] - m_new);
        m_run[j] = m_new;
        l_run[j] *= alpha;
#pragma unroll
        for (int e = 0; e < NEB; ++e) o[j][e] *= alpha;
      }
    }
    v8h ph[QB][2], pl[QB][2];
#pragma unroll
    for (int j = 0; j < QB; ++j)
#pragma unroll
      for (int a = 0; a < 2; ++a) {
        v4f p[2];
#pragma unroll
        for (int w = 0; w < 4; ++w) {         // word w of the operand: keys (kt = 2 a + w / 2, r = 2 (w % 2) .. + 1)
          const int kt = 2 * a + (w >> 1), r = 2 * (w & 1);
          const float p0 = __builtin_amdgcn_exp2f(s[j][kt][r] - m_run[j]), p1 = __builtin_amdgcn_exp2f(s[j][kt][r + 1] - m_run[j]);
          l_run[j] += p0;
          l_run[j] += p1;
          p[w >> 1][r] = p0;
          p[w >> 1][r + 1] = p1;
        }
        split_operand(p[0], p[1], ph[j][a], pl[j][a]);
      }
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
      for (int e = 0; e < NEB; ++e) {
        v8h vh, vl;
        split_operand(vraw[a][e][0], vraw[a][e][1], vh, vl);
#pragma unroll
        for (int j = 0; j < QB; ++j) o[j][e] = __builtin_amdgcn_mfma_f32_16x16x32_f16(vl, ph[j][a], o[j][e], 0, 0, 0);
#pragma unroll
        for (int j = 0; j < QB; ++j) o[j][e] = __builtin_amdgcn_mfma_f32_16x16x32_f16(vh, pl[j][a], o[j][e], 0, 0, 0);
#pragma unroll
        for (int j = 0; j < QB; ++j) o[j][e] = __builtin_amdgcn_mfma_f32_16x16x32_f16(vh, ph[j][a], o[j][e], 0, 0, 0);
      }
    if (k_next < T) load_v(k_next);
  }

  // the wavefronts' sums meet
#pragma unroll
  for (int j = 0; j < QB; ++j) {
    float l = l_run[j];
    l += __shfl_xor(l, 16, 64);
    l += __shfl_xor(l, 32, 64);
    if (g == 0) {
      msum[wave][16 * j + ql] = m_run[j];
      lsum[wave][16 * j + ql] = l;
    }
#pragma unroll
    for (int e = 0; e < NEB; ++e) osum[((wave * QB + j) * NEB + e) * 64 + lane] = o[j][e];
  }
  __syncthreads();
  const QParam t = *qp;
  const float qs = t.s, qz = (float)t.z;
  // the window of the exact decisions, as in the kernel above
  const float tol_k = fmaxf(1.0f, (float)T * (1.0f / 256.0f));
  const float tol_0 = 1.2e-5f * tol_k, tol_q = 4e-7f * tol_k + 2.5e-7f;
  const float doubt_at = 0.5f - tol_0;
  const float inv_qs = 1.0f / qs, zu = qz + 128.0f;
#pragma unroll
  for (int i0 = 0; i0 < QB * NEB * 64; i0 += NT) {
    const int i = i0 + tid;
    if (i >= QB * NEB * 64) break;                // whole wavefronts
    const int je = i >> 6, j = je / NEB, e = je - j * NEB;
    const int qloc = 16 * j + ql, f = 16 * e + 4 * g;
    float M = msum[0][qloc];                      // finite: wavefront 0 has a tile
#pragma unroll
    for (int w = 1; w < NW; ++w) M = fmaxf(M, msum[w][qloc]);
    float l = 0.0f;
    v4f ov = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int w = 0; w < NW; ++w) {                // a wavefront without a tile: 2^(-inf) = 0 times sums that are zero
      const float a = __builtin_amdgcn_exp2f(msum[w][qloc] - M);
      l += lsum[w][qloc] * a;
      ov += osum[(w * QB * NEB + je) * 64 + lane] * a;
    }
    if (e == 0 && g == 0) m_s[qloc] = M;
    const float k = (1.0f / l) * inv_qs;          // value and quotient of Eq. 1 in one multiplication per output
    unsigned w4 = 0;
    float dist[4];                                // distance from the rounding boundary plus the window's relative part
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const float qv = ov[r] * k, rr = __builtin_rintf(qv);
      w4 = __builtin_amdgcn_cvt_pk_u8_f32(__builtin_amdgcn_fmed3f(rr + zu, 0.0f, 255.0f), r, w4);
      dist[r] = fmaf(tol_q, fabsf(qv), fabsf(qv - rr));
    }
    if (fmaxf(fmaxf(dist[0], dist[1]), fmaxf(dist[2], dist[3])) > doubt_at) {
#pragma unroll
      for (int r = 0; r < 4; ++r)
        if (dist[r] > doubt_at && qblk * NQ + qloc < T && f + r < hd) {
          const int slot = atomicAdd(&fix_cnt_s, 1);
          if (slot < FIX_CAP) {
            fix_ent[2 * slot] = qloc;
            fix_ent[2 * slot + 1] = f + r;
          }
        }
    }
    *(unsigned *)(stage + qloc * SRB + f) = w4 ^ 0x80808080u;
  }
  __syncthreads();
  decide_again_and_store<NEB, NQ, NW, FB, ONE>(stage, &fix_cnt_s, fix_ent, (double *)osum, m_s, qbase, kbase, vbase, qblk * NQ, T, Tp, hd, D,
                                          qs, qz, q_out + (size_t)b * T * D + (size_t)h * hd);
}

hipError_t launch_attention_f16(const float *q32, const float *k32, const float *vt32, int B, int T, int Tp, int H, int hd,
                                int DPv, const QParam *qp, int8_t *q_out, int beside, hipStream_t st) {
  const int neb = (hd + 15) / 16, nch = (hd + 31) / 32;
  if (hd > 80 || hd % 4) return hipErrorInvalidValue;      // K prefetch registers are sized for d <= 80
  const float q_mul = 1.4426950408889634f / std::sqrt((float)hd);     // log2(e) / sqrt(d)
  // Keys shared by the wavefronts, 16 (else 32) queries a workgroup, while that makes no more workgroups than this launch's share of
  // the compute units (`beside` launches of its kind run at the same time).  Measured, keys shared with 16 / with 32 queries / not
  // shared, one query block (16 heads of 72; us back to back, 4.5 of them the launch): 1 x 64 tokens 7.1 / 8.9 / 7.2, 1 x 256 9.9 / 12.2 / 12.4, 2 x 256
  // 16.7 / 11.7 / 11.8, 1 x 425 22.1 / 17.2 / 18.4, 3 x 256 22.5 / 19.5 / 12.0, 2 x 425 38.9 / 28.1 / 19.1, 1 x 1024 84 / 58.4 / 40.9; 6 heads of 64:
  // 1 x 256 8.6 / 9.8 / 11.0, 4 x 256 12.7 / 10.2 / 10.6, 5 x 256 12.7 / 10.2 / 11.3, 6 x 256 16.9 / 16.5 / 11.2, 1 x 1024 38.6 / 26.3 / 30.1.  Runs of 12 blocks with
  // 192 | 256 | 384 for the compute units: 1 x 256 tokens 1.43 | 1.36 | 1.36 ms, 1 x 425 2.05 | 1.99 | 2.00, 3 x 256 1.93 | 1.93 | 2.11; 6 heads: 5 x 256
  // 1.32 | 1.29 | 1.29, 1 x 1024 1.64 | 1.64 | 1.92.
  // Otherwise two query blocks per wavefront (128 queries per workgroup) when that makes more workgroups than compute units, else
  // one.  Measured, one / two (16 heads of 72; us): 4 x 256 tokens 12.5 / 16.5, 6 x 256 16.3 / 17.3, 8 x 256 16.9 / 18.0, 9 x 256 23.4 / 23.6, 10 x 256
  // 24.0 / 23.6, 12 x 256 27.2 / 25.0, 16 x 256 31.4 / 27.3, 3 x 425 24.5 / 26.6, 4 x 425 25.1 / 29.3, 5 x 425 34.1 / 34.5, 6 x 425 37.5 / 36.8, 8 x 425 43.3 / 39.8,
  // 1 x 1024 40.9 / 56.2, 2 x 1024 52.2 / 53.0, 3 x 1024 81.9 / 74.2; 6 heads of 64: 20 x 256 14.4 / 15.7, 24 x 256 20.0 / 20.4, 32 x 256 23.9 / 22.0.  Runs with
  // 192 | 256 | 384 there, two halves: 16 x 256 4.25 | 4.31 | 4.32 ms, 14 x 256 4.05 | 4.00 | 4.00, 8 x 425 4.41 | 4.29 | 4.29, 10 x 425 5.09 | 5.07 | 4.99; width 384,
  // 40 x 256 2.83 | 2.87 | 2.87, 56 x 256 3.58 | 3.59 | 3.64.
  const long long share = 256 / (beside > 1 ? beside : 1), heads = (long long)B * H;
  const int kq = heads * ((T + 15) / 16) <= share ? 1 : heads * ((T + 31) / 32) <= share ? 2 : 0;
  const int qb = B * H * ((T + 127) / 128) <= 256 ? 1 : 2;
  const int per_wg = kq ? 16 * kq : 64 * qb;
  dim3 grid((B * H + 7) / 8 * 8, (T + per_wg - 1) / per_wg);
#define QC_ATT_LAUNCH(...) \
  hipLaunchKernelGGL((__VA_ARGS__), grid, dim3(256), 0, st, q32, k32, vt32, B * H, T, Tp, H, hd, DPv, q_mul, qp, q_out)
#define QC_ATT_ONE(NCH, NEB, TAIL, ONE)                                            \
  do {                                                                             \
    if (kq == 1) QC_ATT_LAUNCH(attention_f16_keys_kernel<NCH, NEB, 1, TAIL, ONE>); \
    else if (kq == 2) QC_ATT_LAUNCH(attention_f16_keys_kernel<NCH, NEB, 2, TAIL, ONE>); \
    else if (qb == 1) QC_ATT_LAUNCH(attention_f16_kernel<NCH, NEB, 1, TAIL, ONE>); \
    else QC_ATT_LAUNCH(attention_f16_kernel<NCH, NEB, 2, TAIL, ONE>);              \
  } while (0)
#define QC_ATT(NCH, NEB, TAIL)                      \
  do {  /* 256: 64 keys a wavefront (decide_again_and_store) */ \
    if (T <= 256) QC_ATT_ONE(NCH, NEB, TAIL, true); \
    else QC_ATT_ONE(NCH, NEB, TAIL, false);         \
  } while (0)
  const bool tail = nch > 1 && hd - 32 * (nch - 1) <= 8;      // at most 8 features in the last chunk
  if (nch == 1 && neb == 1) QC_ATT(1, 1, false);
  else if (nch == 1) QC_ATT(1, 2, false);
  else if (nch == 2 && neb == 3 && tail) QC_ATT(2, 3, true);
  else if (nch == 2 && neb == 3) QC_ATT(2, 3, false);
  else if (nch == 2) QC_ATT(2, 4, false);
  else if (nch == 3 && neb == 5 && tail) QC_ATT(3, 5, true);
  else if (nch == 3 && neb == 5) QC_ATT(3, 5, false);
  else return hipErrorInvalidValue;
#undef QC_ATT
#undef QC_ATT_ONE
#undef QC_ATT_LAUNCH
  return hipGetLastError();
}

}  // namespace qc
