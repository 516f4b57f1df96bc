// What the int8 GEMM kernels share: operand types, the XCD grid, and the epilogues (dequantise, GELU + requantise,
// cache store + gated residual, QKV scatter) applied to a tile of integer accumulators.
#pragma once
#include <type_traits>

#include "qc_internal.h"

namespace qc {

typedef int v4i __attribute__((ext_vector_type(4)));
typedef int v2i __attribute__((ext_vector_type(2)));
typedef unsigned v2u __attribute__((ext_vector_type(2)));
typedef unsigned v4u __attribute__((ext_vector_type(4)));
typedef int v16i __attribute__((ext_vector_type(16)));
typedef float v4f __attribute__((ext_vector_type(4)));


constexpr int NUM_XCD = 8;
constexpr int GELU_FIX_CAP = 1024;      // queue of fc1 outputs decided again in float64, per tile

__device__ __forceinline__ int map_col(int j, int sel_D) {
  return sel_D ? (j < sel_D ? j + 2 * sel_D : j + 4 * sel_D) : j;
}

// 8 packed bytes (16 nibbles, element 2j low, 2j+1 high) -> 16 int8 codes.
__device__ __forceinline__ v4i unpack_w4(v2i p) {
  v4i o;
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    unsigned w = (unsigned)(h ? p.y : p.x);
    unsigned lo = w & 0x0F0F0F0Fu;
    unsigned hi = (w >> 4) & 0x0F0F0F0Fu;
    lo |= (lo & 0x08080808u) * 0x1Eu;   // sign-extend each nibble inside its byte
    hi |= (hi & 0x08080808u) * 0x1Eu;
    unsigned e0 = __builtin_amdgcn_perm(hi, lo, 0x05010400u);   // l0 h0 l1 h1
    unsigned e1 = __builtin_amdgcn_perm(hi, lo, 0x07030602u);   // l2 h2 l3 h3
    if (h == 0) { o.x = (int)e0; o.y = (int)e1; } else { o.z = (int)e0; o.w = (int)e1; }
  }
  return o;
}

// Four codes of GELU(v) at once, v = sc * corr + bs.  The codes are formed as the paper's unsigned ones (zero point + 128): qz
// = GELU(v) / s + z leaves one fused multiply-add, v times 1 / (s + s exp(-2u)) (the step folded into the denominator), and one
// instruction rounds it to nearest even, clamps it to 0 .. 255 and places the byte; the sign bit of the four bytes is flipped
// back in the result.
// Bound of the fast path's error in units of the output step, as a multiple of |v| / s (|GELU(v)| <= |v|): 1.5e-6 covers the
// float32 dequantisation (accumulators beyond 2^24 are rounded on conversion) and the exp2 / reciprocal estimates with a margin
// of 2, 2e-7 the unrefined quotient; absolute, 2e-6 cover the bias rounding and 8e-6 = 2^-17 the rounding of qz (below 256;
// beyond, every value clamps to the same code).  An element is in doubt when qz lies closer than the bound to a half:
// | fract(qz) - 1/2 | - tol_v |v| < near_half.
struct GeluQuant {
  float o_s, o_zu, tol_v;
  static constexpr float near_half = 1e-5f;
  __device__ __forceinline__ explicit GeluQuant(const QParam &oq) : o_s(oq.s), o_zu((float)(oq.z + 128)), tol_v(1.7e-6f * (1.0f / oq.s)) {}
  __device__ __forceinline__ unsigned codes(const v4i &corr, const v4f &sc, const v4f &bs, float (&clear)[4]) const {
    const float c1 = -2.0f * 0.7978845608028654f * 1.4426950408889634f, c2 = c1 * 0.044715f;      // -2 sqrt(2/pi) log2(e)
    unsigned w = 0;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const float v = fmaf(sc[e], (float)corr[e], bs[e]);
      const float t = v * fmaf(c2, v * v, c1);
      const float qz = fmaf(v, __builtin_amdgcn_rcpf(fmaf(o_s, __builtin_amdgcn_exp2f(t), o_s)), o_zu);
      w = __builtin_amdgcn_cvt_pk_u8_f32(qz, e, w);
      clear[e] = fmaf(-tol_v, fabsf(v), fabsf(__builtin_amdgcn_fractf(qz) - 0.5f));
    }
    return w ^ 0x80808080u;
  }
  __device__ __forceinline__ bool doubt(const float (&clear)[4]) const {
    return fminf(fminf(clear[0], clear[1]), fminf(clear[2], clear[3])) < near_half;
  }
};

// Dequantised output of a quantised linear as it is stored: the float32 rounding of the float64 value
// (a_s * w_s[n]) * (acc - a_z * wsum[n]) + bias[n] (the product of the two scales is exact in float64; one float64
// multiplication, one float64 addition, one rounding to float32).  Stored tensors then carry no rounding of their own
// beyond the storage format, so the codes quantised from them further down do not depend on the order of operations here.
__device__ __forceinline__ float dequant_f32(double sc, int corr, double bs) {
  return (float)__dadd_rn(__dmul_rn(sc, (double)corr), bs);
}

// The fc1 epilogue's exact path for one output element: float64 from the integer accumulator to the GELU value, one
// rounding to float32, Eq. 1 with an IEEE division.  x / (1 + exp(-2u)) = 0.5 x (1 + tanh u).
__device__ __noinline__ int gelu_code_exact(int corr, float a_s, float w_s, float bias, float o_s, int o_z) {
  const double u = __dadd_rn(__dmul_rn((double)a_s * (double)w_s, (double)corr), (double)bias);
  const double k = 0.7978845608028654 * (u + 0.044715 * u * u * u);
  const float g = (float)(u / (1.0 + exp(-2.0 * k)));
  const float r = __builtin_rintf(g / o_s) + (float)o_z;
  return (int)fminf(fmaxf(r, -128.0f), 127.0f);
}

// Eq. 1 on signed codes with the quotient v / s refined to the correctly rounded
// value by one Newton step on the reciprocal estimate.
__device__ __forceinline__ int quant_code(float v, float s, float inv_s, float z) {
  float q = v * inv_s;
  q = fmaf(fmaf(-q, s, v), inv_s, q);
  float r = __builtin_rintf(q) + z;
  r = fminf(fmaxf(r, -128.0f), 127.0f);
  return (int)r;
}

// What the epilogue of a tile reads from memory besides the accumulators, for kernels that request it in front of their main loop (the
// same tile arguments): of one wavefront's TM x TN blocks of 32 x 32, lane l's column l % 32 of every block column.  X: the residual
// stream's elements too (float32 ones: converting others would wait for them at once).
template <int EPI, int TM, int TN, bool X>
struct EpiPre {
  static_assert(!X || EPI == EPI_RESID, "");
  QParam qp, oq;
  float sc[TN], bs[TN], gate[TN];
  int zw[TN];
  float x[X ? TN : 1][TM][16];
};
template <int BM, int BN, int WM, int WN, int EPI, bool X>
__device__ __forceinline__ void epilogue_request(const GemmArgs &p, EpiPre<EPI, BM / WM / 32, BN / WN / 32, X> &e, const int wave, const int m0,
                                                 const int n0) {
  constexpr int TM = BM / WM / 32, TN = BN / WN / 32;
  const int lane = threadIdx.x & 63, wm0 = (wave / WN) * (BM / WM), wn0 = (wave % WN) * (BN / WN);
  e.qp = p.a_qp ? *p.a_qp : QParam{p.a_scale, p.a_zp};
  if constexpr (EPI == EPI_GELU_Q) e.oq = *p.o_qp;
#pragma unroll
  for (int j = 0; j < TN; ++j) {
    const int n = min(n0 + wn0 + j * 32 + (lane & 31), p.N - 1);
    e.sc[j] = p.w_scale[n];
    e.zw[j] = p.wsum[n];
    e.bs[j] = p.bias ? p.bias[n] : 0.0f;
    if constexpr (EPI == EPI_RESID) e.gate[j] = p.gate[(long long)(m0 / p.rows_per_batch) * p.ld_gate + n];
    if constexpr (X) {
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const int m = min(m0 + wm0 + i * 32 + (r >> 2) * 8 + (lane >> 5) * 4 + (r & 3), p.M - 1);
          e.x[j][i][r] = ((const float *)p.x)[(long long)m * p.N + n];
        }
    }
  }
}

// Epilogue of a tile: acc[i][j] is the 32 x 32 block (i along the rows m of the activations, j along the output
// columns n) of wavefront (wave / WN, wave % WN); for EPI_GELU_Q the weights were the first MFMA operand (register
// index runs along n), otherwise the activations were (register index runs along m).  smem: the workgroup's dynamic
// LDS, free for reuse (every wavefront is past its last fragment read).
// RBF: the residual stream or the cache may be bfloat16 (read from the arguments); false: both are known to be float32.
// pre: what epilogue_request has fetched (z is 0 then), or null.
template <int BM, int BN, int WM, int WN, int EPI, bool RBF = true, bool PRE = false, bool PREX = false>
__device__ __forceinline__ void gemm_epilogue(const GemmArgs &p, v16i (&acc)[BM / WM / 32][BN / WN / 32], unsigned char *smem,
                                              const int m0, const int n0, const int z,
                                              const EpiPre<EPI, BM / WM / 32, BN / WN / 32, PREX> *pre = nullptr) {
  constexpr int TM = BM / WM / 32, TN = BN / WN / 32, NT = 64 * WM * WN;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm0 = (wave / WN) * (BM / WM), wn0 = (wave % WN) * (BN / WN);
  const int ncover = p.sel_D ? 2 * p.sel_D : p.N;
  float a_s = p.a_scale;
  int a_z = p.a_zp;
  if constexpr (PRE) {
    a_s = pre->qp.s;
    a_z = pre->qp.z;
  } else if (p.a_qp) {
    QParam q = p.a_qp[(long long)z * p.zs_qp];
    a_s = q.s;
    a_z = q.z;
  }
  const float *w_scale = p.w_scale + (long long)z * p.zs_vecN;
  const int32_t *wsum = p.wsum + (long long)z * p.zs_vecN;
  const float *bias = p.bias ? p.bias + (long long)z * p.zs_vecN : nullptr;
  if (EPI == EPI_GELU_Q) {
    // per-column constants into LDS: v = sc[n] * float(acc - zw[n]) + bs[n]
    float *c_sc = (float *)smem;
    int *c_zw = (int *)(smem + BN * 4);
    float *c_bs = (float *)(smem + BN * 8);
    unsigned char *stage = smem + BN * 12;             // [BM][BN + 16] codes
    constexpr int SROW = BN + 16;
    // Elements whose fast evaluation lands too close to a rounding boundary of Eq. 1 to be trusted are queued here and
    // decided again in float64 (gelu_code_exact): the codes are then those of exact arithmetic on the accumulators.
    int *fix_cnt = (int *)(stage + BM * SROW);
    int *fix_ent = fix_cnt + 4;                        // [GELU_FIX_CAP][4]: accumulator minus zero-point term, column, row
    if (tid == 0) *fix_cnt = 0;
    if constexpr (PRE) {
      if (wm0 == 0 && lane < 32) {
#pragma unroll
        for (int j = 0; j < TN; ++j) {
          const int nl = wn0 + j * 32 + lane;
          const bool ok = n0 + nl < p.N;
          c_sc[nl] = ok ? a_s * pre->sc[j] : 0.0f;
          c_zw[nl] = ok ? a_z * pre->zw[j] : 0;
          c_bs[nl] = ok ? pre->bs[j] : 0.0f;
        }
      }
    } else if (tid < BN) {
      const int n = n0 + tid;
      const bool ok = n < p.N;
      c_sc[tid] = ok ? a_s * w_scale[n] : 0.0f;
      c_zw[tid] = ok ? a_z * wsum[n] : 0;
      c_bs[tid] = (ok && bias) ? bias[n] : 0.0f;
    }
    __syncthreads();
    QParam oq;
    if constexpr (PRE) oq = pre->oq;
    else oq = *p.o_qp;
    const GeluQuant gq(oq);
    const int g = lane >> 5;
#pragma unroll
    for (int j = 0; j < TN; ++j) {
#pragma unroll
      for (int rg = 0; rg < 4; ++rg) {
        const int nl = wn0 + j * 32 + rg * 8 + g * 4;       // 4 consecutive columns of this lane
        const v4f sc = *(const v4f *)(c_sc + nl);
        const v4i zw = *(const v4i *)(c_zw + nl);
        const v4f bs = *(const v4f *)(c_bs + nl);
#pragma unroll
        for (int i = 0; i < TM; ++i) {
          float clear[4];
          v4i corr;
#pragma unroll
          for (int e = 0; e < 4; ++e) corr[e] = acc[i][j][rg * 4 + e] - zw[e];
          const unsigned w = gq.codes(corr, sc, bs, clear);
          // one comparison and one branch per four outputs; taken by a wavefront about once in a hundred times
          if (gq.doubt(clear)) {
#pragma unroll
            for (int e = 0; e < 4; ++e)
              if (clear[e] < gq.near_half) {
                const int slot = atomicAdd(fix_cnt, 1);
                if (slot < GELU_FIX_CAP) {
                  fix_ent[slot * 4 + 0] = corr[e];
                  fix_ent[slot * 4 + 1] = nl + e;
                  fix_ent[slot * 4 + 2] = wm0 + i * 32 + (lane & 31);
                }
              }
          }
          *(unsigned *)(stage + (wm0 + i * 32 + (lane & 31)) * SROW + nl) = w;
        }
      }
    }
    __syncthreads();
    {
      const int nfix = min(*fix_cnt, GELU_FIX_CAP);
      for (int f = tid; f < nfix; f += NT) {
        const int corr = fix_ent[f * 4 + 0], nl = fix_ent[f * 4 + 1], row = fix_ent[f * 4 + 2];
        const int n = n0 + nl;
        if (n < p.N) stage[row * SROW + nl] = (unsigned char)gelu_code_exact(corr, a_s, w_scale[n], bias ? bias[n] : 0.0f, oq.s, oq.z);
      }
      if (nfix) __syncthreads();
    }
    // coalesced write-out: 16-byte chunks, 8 lanes cover a 128-byte row segment
    constexpr int CH = BN / 16;
    for (int c = tid; c < BM * CH; c += NT) {
      const int r = c / CH, cc = (c % CH) * 16;
      const int m = m0 + r, n = n0 + cc;
      if (m >= p.M || n >= p.N) continue;
      int8_t *dst = p.q_out + (long long)m * p.ldq + n;
      if (n + 16 <= p.N) {
        *(v4i *)dst = *(const v4i *)(stage + r * SROW + cc);
      } else {
        for (int e = 0; n + e < p.N; ++e) dst[e] = (int8_t)stage[r * SROW + cc + e];
      }
    }
    return;
  }

  if (EPI == EPI_QKV) {
    // float32 values scattered to the head-major layouts of the attention kernel: Q and K [B, H, T, hd], V transposed
    // and key-permuted [B, H, DP, Tp]; p.y, when set, also receives them row-major ([M, 3 D], for inspection)
    const int T = p.rows_per_batch, D = p.N / 3;
    const bool fast_t = (T % 4) == 0;
    const bool tile_one_batch = (T % BM) == 0;      // then every row of the tile belongs to batch element m0 / T
    const int b_tile = m0 / T;
    if (BM == 128 && BN == 128 && tile_one_batch && fast_t && m0 + BM <= p.M && D % BN == 0 && (p.hd & 3) == 0 && (p.Tp & 7) == 0) {
      // Tile inside one batch element and inside one of Q, K, V: the values go through LDS (free after
      // the K loop) and leave as 16-byte stores along the contiguous direction of their layout (Q / K: features of a
      // token and head; V^T: tokens of a feature).
      const int tb = m0 - b_tile * T;                         // first token of the tile
      const int part = n0 / D;
      float *stage = (float *)smem;
      constexpr int SR = BN + 4, VR = BM + 4;                 // floats per staged token row (Q / K) and feature row (V^T)
#pragma unroll
      for (int j = 0; j < TN; ++j) {
        const int nl = wn0 + j * 32 + (lane & 31);
        const double sc = (double)a_s * (double)w_scale[n0 + nl];
        const int zw = a_z * wsum[n0 + nl];
        const double bs = bias ? (double)bias[n0 + nl] : 0.0;
        float *ycol = p.y ? p.y + (long long)m0 * p.ldy + n0 + nl : nullptr;     // 32 lanes write 128 contiguous bytes
#pragma unroll
        for (int i = 0; i < TM; ++i) {
#pragma unroll
          for (int rg = 0; rg < 4; ++rg) {
            const int ml = wm0 + i * 32 + rg * 8 + (lane >> 5) * 4;
            v4f v;
#pragma unroll
            for (int q = 0; q < 4; ++q) {
              v[q] = dequant_f32(sc, acc[i][j][rg * 4 + q] - zw, bs);
              if (ycol) ycol[(unsigned)(ml + q) * (unsigned)p.ldy] = v[q];
            }
            if (part < 2) {
#pragma unroll
              for (int q = 0; q < 4; ++q) stage[(ml + q) * SR + nl] = v[q];
            } else {
              // four consecutive tokens stay together under the key permutation of the V^T rows
              *(v4f *)(stage + nl * VR + vt_pos(ml)) = v;
            }
          }
        }
      }
      __syncthreads();
      if (part < 2) {
        // thread -> four features cc .. cc + 3 (inside one head: heads start at multiples of hd, a multiple of 4) of
        // the rows cr, cr + NT / 32, ...
        const int cr = tid >> 5, cc = (tid & 31) * 4;
        const int nn = n0 - part * D + cc, h = nn / p.hd, e = nn - h * p.hd;
        float *dst = (part == 0 ? p.q32 : p.k32) +
                     ((unsigned)(b_tile * p.heads + h) * (unsigned)T + (unsigned)(tb + cr)) * (unsigned)p.hd + (unsigned)e;
#pragma unroll
        for (int q = 0; q < BM * 32 / NT; ++q)
          *(v4f *)(dst + (unsigned)(q * (NT / 32)) * (unsigned)p.hd) = *(const v4f *)(stage + (cr + q * (NT / 32)) * SR + cc);
      } else {
        // thread -> 4 consecutive token positions ch of the features fc, fc + NT / 32, ...
        const int fc = tid >> 5, ch = (tid & 31) * 4;
#pragma unroll
        for (int q = 0; q < BN * 32 / NT; ++q) {
          const int col = fc + q * (NT / 32);
          const int nn = n0 - 2 * D + col, h = nn / p.hd, e = nn - h * p.hd;
          const unsigned o = ((unsigned)(b_tile * p.heads + h) * (unsigned)p.DP + (unsigned)e) * (unsigned)p.Tp + (unsigned)(tb + ch);
          *(v4f *)(p.vt32 + o) = *(const v4f *)(stage + col * VR + ch);
        }
      }
      return;
    }
#pragma unroll
    for (int j = 0; j < TN; ++j) {
      const int n = n0 + wn0 + j * 32 + (lane & 31);
      if (n >= p.N) continue;
      const double sc = (double)a_s * (double)(PRE ? pre->sc[j] : w_scale[n]);
      const int zw = a_z * (PRE ? pre->zw[j] : wsum[n]);
      const double bs = PRE ? (double)pre->bs[j] : bias ? (double)bias[n] : 0.0;
      const int part = n / D, nn = n - part * D, h = nn / p.hd, e = nn - h * p.hd;
      float *dqk = part == 0 ? p.q32 : p.k32;
#pragma unroll
      for (int i = 0; i < TM; ++i) {
#pragma unroll
        for (int rg = 0; rg < 4; ++rg) {
          const int mb = m0 + wm0 + i * 32 + rg * 8 + (lane >> 5) * 4;   // 4 consecutive rows mb .. mb+3
          if (mb >= p.M) continue;
          v4f v;
#pragma unroll
          for (int q = 0; q < 4; ++q) v[q] = dequant_f32(sc, acc[i][j][rg * 4 + q] - zw, bs);
          const int b0 = tile_one_batch ? b_tile : mb / T, t0 = mb - b0 * T;
          if (part == 2 && fast_t && mb + 3 < p.M) {
            // T is a multiple of 4: the four rows are tokens t0 .. t0 + 3 of one batch element, contiguous in V^T
            *(v4f *)(p.vt32 + ((long long)(b0 * p.heads + h) * p.DP + e) * p.Tp + vt_pos(t0)) = v;
          } else {
#pragma unroll
            for (int q = 0; q < 4; ++q) {
              if (mb + q >= p.M) continue;
              int b = b0, t = t0 + q;
              while (t >= T) { t -= T; ++b; }
              if (part == 2) p.vt32[((long long)(b * p.heads + h) * p.DP + e) * p.Tp + vt_pos(t)] = v[q];
              else dqk[((long long)(b * p.heads + h) * T + t) * p.hd + e] = v[q];
            }
          }
          if (p.y) {
#pragma unroll
            for (int q = 0; q < 4; ++q)
              if (mb + q < p.M) p.y[(long long)(mb + q) * p.ldy + n] = v[q];
          }
        }
      }
    }
    return;
  }

  if (EPI == EPI_RESID) {
    // read-modify-write of the residual stream: every load of the tile is issued before the first use, so the epilogue pays
    // one memory round trip
    const bool uniform_batch = (p.rows_per_batch % BM) == 0;
    const int b_uniform = m0 / p.rows_per_batch;
    const int x_bf16 = RBF ? p.x_bf16 : 0, cache_bf16 = RBF ? p.cache_bf16 : 0;
    const bool interior = uniform_batch && m0 + BM <= p.M && n0 + BN <= p.N;
    float xv[TN][TM][16], gv[TN];
    double scv[TN], bsv[TN];
    int zwv[TN];
#pragma unroll
    for (int j = 0; j < TN; ++j) {
      const int n = min(n0 + wn0 + j * 32 + (lane & 31), p.N - 1);
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const int m = min(m0 + wm0 + i * 32 + (r >> 2) * 8 + (lane >> 5) * 4 + (r & 3), p.M - 1);
          if constexpr (PREX) xv[j][i][r] = pre->x[j][i][r];
          else xv[j][i][r] = stream_load(p.x, (long long)m * p.N + n, x_bf16);
        }
      scv[j] = (double)a_s * (double)(PRE ? pre->sc[j] : w_scale[n]);
      zwv[j] = a_z * (PRE ? pre->zw[j] : wsum[n]);
      bsv[j] = PRE ? (double)pre->bs[j] : bias ? (double)bias[n] : 0.0;
      gv[j] = PRE ? pre->gate[j] : p.gate[(long long)b_uniform * p.ld_gate + n];
    }
#pragma unroll
    for (int j = 0; j < TN; ++j) {
      const int n = n0 + wn0 + j * 32 + (lane & 31);
      if (interior) {
        // interior tile inside one batch element: no bounds checks, one gate per column
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
          for (int r = 0; r < 16; ++r) {
            const float v = dequant_f32(scv[j], acc[i][j][r] - zwv[j], bsv[j]);
            // 32-bit offset inside the tile's rows from one 64-bit base per column
            const long long ob = (long long)m0 * p.N + n;
            const unsigned o = (unsigned)(wm0 + i * 32 + (r >> 2) * 8 + (lane >> 5) * 4 + (r & 3)) * (unsigned)p.N;
            if (cache_bf16) ((unsigned short *)p.cache_out + ob)[o] = bf16_bits(v);
            else ((float *)p.cache_out + ob)[o] = v;
            stream_store(p.x, ob + o, fmaf(gv[j], v, xv[j][i][r]), x_bf16);
          }
      } else {
        if (n >= p.N) continue;
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
          for (int r = 0; r < 16; ++r) {
            const int m = m0 + wm0 + i * 32 + (r >> 2) * 8 + (lane >> 5) * 4 + (r & 3);
            if (m >= p.M) continue;
            const float v = dequant_f32(scv[j], acc[i][j][r] - zwv[j], bsv[j]);
            const long long o = (long long)m * p.N + n;
            if (cache_bf16) ((unsigned short *)p.cache_out)[o] = bf16_bits(v);
            else ((float *)p.cache_out)[o] = v;
            const float g = p.gate[(long long)(m / p.rows_per_batch) * p.ld_gate + n];
            stream_store(p.x, o, fmaf(g, v, xv[j][i][r]), x_bf16);
          }
      }
    }
    return;
  }

#pragma unroll
  for (int j = 0; j < TN; ++j) {
    const int jl = n0 + wn0 + j * 32 + (lane & 31);
    if (jl >= ncover) continue;
    const int n = map_col(jl, p.sel_D);                // (PRE: sel_D is 0)
    const double sc = (double)a_s * (double)(PRE ? pre->sc[j] : w_scale[n]);
    const int zw = a_z * (PRE ? pre->zw[j] : wsum[n]);
    const double bs = PRE ? (double)pre->bs[j] : bias ? (double)bias[n] : 0.0;
#pragma unroll
    for (int i = 0; i < TM; ++i) {
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int m = m0 + wm0 + i * 32 + (r >> 2) * 8 + (lane >> 5) * 4 + (r & 3);
        if (m >= p.M) continue;
        const int a = acc[i][j][r];
        float *y = p.y + (long long)z * p.zs_out;
        y[(long long)m * p.ldy + n] = dequant_f32(sc, a - zw, bs);
        if (p.acc_out) p.acc_out[(long long)m * p.N + n] = a;
      }
    }
  }
}

// XCD grid rows that move the fewest bytes into the eight L2s, weighted by load imbalance
inline int xcd_rows(int tiles_m, int tiles_n, double bytes_a, double bytes_w) {
  int best_xm = 1;
  double best = 1e300;
  for (int xm = 1; xm <= NUM_XCD; xm *= 2) {
    const int xn = NUM_XCD / xm;
    const int cm = (tiles_m + xm - 1) / xm, cn = (tiles_n + xn - 1) / xn;
    const double cost = (xn * bytes_a + xm * bytes_w) * ((double)cm * cn * NUM_XCD / ((double)tiles_m * tiles_n));
    if (cost < best) { best = cost; best_xm = xm; }
  }
  return best_xm;
}

}  // namespace qc
