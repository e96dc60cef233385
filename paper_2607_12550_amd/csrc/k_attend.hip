// Decode-time attention evaluated on the compressed factors (the fused path that section 8
// and the conclusion name as the route to decode parity): the decoded cache
// X^_s = U_T (2^e_s G_s) U_d^T + R_s, R_s[t] = signs . H r'_s[t] / sqrt(d), is never formed.
//
//   key side:   q . X^_s[t] = U_T[t] . g + r'_s[t] . q',   g = 2^e_s G_s (U_d^T q),
//               q' = H (signs . q) / sqrt(d)           (H symmetric, entries +-1)
//   value side: sum_t p_t X^_s[t] = ((sum_t p_t U_T[t]) 2^e_s G_s) U_d^T
//                                   + signs . H (sum_t p_t r'_s[t]) / sqrt(d)
//
// Three kernels a call: k_attend_prep forms g and q' of the query heads of one key-value head of
// one item; a chunk pass runs over token chunks of one such key-value head (scores, softmax, and
// the value-side sums of U_T rows and dequantised codes, weighted by the unnormalised
// probabilities, for all its query heads at once); k_attend_combine merges the chunks with the
// usual max / rescale rule in a fixed order and applies the value factors and the inverse
// rotation.  The chunk pass is k_attend_mfma, on the matrix cores and over several 64-token tiles
// per workgroup, for fp16 factors with ranks in multiples of 8 and quantiser groups of 32 and more,
// the ordinary compressed cache; k_attend_chunk, vector code over one 64-token tile, for the rest
// (attend_use_mfma).  Per token a query head reads r_T factor values and d codes instead of d
// decoded values plus the decompression.
#include <algorithm>
#include <cmath>
#include <mutex>
#include <type_traits>

#include "common.h"
#include "kernels.h"
#include "rowops.h"

namespace {

// Blob pointers come from a table in memory, so the compiler cannot tell their address
// space: every load through them goes through gptr() (global_* instructions, which do not
// hold the LDS counter the way flat_* ones do).
JOLT_DEV float factor(const void *p, int64_t i, int f16) {
  return f16 ? (float)gptr(reinterpret_cast<const _Float16 *>(p))[i] : gptr(reinterpret_cast<const float *>(p))[i];
}

// The codes of one slice over a chunk (ATTN_CHUNK rows of D elements), held in registers
// between their global loads and the LDS dequantisation, so that the next slice's loads are
// in flight while the current slice is used.  Thread blocks of 8 elements, consecutive
// threads on consecutive blocks (coalesced); a block lies in one quantiser group (the group
// size is a multiple of 8).
template <int D>
struct CodeRegs {
  static constexpr int NB = ATTN_CHUNK * D / 8;
  static constexpr int BPT = (NB + 255) / 256;
  uint2 w[BPT];
  float sc[BPT];
};

template <int D>
JOLT_DEV void codes_load(CodeRegs<D> &c, const AttnBlob &b, int64_t row0, int nt, int group) {
#pragma unroll
  for (int k = 0; k < CodeRegs<D>::BPT; ++k) {
    const int blk = threadIdx.x + k * 256, t = blk / (D / 8), f = (blk % (D / 8)) * 8;
    c.w[k] = make_uint2(0u, 0u);
    c.sc[k] = 0.f;
    if (blk < CodeRegs<D>::NB && t < nt) {
      const int64_t elem = (row0 + t) * D + f;
      if (b.bits == 8) {
        const uint64_t v = *gptr(reinterpret_cast<const uint64_t *>(b.codes + elem));
        c.w[k].x = (uint32_t)v;
        c.w[k].y = (uint32_t)(v >> 32);
      }
      else if (b.bits == 4) c.w[k].x = *gptr(reinterpret_cast<const uint32_t *>(b.codes + elem / 2));
      else c.w[k].x = *gptr(reinterpret_cast<const uint16_t *>(b.codes + elem / 4));
      c.sc[k] = (float)*gptr(reinterpret_cast<const _Float16 *>(b.scales + elem / group));
    }
  }
}

// code - (2^b - 1)/2 (a half-integer of magnitude <= 127.5: exact in fp16) into ct[t][f .. f+7]
// and the block's scale into csc[t][f / 8]; rows past the chunk's end get scale 0
template <int D>
JOLT_DEV void codes_stash16(const CodeRegs<D> &c, int bits, _Float16 (*ct)[D + 8], float (*csc)[D / 8]) {
  const float mid = 0.5f * (float)((1 << bits) - 1);
  const uint32_t mask = (1u << bits) - 1u;
#pragma unroll
  for (int k = 0; k < CodeRegs<D>::BPT; ++k) {
    const int blk = threadIdx.x + k * 256, t = blk / (D / 8), f = (blk % (D / 8)) * 8;
    if (blk >= CodeRegs<D>::NB) continue;
    _Float16 v[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const int bit = i * bits;
      const uint32_t word = bit < 32 ? c.w[k].x : c.w[k].y;
      v[i] = (_Float16)((float)((word >> (bit & 31)) & mask) - mid);
    }
    uint4 pk;
    __builtin_memcpy(&pk, v, 16);
    *reinterpret_cast<uint4 *>(&ct[t][f]) = pk;
    csc[t][f / 8] = c.sc[k];
  }
}

// dst[q] = src(q) for q < n by all 256 threads: each thread issues eight loads before it
// stores any of them, so a pass costs one memory round trip, not eight
template <int NT = 256, class F>
JOLT_DEV void stage_lds(float *dst, int n, F src) {
  for (int q0 = threadIdx.x; q0 < n; q0 += NT * 8) {
    float v[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) {
      const int q = q0 + k * NT;
      v[k] = q < n ? src(q) : 0.f;
    }
#pragma unroll
    for (int k = 0; k < 8; ++k) {
      const int q = q0 + k * NT;
      if (q < n) dst[q] = v[k];
    }
  }
}

// eight consecutive factor values of a row (16-byte loads when the row start allows)
JOLT_DEV void factor8(const void *p, int64_t i, int f16, bool vec, float (&v)[8]) {
  if (f16 && vec) {
    const ju4 u = gload_u4(reinterpret_cast<const _Float16 *>(p) + i);
    const uint32_t w[4] = {u.x, u.y, u.z, u.w};
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      _Float16 lo, hi;
      const uint16_t l16 = (uint16_t)(w[k] & 0xffff), h16 = (uint16_t)(w[k] >> 16);
      __builtin_memcpy(&lo, &l16, 2); __builtin_memcpy(&hi, &h16, 2);
      v[2 * k] = (float)lo; v[2 * k + 1] = (float)hi;
    }
  } else if (!f16 && vec) {
    const jf4 x = gload_f4(reinterpret_cast<const float *>(p) + i), y = gload_f4(reinterpret_cast<const float *>(p) + i + 4);
    v[0] = x.x; v[1] = x.y; v[2] = x.z; v[3] = x.w; v[4] = y.x; v[5] = y.y; v[6] = y.z; v[7] = y.w;
  } else {
#pragma unroll
    for (int k = 0; k < 8; ++k) v[k] = factor(p, i + k, f16);
  }
}

// y[r][k] = sum_i M[i][k] x[r][i] for the n x rd factor M at element off and RM vectors x (rows of
// ldx floats in LDS): thread (8 columns, row stripe), 16-byte loads of M with several rows in
// flight, the stripes' partial sums added in order.  red: VM_RED floats of LDS; y in LDS, rows of
// ldy; all 256 threads call it and it ends with a barrier.
constexpr int VM_RED = 8192;
template <int RM>
JOLT_DEV void vecmat(const void *M, int64_t off, int n, int rd, int f16, const float *x, int ldx, int rep,
                     float *red, float *y, int ldy) {
  const int tid = threadIdx.x, c8 = (rd + 7) / 8, ldr = c8 * 8;
  const int stripes = min(256 / c8, VM_RED / (rep * ldr));
  const int st = tid / c8, k0 = (tid - st * c8) * 8;
  const bool vec = rd % 8 == 0;
  float acc[RM][8];
#pragma unroll
  for (int r = 0; r < RM; ++r)
#pragma unroll
    for (int e = 0; e < 8; ++e) acc[r][e] = 0.f;
  if (st < stripes) {
    auto row = [&](int i, float (&v)[8]) {
      if (i < n && vec) factor8(M, off + (int64_t)i * rd + k0, f16, true, v);
      else {
#pragma unroll
        for (int e = 0; e < 8; ++e) v[e] = i < n && k0 + e < rd ? factor(M, off + (int64_t)i * rd + k0 + e, f16) : 0.f;
      }
    };
    for (int i0 = st; i0 < n; i0 += 4 * stripes) {
      float v[4][8];
#pragma unroll
      for (int u = 0; u < 4; ++u) row(i0 + u * stripes, v[u]);
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int i = min(i0 + u * stripes, n - 1);
#pragma unroll
        for (int r = 0; r < RM; ++r)
          if (r < rep) {
            const float xi = x[r * ldx + i];
#pragma unroll
            for (int e = 0; e < 8; ++e) acc[r][e] = i0 + u * stripes < n ? fmaf(v[u][e], xi, acc[r][e]) : acc[r][e];
          }
      }
    }
#pragma unroll
    for (int r = 0; r < RM; ++r)
      if (r < rep) {
#pragma unroll
        for (int e = 0; e < 8; ++e) red[(st * rep + r) * ldr + k0 + e] = acc[r][e];
      }
  }
  __syncthreads();
  for (int q = tid; q < rep * rd; q += 256) {
    const int r = q / rd, k = q - r * rd;
    float sum = 0.f;
    for (int t = 0; t < stripes; ++t) sum += red[(t * rep + r) * ldr + k];
    y[r * ldy + k] = sum;
  }
  __syncthreads();
}

// out(r, i) receives sum_k M[i][k] y[r][k], rows i of the n x rd factor M one per thread
template <int RM, class F>
JOLT_DEV void matvec(const void *M, int64_t off, int n, int rd, int f16, const float *y, int ldy, int rep, F out) {
  const bool vec = rd % 8 == 0;
  for (int i = threadIdx.x; i < n; i += 256) {
    float acc[RM];
#pragma unroll
    for (int r = 0; r < RM; ++r) acc[r] = 0.f;
    auto dot8 = [&](int k, const float (&v)[8]) {
#pragma unroll
      for (int r = 0; r < RM; ++r)
        if (r < rep) {
#pragma unroll
          for (int e = 0; e < 8; ++e) acc[r] = fmaf(v[e], y[r * ldy + k + e], acc[r]);
        }
    };
    int k = 0;
    if (vec) {
      for (; k + 24 <= rd; k += 24) {          // three loads in flight
        float v[3][8];
#pragma unroll
        for (int u = 0; u < 3; ++u) factor8(M, off + (int64_t)i * rd + k + 8 * u, f16, true, v[u]);
#pragma unroll
        for (int u = 0; u < 3; ++u) dot8(k + 8 * u, v[u]);
      }
      for (; k < rd; k += 8) {
        float v[8];
        factor8(M, off + (int64_t)i * rd + k, f16, true, v);
        dot8(k, v);
      }
    } else {
      for (; k < rd; ++k) {
        const float u = factor(M, off + (int64_t)i * rd + k, f16);
#pragma unroll
        for (int r = 0; r < RM; ++r)
          if (r < rep) acc[r] = fmaf(u, y[r * ldy + k], acc[r]);
      }
    }
#pragma unroll
    for (int r = 0; r < RM; ++r)
      if (r < rep) out(r, i, acc[r]);
  }
}

// rotation sign of feature f: bit 0 of word 0 of Philox at counter (f, 0, 0, STREAM_SIGN)
JOLT_DEV float rot_sign(uint64_t seed, int f) {
  const u32x4 w = philox4x32_10(u32x4{(uint32_t)f, 0u, 0u, (uint32_t)STREAM_SIGN}, (uint32_t)seed, (uint32_t)(seed >> 32));
  return (w.x & 1u) ? -1.f : 1.f;
}

// Prep: one workgroup per (item, key-value head) for its rep query heads: q' by a fast
// Walsh-Hadamard transform (D / 8 lanes a row), q~ = U_d^T q, g = 2^e_s G_s q~.  Small calls
// carry their items as a kernel argument and this kernel stores them for the next two (no
// host-to-device copy in front of it).  One call of 32 items x 8 heads at ranks (128, 24):
// 28.2 us with one workgroup per query head and staged rows, 10.9 us here.
template <int D, int RM>
__global__ void __launch_bounds__(256) k_attend_prep(AttnArgs a, AttnItemTable tab) {
  constexpr int LW = D / 8;
  const int item = blockIdx.x, h = blockIdx.y, tid = threadIdx.x;
  if (tab.n > 0 && h == 0) {
    const uint32_t *src = reinterpret_cast<const uint32_t *>(&tab.it[item]);
    uint32_t *dst = reinterpret_cast<uint32_t *>(const_cast<AttnItem *>(a.items + item));
    for (int i = tid; i < (int)(sizeof(AttnItem) / 4); i += 256) dst[i] = src[i];
  }
  const AttnItem it = tab.n > 0 ? tab.it[item] : a.items[item];
  const AttnBlob &kb = it.k;
  const int rep = a.n_q / a.heads, s = it.layer * a.heads + h;
  __shared__ float q[RM][D], qt[RM][D], sg[D];
  __shared__ float red[VM_RED];
  const float *qin = a.Q + ((int64_t)item * a.n_q + h * rep) * D;
  for (int f = tid; f < rep * D; f += 256) q[f / D][f % D] = qin[f];
  for (int f = tid; f < D; f += 256) sg[f] = rot_sign(kb.seed, f);
  __syncthreads();
  if (kb.bits && tid < RM * LW) {
    const int r = tid / LW, lr = tid % LW;
    float v[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) v[e] = r < rep ? sg[lr * 8 + e] * q[r][lr * 8 + e] : 0.f;
    rowops::fwht_row<D>(v, lr);
    if (r < rep) {
      float *qr = a.qr + ((int64_t)item * a.n_q + h * rep + r) * D + lr * 8;
#pragma unroll
      for (int e = 0; e < 8; ++e) qr[e] = v[e] * a.inv_sqrt_d;
    }
  }
  if (kb.rT > 0) {
    vecmat<RM>(kb.Ud, 0, D, kb.rd, kb.f16, &q[0][0], D, rep, red, &qt[0][0], D);
    const int ge = (int)gptr(kb.gexp)[s];       // applied per value: 2^ge may not be an fp32
    float *gk = a.gk + ((int64_t)item * a.n_q + h * rep) * a.rk_max;
    const int rk = a.rk_max;
    matvec<RM>(kb.G, (int64_t)s * kb.rT * kb.rd, kb.rT, kb.rd, kb.f16, &qt[0][0], D, rep,
               [&](int r, int i, float v) { gk[(int64_t)r * rk + i] = ldexpf(v, ge); });
  }
}

// One rank block of U_T rows of a chunk: thread (row t = tid / 4, ranks (tid % 4) * 8 + 0..7
// of the block), loaded into registers ahead of its LDS stash.
constexpr int ATTN_RB = 32;

JOLT_DEV void urows_load(float (&u)[8], const AttnBlob &b, int t0, int nt, int i0) {
  const int t = threadIdx.x >> 2, i = i0 + (threadIdx.x & 3) * 8;
#pragma unroll
  for (int k = 0; k < 8; ++k) u[k] = 0.f;
  if (t >= nt || i >= b.rT) return;
  const int64_t e = (int64_t)(t0 + t) * b.rT + i;
  if (i + 8 <= b.rT && (b.f16 ? (e & 7) == 0 : (e & 3) == 0)) {
    factor8(b.UT, e, b.f16, true, u);
  } else {
#pragma unroll
    for (int k = 0; k < 8; ++k) u[k] = i + k < b.rT ? factor(b.UT, e + k, b.f16) : 0.f;
  }
}

// Chunk pass: one workgroup per (64-token chunk, key-value head, item), so that every
// workgroup issues all of its global loads at once (the slice's key and value codes of the
// chunk, the first rank block of both token factors, the slice's queries) and several
// workgroups share a CU.  For the rep query heads of slice s:
//   1. key scores: residual part from the dequantised codes staged in LDS (fp16 code
//      offsets, one scale per 8 elements) against the rotated queries, plus the low-rank
//      part U_T[t] . g over rank blocks of 32;
//   2. chunk-local softmax: wave r holds head r, lane t token t (scores never leave
//      registers);
//   3. value residual sums b[r][f] = sum_t p[r][t] r'[t][f] and value low-rank sums
//      a[r][i] = sum_t p[r][t] U_T[t][i]: thread (column, token stripe), stripes added in a
//      fixed order.
// REP > 0: the number of query heads per key-value head, fixed at compile time (the head
// loops unroll without predicates); REP = 0 takes it from the call (at most ATTN_REP_MAX).
template <int D, int REP>
__global__ void __launch_bounds__(256) k_attend_chunk(AttnArgs a) {
  constexpr int CH = ATTN_CHUNK, RB = ATTN_RB, RMAX = REP ? REP : ATTN_REP_MAX, P = 256 / D;
  static_assert(CH == 64, "one lane per token of a chunk");
  const int chunk = blockIdx.x, h = blockIdx.y, item = blockIdx.z, tid = threadIdx.x;
  const int lane = tid & 63, wave = tid >> 6;
  const AttnItem it = a.items[item];     // by value: one set of scalar loads
  const AttnBlob &kb = it.k, &vb = it.v;
  const int T = a.T, t0 = chunk * CH, nt = min(CH, T - t0);
  const int nq = a.n_q, rep = REP ? REP : nq / a.heads, s = it.layer * a.heads + h, j0 = h * rep;
  __shared__ __attribute__((aligned(16))) _Float16 ct[CH][D + 8];
  __shared__ float csc[CH][D / 8];
  __shared__ float ut[CH][RB + 1];
  __shared__ float gq[RMAX][RB];
  __shared__ __attribute__((aligned(16))) float qv[RMAX][D];
  __shared__ float pp[CH][RMAX];
  __shared__ float red[256 * RMAX];
  // every global load of the workgroup that does not depend on a later result
  CodeRegs<D> kr, vr;
  const int64_t row0 = (int64_t)s * T + t0;
  if (kb.bits) codes_load(kr, kb, row0, nt, a.group);
  if (vb.bits) codes_load(vr, vb, row0, nt, a.group);
  float uk[8], uv[8];
  urows_load(uk, kb, t0, nt, 0);
  urows_load(uv, vb, t0, nt, 0);
  {
    const float *qsrc = a.qr + ((int64_t)item * nq + j0) * D;     // rep consecutive rows
    stage_lds(&qv[0][0], rep * D, [&](int q) { return qsrc[q]; });
    const float *gsrc = a.gk + ((int64_t)item * nq + j0) * a.rk_max;
    const int rk = a.rk_max, rT = kb.rT;
    stage_lds(&gq[0][0], RMAX * RB, [&](int q) {
      const int r = q / RB, i = q % RB;
      return r < rep && i < rT ? gsrc[(int64_t)r * rk + i] : 0.f;
    });
  }
  if (kb.bits) codes_stash16(kr, kb.bits, ct, csc);
  {
    const int t = tid >> 2, c = (tid & 3) * 8;
#pragma unroll
    for (int k = 0; k < 8; ++k) ut[t][c + k] = uk[k];
  }
  __syncthreads();
  // 1. key scores: item k of a thread is head r = wave + 4 k, token t = lane
  float sc[2] = {0.f, 0.f};
  if (kb.bits) {
#pragma unroll
    for (int k = 0; k < 2; ++k) {
      const int r = wave + 4 * k;
      if (r >= rep) continue;
      float acc = 0.f;
      for (int b8 = 0; b8 < D / 8; ++b8) {
        const uint4 pk = *reinterpret_cast<const uint4 *>(&ct[lane][b8 * 8]);
        _Float16 cv[8];
        __builtin_memcpy(cv, &pk, 16);
        const float4 x = *reinterpret_cast<const float4 *>(&qv[r][b8 * 8]);
        const float4 y = *reinterpret_cast<const float4 *>(&qv[r][b8 * 8 + 4]);
        float d8 = (float)cv[0] * x.x;
        d8 = fmaf((float)cv[1], x.y, d8); d8 = fmaf((float)cv[2], x.z, d8); d8 = fmaf((float)cv[3], x.w, d8);
        d8 = fmaf((float)cv[4], y.x, d8); d8 = fmaf((float)cv[5], y.y, d8); d8 = fmaf((float)cv[6], y.z, d8);
        d8 = fmaf((float)cv[7], y.w, d8);
        acc = fmaf(csc[lane][b8], d8, acc);
      }
      sc[k] = acc;
    }
  }
  for (int i0 = 0; i0 < kb.rT; i0 += RB) {
    if (i0 > 0) {
      // next rank block: its loads were issued during the previous block
      __syncthreads();
      const int t = tid >> 2, c = (tid & 3) * 8;
#pragma unroll
      for (int k = 0; k < 8; ++k) ut[t][c + k] = uk[k];
      {
        const float *gsrc = a.gk + ((int64_t)item * nq + j0) * a.rk_max + i0;
        const int rk = a.rk_max, nr = kb.rT - i0;
        stage_lds(&gq[0][0], RMAX * RB, [&](int q) {
          const int r = q / RB, i = q % RB;
          return r < rep && i < nr ? gsrc[(int64_t)r * rk + i] : 0.f;
        });
      }
      __syncthreads();
    }
    if (i0 + RB < kb.rT) urows_load(uk, kb, t0, nt, i0 + RB);
    const int ni = min(RB, kb.rT - i0);
#pragma unroll
    for (int k = 0; k < 2; ++k) {
      const int r = wave + 4 * k;
      if (r >= rep) continue;
      float acc = sc[k];
      for (int i = 0; i < ni; ++i) acc = fmaf(ut[lane][i], gq[r][i], acc);
      sc[k] = acc;
    }
  }
  // 2. chunk-local softmax
  const int stride = 2 + a.rv_max + D;
  float *part = a.part + ((int64_t)item * a.chunks + chunk) * nq * stride;
#pragma unroll
  for (int k = 0; k < 2; ++k) {
    const int r = wave + 4 * k;
    if (r >= rep) continue;                       // uniform across the wave
    const float v = lane < nt ? sc[k] * a.scale : -INFINITY;
    float mx = v;
    for (int o = 32; o >= 1; o >>= 1) mx = fmaxf(mx, __shfl_xor(mx, o, 64));
    const float e = lane < nt ? expf(v - mx) : 0.f;
    float sum = e;
    for (int o = 32; o >= 1; o >>= 1) sum += __shfl_xor(sum, o, 64);
    pp[lane][r] = e;
    if (lane == 0) { part[(int64_t)(j0 + r) * stride] = mx; part[(int64_t)(j0 + r) * stride + 1] = sum; }
  }
  __syncthreads();
  // 3a. value residual sums
  if (vb.bits) codes_stash16(vr, vb.bits, ct, csc);
  {
    const int t = tid >> 2, c = (tid & 3) * 8;
#pragma unroll
    for (int k = 0; k < 8; ++k) ut[t][c + k] = uv[k];
  }
  __syncthreads();
  {
    const int f = tid % D, stripe = tid / D;
    float acc[RMAX];
#pragma unroll
    for (int r = 0; r < RMAX; ++r) acc[r] = 0.f;
    if (vb.bits) {
      for (int t = stripe; t < nt; t += P) {
        const float v = csc[t][f / 8] * (float)ct[t][f];
#pragma unroll
        for (int r = 0; r < RMAX; ++r)
          if (r < rep) acc[r] = fmaf(pp[t][r], v, acc[r]);
      }
    }
#pragma unroll
    for (int r = 0; r < RMAX; ++r) red[(stripe * RMAX + r) * D + f] = acc[r];
  }
  __syncthreads();
  for (int q = tid; q < rep * D; q += 256) {
    const int r = q / D, f = q % D;
    float sum = 0.f;
    for (int st = 0; st < P; ++st) sum += red[(st * RMAX + r) * D + f];
    part[(int64_t)(j0 + r) * stride + 2 + a.rv_max + f] = sum;
  }
  // 3b. value low-rank sums, rank block by rank block (stripes of 8 tokens)
  for (int i0 = 0; i0 < vb.rT; i0 += RB) {
    __syncthreads();
    if (i0 > 0) {
      const int t = tid >> 2, c = (tid & 3) * 8;
#pragma unroll
      for (int k = 0; k < 8; ++k) ut[t][c + k] = uv[k];
      __syncthreads();
    }
    if (i0 + RB < vb.rT) urows_load(uv, vb, t0, nt, i0 + RB);
    {
      const int i = tid % RB, stripe = tid / RB;   // 8 stripes
      float acc[RMAX];
#pragma unroll
      for (int r = 0; r < RMAX; ++r) acc[r] = 0.f;
      for (int t = stripe; t < nt; t += 256 / RB) {
        const float u = ut[t][i];
#pragma unroll
        for (int r = 0; r < RMAX; ++r)
          if (r < rep) acc[r] = fmaf(pp[t][r], u, acc[r]);
      }
#pragma unroll
      for (int r = 0; r < RMAX; ++r) red[(stripe * RMAX + r) * RB + i] = acc[r];
    }
    __syncthreads();
    const int ni = min(RB, vb.rT - i0);
    for (int q = tid; q < rep * ni; q += 256) {
      const int r = q / ni, i = q % ni;
      float sum = 0.f;
      for (int st = 0; st < 256 / RB; ++st) sum += red[(st * RMAX + r) * RB + i];
      part[(int64_t)(j0 + r) * stride + 2 + i0 + i] = sum;
    }
  }
}


// ---------------------------------------------------------------- chunk pass on the matrix cores
// The same sums as k_attend_chunk for fp16 factors with ranks in multiples of 8 and quantiser
// groups of at least 32, as 16x16x32 MFMA products with the query heads of a key-value head on
// the 16-wide side.  Nothing is held in fewer bits than fp32: the matrix that carries the
// queries or the probabilities goes in as three terms x = hi + mid + lo of 11 (fp16) or 8
// (bf16) bits each, side by side in the 16 columns (term * 4 + head for up to four heads per
// key-value head, term * 8 + head in two tiles otherwise), the other operand (factors, code
// offsets) is exact, and the terms' fp32 sums are added smallest first.
//
// One workgroup walks TILES tiles of 64 tokens of one (item, key-value head):
//   1. wave w scores tokens 16 w .. + 15: codes and U_T rows go from memory into the A
//      operand's registers directly (lane = token, 8 consecutive features or ranks per step),
//      one accumulator per quantiser group;
//   2. thread (token, head) applies the group scales, keeps the running maximum and
//      denominator, and writes p (for U_T) and p * scale (per group) as split terms;
//   3. the waves share out the 16-wide feature and rank tiles of the value sums; code offsets
//      and U_T rows lie token-major in LDS and are read transposed (ds_read_b64_tr_b16), row
//      strides 16 * odd halves so that the 16 rows of a read fall in distinct banks.
// The next tile's codes, factor rows and scales are requested before phase 2.
// What bounds it: HBM for the codes plus U_T through L2 once per key-value head; the heads of
// one chunk are neighbours in the launch order of one XCD so that they share its L2.  Measured,
// vector pass -> this: 32 items x 8 heads x 4096 tokens (4 queries a head) 398 -> 178 us, 1.6 TB/s;
// 5 x 40 x 4001 (1 query) 228 -> 152 us; 8 x 8 x 32768 (4) 972 -> 389 us.
typedef _Float16 h8_t __attribute__((ext_vector_type(8)));
typedef __bf16 b8_t __attribute__((ext_vector_type(8)));
typedef float f4_t __attribute__((ext_vector_type(4)));
typedef short s4_t __attribute__((ext_vector_type(4)));

// LDS carve of the matrix-core chunk pass, in bytes (host and device)
struct AttnLds {
  int bq, bg, s, p, al, vc, vu, total;
  int p_ld, vc_ld, vu_ld;
};
JOLT_HD AttnLds attn_lds(int D, int group, int rep, int rk, int rv) {
  AttnLds l{};
  const int nt = rep > 4 ? 2 : 1, ng = D / group, r4 = rep > 4 ? 8 : 4;
  int o = 0;
  l.bq = o; o += D / 32 * nt * 1024;              // rotated queries, B operand order
  l.bg = o; o += (rk + 31) / 32 * nt * 1024;              // g, B operand order
  l.s = o; o += (ng + 1) * r4 * 64 * 4;                   // scores per group and of the backbone
  l.p_ld = 72;
  l.p = o; o += ((ng + 1) * 3 * r4 + 16) * l.p_ld * 2;    // split probabilities (tiles read past the last term)
  l.al = o; o += 64;
  l.vc_ld = 16 * ((D / 16) | 1);
  l.vc = o; o += 64 * l.vc_ld * 2;
  l.vu_ld = 16 * (((rv + 15) / 16) | 1);
  l.vu = o; o += rv > 0 ? 64 * l.vu_ld * 2 : 0;
  l.total = o;
  return l;
}

// eight b-bit codes (LSB first) minus (2^b - 1)/2 as bf16: exact (8 significant bits)
template <int BITS>
JOLT_DEV b8_t codes_bf16(uint64_t w) {
  const uint32_t x = (uint32_t)w, y = (uint32_t)(w >> 32);
  uint32_t e[2];                     // bytes: codes 0..3, 4..7
  if constexpr (BITS == 8) { e[0] = x; e[1] = y; }
  else if constexpr (BITS == 4) {
    const uint32_t lo = x & 0x0f0f0f0fu, hi = (x >> 4) & 0x0f0f0f0fu;    // codes 0 2 4 6, 1 3 5 7
    e[0] = __builtin_amdgcn_perm(hi, lo, 0x05010400u);
    e[1] = __builtin_amdgcn_perm(hi, lo, 0x07030602u);
  } else {
    const uint32_t v = (x & 0xffu) | ((x & 0xff00u) << 8);                // codes 0..3 | 4..7
    const uint32_t t = (v | (v << 4)) & 0x0f0f0f0fu;
    const uint32_t lo = t & 0x03030303u, hi = (t >> 2) & 0x03030303u;
    e[0] = __builtin_amdgcn_perm(hi, lo, 0x05010400u);
    e[1] = __builtin_amdgcn_perm(hi, lo, 0x07030602u);
  }
  constexpr float mid = 0.5f * (float)((1 << BITS) - 1);
  uint32_t o[4];
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    const uint32_t a = (e[k >> 1] >> (16 * (k & 1))) & 255u, b = (e[k >> 1] >> (16 * (k & 1) + 8)) & 255u;
    o[k] = __builtin_amdgcn_perm(__float_as_uint((float)b - mid), __float_as_uint((float)a - mid), 0x07060302u);
  }
  b8_t v;
  __builtin_memcpy(&v, o, 16);
  return v;
}

// x = t[0] + t[1] + t[2], each rounded to nearest in the 16-bit format
JOLT_DEV void split3_h(float x, uint16_t (&t)[3]) {
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    const _Float16 h = (_Float16)x;
    __builtin_memcpy(&t[k], &h, 2);
    x -= (float)h;
  }
}
JOLT_DEV void split3_b(float x, uint16_t (&t)[3]) {
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    const __bf16 h = (__bf16)x;
    __builtin_memcpy(&t[k], &h, 2);
    x -= (float)h;
  }
}

constexpr float ATTN_PSCALE = 16384.f;      // p <= 1 into fp16's upper range

// value from column n + delta of the row of 16 lanes (rotation within the row)
template <int DELTA>
JOLT_DEV float row_ahead(float x) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), 0x120 + 16 - DELTA, 0xf, 0xf, false));
}

// maximum over the wave: rotations within the rows of 16 lanes, then one lane of each row
JOLT_DEV float wave_max_f(float v) {
  v = fmaxf(v, row_ahead<8>(v));
  v = fmaxf(v, row_ahead<4>(v));
  v = fmaxf(v, row_ahead<2>(v));
  v = fmaxf(v, row_ahead<1>(v));
  const int x = __float_as_int(v);
  const float a = __int_as_float(__builtin_amdgcn_readlane(x, 0)), b = __int_as_float(__builtin_amdgcn_readlane(x, 16));
  const float c = __int_as_float(__builtin_amdgcn_readlane(x, 32)), d = __int_as_float(__builtin_amdgcn_readlane(x, 48));
  return fmaxf(fmaxf(a, b), fmaxf(c, d));
}

// What one side's loads of a tile need, wave-uniform.  Every load is unconditional: rows past
// the end read the last row again (their probabilities are zero), ranks past r_T the last ranks
// (their operand is zero), and a side without codes or backbone reads its item's record, so
// that no branch or merge stands between a load and its use.
struct AttnSide {
  const uint8_t *codes, *scales, *UT;    // slice s (codes, scales); all token rows
  uint32_t last8;                        // byte offset of the slice's last 8 code bytes
  int bits, ng, rT, r_last;              // 0 where absent; r_last: first of the last 8 ranks
};
template <int D>
JOLT_DEV AttnSide attn_side(const AttnBlob &b, const AttnItem *safe, int s, int T, int ng) {
  AttnSide v;
  const uint8_t *p = reinterpret_cast<const uint8_t *>(safe);
  const int64_t srow = (int64_t)s * T;
  v.bits = b.bits;
  v.ng = b.bits ? ng : 0;
  v.rT = b.rT;
  v.codes = b.bits ? b.codes + srow * (D / 8) * b.bits : p;
  v.scales = b.bits ? reinterpret_cast<const uint8_t *>(b.scales + srow * ng) : p;
  v.UT = b.rT ? reinterpret_cast<const uint8_t *>(b.UT) : p;
  v.last8 = b.bits ? (uint32_t)T * (D / 8) * b.bits - 8u : 0u;
  v.r_last = b.rT ? b.rT - 8 : 0;
  return v;
}
// 8 codes of row t from feature f on (LSB first): 8 bytes, moved back inside the slice at its end
template <int D>
JOLT_DEV uint64_t code_word(const AttnSide &v, int t, int f) {
  const uint32_t want = (uint32_t)((t * D + f) >> 3) * v.bits, at = min(want, v.last8);
  return *gptr(reinterpret_cast<const uint64_t *>(v.codes + at)) >> (8 * (want - at));
}
// up to four fp16 scales of row t (the codes section follows the scales, so 8 bytes are there)
JOLT_DEV uint64_t scale_word(const AttnSide &v, int t) {
  return *gptr(reinterpret_cast<const uint64_t *>(v.scales + (uint32_t)(t * v.ng) * 2u));
}

// KS: rank steps of 32 of the key factor held in registers per tile (more are loaded as they
// are needed); VU: rank tiles of 16 of the value factor per wave
template <int D, int NT, int KS, int VU>
__global__ void __launch_bounds__(256, VU > 4 ? 1 : 2) k_attend_mfma(AttnArgs a) {
  constexpr int J = D / 32;                           // feature steps
  constexpr int CT = D >= 64 ? D / 64 : 1;            // feature tiles of 16 per wave
  constexpr int R4 = NT == 2 ? 8 : 4;                 // column stride between the terms
  constexpr int UQ = VU * 2;                          // 16-byte pieces of U_T rows per thread
  const int i_ = blockIdx.x, job = (i_ & 7) * a.per_xcd + (i_ >> 3);
  const int per_item = a.chunks * a.heads;
  if (job >= a.n_items * per_item) return;
  const int item = job / per_item, rem = job - item * per_item, chunk = rem / a.heads, h = rem - chunk * a.heads;
  const AttnItem it = a.items[item];
  const AttnBlob &kb = it.k, &vb = it.v;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, n16 = lane & 15, kg = lane >> 4;
  const int T = a.T, nq = a.n_q, rep = nq / a.heads, s = it.layer * a.heads + h, j0 = h * rep;
  const int group = a.group, ng = D / group, spg = group / 32;
  const bool wide = group % 64 == 0;
  const int rTk = kb.rT, rTv = vb.rT, ksteps = (rTk + 31) / 32;
  const int t_begin = chunk * a.chunk_tokens, t_end = min(T, t_begin + a.chunk_tokens);
  extern __shared__ __attribute__((aligned(16))) uint8_t lds[];
  const AttnLds L = attn_lds(D, group, rep, a.rk_max, a.rv_max);
  uint16_t *bq = reinterpret_cast<uint16_t *>(lds + L.bq), *bg = reinterpret_cast<uint16_t *>(lds + L.bg);
  float *S = reinterpret_cast<float *>(lds + L.s), *al = reinterpret_cast<float *>(lds + L.al);
  uint16_t *Pm = reinterpret_cast<uint16_t *>(lds + L.p);
  uint16_t *Vc = reinterpret_cast<uint16_t *>(lds + L.vc), *Vu = reinterpret_cast<uint16_t *>(lds + L.vu);
  __shared__ float gmax[ATTN_REP_MAX];

  // ---- loads of one tile
  const AttnSide ks_ = attn_side<D>(kb, a.items + item, s, T, ng), vs_ = attn_side<D>(vb, a.items + item, s, T, ng);
  uint64_t kc[J], vc[J], ksc, vsc;
  ju4 ku[KS], vu[UQ];
  uint16_t vu_at[UQ];                    // LDS position (16-byte units) of this thread's U_T pieces
  const int vr8 = rTv >> 3;
#pragma unroll
  for (int q = 0; q < UQ; ++q) {
    const int c = tid + 256 * q, row = vr8 > 0 ? c / vr8 : 64;
    vu_at[q] = (uint16_t)(row < 64 ? row * (L.vu_ld / 8) + (c - row * vr8) : 0xffff);
  }
  const int kf0 = wide ? kg * 16 : kg * 8;          // step j starts at kf0 + kf(j)
  auto kf = [&](int j) { return wide ? (j >> 1) * 64 + (j & 1) * 8 : j * 32; };
  auto load_ku = [&](int t, int step) -> ju4 {
    const uint32_t e = (uint32_t)(t * ks_.rT + min(step * 32 + kg * 8, ks_.r_last));
    return gload_u4(ks_.UT + 2u * e);
  };
  auto load_tile = [&](int t0) {
    const int t = min(t0 + 16 * wave + n16, T - 1), tl = min(t0 + lane, T - 1);
    ksc = scale_word(ks_, tl);
    vsc = scale_word(vs_, tl);
#pragma unroll
    for (int j = 0; j < J; ++j) kc[j] = code_word<D>(ks_, t, kf0 + kf(j));
#pragma unroll
    for (int q = 0; q < KS; ++q)
      if (q < ksteps) ku[q] = load_ku(t, q);
    // units of 8 codes, consecutive threads on consecutive units
#pragma unroll
    for (int j = 0; j < J; ++j) {
      const int u = tid + 256 * j;
      vc[j] = code_word<D>(vs_, min(t0 + u / (D / 8), T - 1), u % (D / 8) * 8);
    }
    const int last = max(min(64, T - t0) * vr8 - 1, 0);
    const uint8_t *ut = vs_.UT + (int64_t)t0 * rTv * 2;
#pragma unroll
    for (int q = 0; q < UQ; ++q)
      if (256 * q < 64 * vr8) vu[q] = gload_u4(ut + 16u * (uint32_t)min(tid + 256 * q, last));
  };
  auto scale_of = [&](uint64_t sc, int g) -> float {
    _Float16 x;
    const uint16_t b = (uint16_t)(sc >> (16 * g));
    __builtin_memcpy(&x, &b, 2);
    return (float)x;
  };
  load_tile(t_begin);

  // ---- B operands of the scores: element (k, n) at [tile][step][k group * 16 + n][k % 8]
  const float *qsrc = a.qr + ((int64_t)item * nq + j0) * D;
  const float *gsrc = a.gk + ((int64_t)item * nq + j0) * a.rk_max;
  auto put_b = [&](uint16_t *b, int steps, int step, int k, int e, int r, const uint16_t (&t)[3]) {
#pragma unroll
    for (int m = 0; m < 3; ++m) {
      const int col = m * R4 + r, tile = col >> 4;
      b[((tile * steps + step) * 64 + k * 16 + (col & 15)) * 8 + e] = t[m];
    }
  };
  for (int q = tid; q < rep * D; q += 256) {
    const int r = q / D, f = q % D;
    uint16_t t3[3];
    split3_b(qsrc[q], t3);
    // feature f is element e of k group k in step j of the A operand's order
    int j, k, e;
    if (wide) { j = (f >> 6) * 2 + ((f >> 3) & 1); k = (f >> 4) & 3; e = f & 7; }
    else { j = f >> 5; k = (f >> 3) & 3; e = f & 7; }
    put_b(bq, J, j, k, e, r, t3);
  }
  // g scaled by a power of two per head into fp16's range (max in [2^14, 2^15))
  for (int r = wave; r < rep; r += 4) {
    float mx = 0.f;
    for (int i = lane; i < rTk; i += 64) mx = fmaxf(mx, fabsf(gsrc[(int64_t)r * a.rk_max + i]));
    mx = wave_max_f(mx);
    if (lane == 0) gmax[r] = mx;
  }
  __syncthreads();
  auto gexp_of = [&](int r) -> int {
    const float mx = gmax[r];
    int ex = 0;
    if (mx > 0.f && mx < INFINITY) { (void)frexpf(mx, &ex); ex -= 15; }
    return ex;
  };
  for (int q = tid; q < rep * ksteps * 32; q += 256) {
    const int r = q / (ksteps * 32), i = q - r * (ksteps * 32);
    uint16_t t3[3] = {0, 0, 0};
    if (i < rTk) split3_h(ldexpf(gsrc[(int64_t)r * a.rk_max + i], -gexp_of(r)), t3);
    put_b(bg, ksteps, i >> 5, (i >> 3) & 3, i & 7, r, t3);
  }
  // softmax state: wave w keeps heads w and (NT == 2) w + 4
  float m_run[NT], l_run[NT];
  int gex[NT];
#pragma unroll
  for (int x = 0; x < NT; ++x) {
    m_run[x] = -INFINITY; l_run[x] = 0.f;
    gex[x] = wave + 4 * x < rep ? gexp_of(wave + 4 * x) : 0;
  }
  f4_t oc[CT][NT], ou[VU][NT];
#pragma unroll
  for (int x = 0; x < NT; ++x) {
#pragma unroll
    for (int c = 0; c < CT; ++c) oc[c][x] = f4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int c = 0; c < VU; ++c) ou[c][x] = f4_t{0.f, 0.f, 0.f, 0.f};
  }
  __syncthreads();

  // sum of the three terms' columns, then four tokens of head n16 to the score table
  auto put_s = [&](int v, const f4_t (&acc)[NT]) {
    f4_t x;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      if constexpr (NT == 1) x[q] = (row_ahead<8>(acc[0][q]) + row_ahead<4>(acc[0][q])) + acc[0][q];
      else x[q] = (acc[NT - 1][q] + row_ahead<8>(acc[0][q])) + acc[0][q];
    }
    if (n16 < rep) *reinterpret_cast<f4_t *>(S + (v * R4 + n16) * 64 + 16 * wave + 4 * kg) = x;
  };

  f4_t acc[NT];
  auto stash_codes = [&](auto bits) {
#pragma unroll
    for (int j = 0; j < J; ++j) {
      const int u = tid + 256 * j, row = u / (D / 8), f8 = u % (D / 8);
      *reinterpret_cast<b8_t *>(Vc + row * L.vc_ld + f8 * 8) = codes_bf16<decltype(bits)::value>(vc[j]);
    }
  };
  auto score_codes = [&](auto bits) {
#pragma unroll
    for (int j = 0; j < J; ++j) {
      const b8_t fa = codes_bf16<decltype(bits)::value>(kc[j]);
#pragma unroll
      for (int x = 0; x < NT; ++x) {
        const b8_t fb = *reinterpret_cast<const b8_t *>(bq + ((x * J + j) * 64 + lane) * 8);
        acc[x] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fa, fb, acc[x], 0, 0, 0);
      }
      if ((j + 1) % spg == 0) {
        put_s(j / spg, acc);
#pragma unroll
        for (int x = 0; x < NT; ++x) acc[x] = f4_t{0.f, 0.f, 0.f, 0.f};
      }
    }
  };
  auto by_bits = [&](int bits, auto f) {
    if (bits == 8) f(std::integral_constant<int, 8>{});
    else if (bits == 4) f(std::integral_constant<int, 4>{});
    else if (bits == 2) f(std::integral_constant<int, 2>{});
  };

  for (int t0 = t_begin; t0 < t_end; t0 += 64) {
    // ---- value operands to LDS
    by_bits(vb.bits, stash_codes);
#pragma unroll
    for (int q = 0; q < UQ; ++q)
      if (vu_at[q] != 0xffff) *reinterpret_cast<ju4 *>(Vu + 8 * (int)vu_at[q]) = vu[q];
    // ---- 1. scores
#pragma unroll
    for (int x = 0; x < NT; ++x) acc[x] = f4_t{0.f, 0.f, 0.f, 0.f};
    by_bits(kb.bits, score_codes);
    if (rTk > 0) {
      auto step = [&](int q, ju4 w) {
        h8_t fa;
        __builtin_memcpy(&fa, &w, 16);
#pragma unroll
        for (int x = 0; x < NT; ++x) {
          const h8_t fb = *reinterpret_cast<const h8_t *>(bg + ((x * ksteps + q) * 64 + lane) * 8);
          acc[x] = __builtin_amdgcn_mfma_f32_16x16x32_f16(fa, fb, acc[x], 0, 0, 0);
        }
      };
#pragma unroll
      for (int q = 0; q < KS; ++q)
        if (q < ksteps) step(q, ku[q]);
      for (int q = KS; q < ksteps; ++q) step(q, load_ku(min(t0 + 16 * wave + n16, T - 1), q));
      put_s(ng, acc);
    }
    const uint64_t ksw = ksc, vsw = vsc;
    if (t0 + 64 < t_end) load_tile(t0 + 64);
    __syncthreads();
    // ---- 2. running softmax: thread (token = lane, heads wave and wave + 4)
#pragma unroll
    for (int x = 0; x < NT; ++x) {
      const int r = wave + 4 * x;
      if (r < rep) {
        float sc = 0.f;
        if (kb.bits) {
#pragma unroll
          for (int g = 0; g < 4; ++g)
            if (g < ng) sc = fmaf(scale_of(ksw, g), S[(g * R4 + r) * 64 + lane], sc);
        }
        if (rTk > 0) sc += ldexpf(S[(ng * R4 + r) * 64 + lane], gex[x]);
        const bool live = t0 + lane < t_end;
        const float v = live ? sc * a.scale : -INFINITY;
        const float mn = fmaxf(m_run[x], wave_max_f(v));
        const float p = live ? expf(v - mn) : 0.f;
        const float alpha = expf(m_run[x] - mn);       // 0 before the first tile
        l_run[x] = fmaf(l_run[x], alpha, p);
        m_run[x] = mn;
        if (lane == 0) al[r] = alpha;
        auto put_p = [&](int var, const uint16_t (&t3)[3]) {
#pragma unroll
          for (int m = 0; m < 3; ++m) {
            const int row = m * R4 + r;
            Pm[(var * 3 * R4 + row) * L.p_ld + lane] = t3[m];
          }
        };
        uint16_t t3[3];
        if (vb.bits) {
#pragma unroll
          for (int g = 0; g < 4; ++g)
            if (g < ng) { split3_b(p * scale_of(vsw, g), t3); put_p(g, t3); }
        }
        if (rTv > 0) { split3_h(p * ATTN_PSCALE, t3); put_p(ng, t3); }
      }
    }
    __syncthreads();
    // ---- 3. value sums
    f4_t av;
#pragma unroll
    for (int q = 0; q < 4; ++q) av[q] = al[(NT == 1 ? 0 : (kg & 1) * 4) + q];
    // B operand: 8 tokens kg * 8 .. of column n16, two transposed reads of 4 rows x 16 columns
    auto rd_b = [&](const uint16_t *m, int ld, int col0, int ks) {
      const uint16_t *p = m + (32 * ks + 8 * kg + (n16 >> 2)) * ld + col0 + (n16 & 3) * 4;
      const s4_t x = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s4_t *)p);
      const s4_t y = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s4_t *)(p + 4 * ld));
      return __builtin_shufflevector(x, y, 0, 1, 2, 3, 4, 5, 6, 7);
    };
    if (vb.bits) {
#pragma unroll
      for (int c = 0; c < CT; ++c) {
        const int ct = wave * CT + c;
        if (ct * 16 < D) {
          const int g = ct * 16 / group;
#pragma unroll
          for (int x = 0; x < NT; ++x) oc[c][x] *= av;
#pragma unroll
          for (int ks = 0; ks < 2; ++ks) {
            const auto w = rd_b(Vc, L.vc_ld, ct * 16, ks);
            b8_t fb;
            __builtin_memcpy(&fb, &w, 16);
#pragma unroll
            for (int x = 0; x < NT; ++x) {
              const b8_t fa = *reinterpret_cast<const b8_t *>(Pm + (g * 3 * R4 + x * 16 + n16) * L.p_ld + 32 * ks + 8 * kg);
              oc[c][x] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fa, fb, oc[c][x], 0, 0, 0);
            }
          }
        }
      }
    }
#pragma unroll
    for (int c = 0; c < VU; ++c) {
      const int rt = wave + 4 * c;
      if (rt * 16 < rTv) {
#pragma unroll
        for (int x = 0; x < NT; ++x) ou[c][x] *= av;
#pragma unroll
        for (int ks = 0; ks < 2; ++ks) {
          const auto w = rd_b(Vu, L.vu_ld, rt * 16, ks);
          h8_t fb;
          __builtin_memcpy(&fb, &w, 16);
#pragma unroll
          for (int x = 0; x < NT; ++x) {
            const h8_t fa = *reinterpret_cast<const h8_t *>(Pm + (ng * 3 * R4 + x * 16 + n16) * L.p_ld + 32 * ks + 8 * kg);
            ou[c][x] = __builtin_amdgcn_mfma_f32_16x16x32_f16(fa, fb, ou[c][x], 0, 0, 0);
          }
        }
      }
    }
    __syncthreads();
  }
  // ---- partial results of the chunk
  const int stride = 2 + a.rv_max + D;
  float *part = a.part + (((int64_t)item * a.chunks + chunk) * nq + j0) * stride;
#pragma unroll
  for (int x = 0; x < NT; ++x) {
    const int r = wave + 4 * x;
    float l = l_run[x];
    for (int o = 32; o >= 1; o >>= 1) l += __shfl_xor(l, o, 64);
    if (r < rep && lane == 0) { part[(int64_t)r * stride] = m_run[x]; part[(int64_t)r * stride + 1] = l; }
  }
  // row m of a tile is (term, head): four heads per lane group kg = term, or eight over two
  auto put_o = [&](const f4_t (&acc)[NT], int col, bool in, float mul) {
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      float v;
      int r;
      if constexpr (NT == 1) {
        const float mid = __shfl(acc[0][q], n16 + 16, 64), lo = __shfl(acc[0][q], n16 + 32, 64);
        v = (lo + mid) + acc[0][q];
        r = kg == 0 ? q : rep;
      } else {
        const float mid = __shfl(acc[0][q], (lane + 32) & 63, 64);
        v = (acc[NT - 1][q] + mid) + acc[0][q];
        r = kg < 2 ? kg * 4 + q : rep;
      }
      if (in && r < rep) part[(int64_t)r * stride + 2 + col] = v * mul;
    }
  };
#pragma unroll
  for (int c = 0; c < CT; ++c) {
    const int ct = wave * CT + c;
    if (ct * 16 < D) put_o(oc[c], a.rv_max + ct * 16 + n16, true, 1.f);
  }
#pragma unroll
  for (int c = 0; c < VU; ++c) {
    const int rt = wave + 4 * c;
    if (rt * 16 < rTv) put_o(ou[c], rt * 16 + n16, rt * 16 + n16 < rTv, 1.f / ATTN_PSCALE);
  }
}

// Combine: one workgroup per (item, key-value head) and RM of its query heads: chunk weights,
// the chunk partials' columns (four columns of four chunks in flight per thread), then
// w = 2^e_s G_s^T a and U_d w with the factors read once for all of them and the residual's
// inverse rotation by a fast Walsh-Hadamard transform.  32 items x 32 query heads at ranks
// (136, 72): 48.5 us with one workgroup per query head over 64 chunks, 18.3 us here
// over 8.
template <int D, int RM>
__global__ void __launch_bounds__(256) k_attend_combine(AttnArgs a) {
  constexpr int LW = D / 8;
  const int item = blockIdx.x, h = blockIdx.y, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const AttnItem it = a.items[item];     // by value: one set of scalar loads
  const AttnBlob &vb = it.v;
  const int nrep = a.n_q / a.heads, r0 = blockIdx.z * RM, rep = min(RM, nrep - r0);
  const int s = it.layer * a.heads + h, j0 = h * nrep + r0;
  const int stride = 2 + a.rv_max + D, ncol = vb.rT + D;
  const float *part = a.part + ((int64_t)item * a.chunks * a.n_q + j0) * stride;
  const int64_t cstride = (int64_t)a.n_q * stride;
  __shared__ float w[RM][D], bv[RM][D], sg[D], Ls[RM];
  __shared__ float red[VM_RED];
  extern __shared__ float dyn[];          // chunk weights [rep][chunks], then a [rep][rT]
  float *cw = dyn, *av = dyn + (int64_t)RM * a.chunks;
  const int lda = vb.rT;
  for (int f = tid; f < D; f += 256) sg[f] = rot_sign(vb.seed, f);
  // per head (one wave each): M = max over chunks, weights exp(m_c - M), L = sum_c l_c w_c in
  // a fixed order
  for (int r = wave; r < rep; r += 4) {
    const float *pr = part + (int64_t)r * stride;
    float M = -INFINITY;
    for (int c = lane; c < a.chunks; c += 64) M = fmaxf(M, pr[c * cstride]);
    for (int o = 32; o >= 1; o >>= 1) M = fmaxf(M, __shfl_xor(M, o, 64));
    float L = 0.f;
    for (int c = lane; c < a.chunks; c += 64) {
      const float wgt = expf(pr[c * cstride] - M);
      cw[r * a.chunks + c] = wgt;
      L = fmaf(pr[c * cstride + 1], wgt, L);
    }
    for (int o = 32; o >= 1; o >>= 1) L += __shfl_xor(L, o, 64);
    if (lane == 0) Ls[r] = L;
  }
  __syncthreads();
  // a_r[i] = sum_c w_c a_c[i], b_r[f] = sum_c w_c b_c[f], chunks in order: U columns of 16 / U
  // chunks in flight per thread, no more columns than the call has (three of four loads of 160
  // columns repeated the last one: 1 item of 4 x 2 heads over 32768 tokens 135 -> 93 us in all)
  const int nc = rep * ncol;
  auto sum_columns = [&](auto u_) {
    constexpr int U = decltype(u_)::value, K = 16 / U;
    for (int q0 = tid; q0 < nc; q0 += U * 256) {
      const JOLT_GLOBAL float *pc[U];
      const float *wc[U];
      float acc[U];
      int rr[U], ii[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int q = min(q0 + 256 * u, nc - 1);
        acc[u] = 0.f;
        rr[u] = q / ncol; ii[u] = q - rr[u] * ncol;
        pc[u] = gptr(part) + (int64_t)rr[u] * stride + 2 + (ii[u] < vb.rT ? ii[u] : a.rv_max + (ii[u] - vb.rT));
        wc[u] = cw + rr[u] * a.chunks;
      }
      for (int c0 = 0; c0 < a.chunks; c0 += K) {
        float v[K][U];
#pragma unroll
        for (int k = 0; k < K; ++k)
#pragma unroll
          for (int u = 0; u < U; ++u) v[k][u] = c0 + k < a.chunks ? pc[u][(int64_t)(c0 + k) * cstride] : 0.f;
#pragma unroll
        for (int k = 0; k < K; ++k)
          if (c0 + k < a.chunks) {
#pragma unroll
            for (int u = 0; u < U; ++u) acc[u] = fmaf(wc[u][c0 + k], v[k][u], acc[u]);
          }
      }
#pragma unroll
      for (int u = 0; u < U; ++u) {
        if (q0 + 256 * u >= nc) break;
        if (ii[u] < vb.rT) av[rr[u] * lda + ii[u]] = acc[u];
        else bv[rr[u]][ii[u] - vb.rT] = acc[u];
      }
    }
  };
  if (nc <= 256) sum_columns(std::integral_constant<int, 1>{});
  else if (nc <= 512) sum_columns(std::integral_constant<int, 2>{});
  else sum_columns(std::integral_constant<int, 4>{});
  __syncthreads();
  // inverse rotation of the residual sums (in place), while the factor products follow
  if (vb.bits && tid < RM * LW) {
    const int r = tid / LW, lr = tid % LW;
    float v[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) v[e] = r < rep ? bv[r][lr * 8 + e] : 0.f;
    rowops::fwht_row<D>(v, lr);
#pragma unroll
    for (int e = 0; e < 8; ++e)
      if (r < rep) bv[r][lr * 8 + e] = v[e] * (sg[lr * 8 + e] * a.inv_sqrt_d);
  }
  float *o = a.O + ((int64_t)item * a.n_q + j0) * D;
  auto finish = [&](int r, int f, float lr) {
    o[(int64_t)r * D + f] = (lr + (vb.bits ? bv[r][f] : 0.f)) * (1.f / Ls[r]);
  };
  if (vb.rT > 0) {
    vecmat<RM>(vb.G, (int64_t)s * vb.rT * vb.rd, vb.rT, vb.rd, vb.f16, av, lda, rep, red, &w[0][0], D);
    const int ge = (int)gptr(vb.gexp)[s];       // applied per value: 2^ge may not be an fp32
    for (int q = tid; q < rep * vb.rd; q += 256) w[q / vb.rd][q % vb.rd] = ldexpf(w[q / vb.rd][q % vb.rd], ge);
    __syncthreads();
    matvec<RM>(vb.Ud, 0, D, vb.rd, vb.f16, &w[0][0], D, rep, finish);
  } else {
    __syncthreads();
    for (int q = tid; q < rep * D; q += 256) finish(q / D, q % D, 0.f);
  }
}

}  // namespace

namespace {

// workgroups that may need more than 64 KB of LDS in all have to declare it: the kernel's limit,
// the same from every call, so that calls of two threads cannot lower each other's
hipError_t allow_lds(const void *kernel, size_t dynamic, size_t limit) {
  if (dynamic <= 20 * 1024) return hipSuccess;
  if (dynamic > limit) return hipErrorInvalidValue;
  return hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)limit);
}
constexpr size_t MFMA_LDS_MAX = 150 * 1024, COMBINE_LDS_MAX = 112 * 1024;

template <int D, int NT, int KS, int VU>
hipError_t launch_mfma(const AttnArgs &a, hipStream_t st) {
  const AttnLds l = attn_lds(D, a.group, a.n_q / a.heads, a.rk_max, a.rv_max);
  const hipError_t e = allow_lds(reinterpret_cast<const void *>(&k_attend_mfma<D, NT, KS, VU>), l.total, MFMA_LDS_MAX);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL((k_attend_mfma<D, NT, KS, VU>), dim3(a.per_xcd * 8), dim3(256), l.total, st, a);
  return hipGetLastError();
}

template <int D, int NT>
hipError_t launch_mfma_ranks(const AttnArgs &a, hipStream_t st) {
  const int ks = (a.rk_max + 31) / 32, vu = (a.rv_max + 63) / 64;
  if (vu > 4) return launch_mfma<D, NT, 4, 8>(a, st);
  if (ks > 4 || vu > 3) return launch_mfma<D, NT, 6, 4>(a, st);
  return launch_mfma<D, NT, 4, 3>(a, st);
}

template <int D, int RM>
hipError_t launch_ends(const AttnArgs &a, const AttnItemTable &tab, bool prep, hipStream_t st) {
  if (prep) {
    hipLaunchKernelGGL((k_attend_prep<D, RM>), dim3(a.n_items, a.heads), dim3(256), 0, st, a, tab);
  } else {
    const int rep = a.n_q / a.heads;
    const size_t dyn = (size_t)RM * (a.chunks + a.rv_max) * sizeof(float);
    const hipError_t e = allow_lds(reinterpret_cast<const void *>(&k_attend_combine<D, RM>), dyn, COMBINE_LDS_MAX);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL((k_attend_combine<D, RM>), dim3(a.n_items, a.heads, (rep + RM - 1) / RM), dim3(256), dyn,
                       st, a);
  }
  return hipGetLastError();
}

constexpr int COMBINE_WGS = 256;

template <int D>
hipError_t launch_attend_d(const AttnArgs &a, const AttnItemTable &tab, hipStream_t st) {
  const int rep = a.n_q / a.heads;
  hipError_t e = rep == 1 ? launch_ends<D, 1>(a, tab, true, st)
                 : rep <= 4 ? launch_ends<D, 4>(a, tab, true, st) : launch_ends<D, 8>(a, tab, true, st);
  if (e != hipSuccess) return e;
  if (a.mfma) {
    e = rep > 4 ? launch_mfma_ranks<D, 2>(a, st) : launch_mfma_ranks<D, 1>(a, st);
  } else {
    const dim3 g(a.chunks, a.heads, a.n_items);
    if (rep == 1) hipLaunchKernelGGL((k_attend_chunk<D, 1>), g, dim3(256), 0, st, a);
    else if (rep == 2) hipLaunchKernelGGL((k_attend_chunk<D, 2>), g, dim3(256), 0, st, a);
    else if (rep == 4) hipLaunchKernelGGL((k_attend_chunk<D, 4>), g, dim3(256), 0, st, a);
    else if (rep == 8) hipLaunchKernelGGL((k_attend_chunk<D, 8>), g, dim3(256), 0, st, a);
    else hipLaunchKernelGGL((k_attend_chunk<D, 0>), g, dim3(256), 0, st, a);
    e = hipGetLastError();
  }
  if (e != hipSuccess) return e;
  // The heads of a key-value head share one combine workgroup (its factors are read once) while the
  // chunk weights fit 16 KB of LDS and the call still fills the chip.  A workgroup walks all chunks of
  // its heads, so few items get one workgroup per query head: 1 item of 8 x 8 heads, shared to not,
  // in all: 300 tokens 45 to 35 us, 8192 99 to 65, 32768 at ranks (300, 260) 794 to 523.
  const int64_t wgs = (int64_t)a.n_items * a.heads;
  if (rep > 4 && a.chunks <= 512 && wgs >= COMBINE_WGS) return launch_ends<D, 8>(a, tab, false, st);
  if (rep > 1 && a.chunks <= 1024 && wgs * ((rep + 3) / 4) >= COMBINE_WGS) return launch_ends<D, 4>(a, tab, false, st);
  return launch_ends<D, 1>(a, tab, false, st);
}

}  // namespace

// How a call is split: the matrix-core chunk pass takes fp16 factors with ranks in multiples of
// 8 (aligned 16-byte factor rows), groups of 32 features or more (one scale per 32-wide step)
// and value ranks up to 512 with key ranks up to 1024 (its LDS); the rest runs on the vector
// kernel.  Past value ranks of 256 its registers leave one workgroup to a CU, which pays only where
// four or more query heads share it and it walks several tiles: at value rank 264, matrix cores to
// vector pass, 8 heads of 4096 tokens: 32 items x 8 queries 572 to 1014 us, x 4 600 to 635, x 2 582
// to 533, x 1 574 to 428; 8 items x 8 226 to 276, x 4 218 to 179; 4 items x 8 173 to 160.  A workgroup walks several 64-token tiles (fewer partials to write and merge) as long
// as about 2048 workgroups remain, four rounds of the 512 that fit the chip.
bool attend_use_mfma(const AttnItem *items, int n, int heads, int T, int d, int group, int rep, int rk, int rv) {
  if (group % 32 || d % group || rv > 512) return false;
  if (rv > 256 && (rep < 4 || (int64_t)((T + 63) / 64) * heads * n * rep < 32768)) return false;
  for (int i = 0; i < n; ++i)
    for (const AttnBlob *b : {&items[i].k, &items[i].v})
      if (!b->f16 || b->rT % 8 || (b->bits != 0 && b->bits != 2 && b->bits != 4 && b->bits != 8)) return false;
  return attn_lds(d, group, rep, rk, rv).total <= (int)MFMA_LDS_MAX;
}

int attend_chunk_tokens(int n_items, int heads, int T) {
  const int64_t tiles = (int64_t)((T + 63) / 64) * heads * n_items;
  return 64 * (int)std::min<int64_t>(64, std::max<int64_t>(1, tiles / 2048));
}

hipError_t launch_attend(const AttnArgs &a, const AttnItemTable &tab, int d, hipStream_t st) {
  if (d == 32) return launch_attend_d<32>(a, tab, st);
  if (d == 64) return launch_attend_d<64>(a, tab, st);
  if (d == 128) return launch_attend_d<128>(a, tab, st);
  return hipErrorInvalidValue;
}

// Fixed device scratch of jolt_attend_noalloc: the attention workspace of callers that
// cannot allocate device memory.  One array per device that loads the library, held until
// the process ends; every call on a device shares it.
static __device__ __align__(256) uint8_t scratch[ATTN_SCRATCH_BYTES];

namespace {
std::mutex g_scratch_mu;
void *g_scratch_dev[ATTN_SCRATCH_DEVICES] = {};
}  // namespace

// Device address of this device's scratch array, resolved once per device with
// hipGetSymbolAddress while that device is current (the array's name in host code is not a
// device address).
hipError_t attend_scratch_address(int device, void **ptr) {
  if (!ptr || device < 0 || device >= ATTN_SCRATCH_DEVICES) return hipErrorInvalidValue;
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  if (!g_scratch_dev[device]) {
    void *p = nullptr;
    const hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return e;
    if (!p) return hipErrorInvalidSymbol;
    g_scratch_dev[device] = p;
  }
  *ptr = g_scratch_dev[device];
  return hipSuccess;
}
