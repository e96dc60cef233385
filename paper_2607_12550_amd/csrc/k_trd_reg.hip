// Householder tridiagonalisation A = Q T Q^T with the matrix held in registers, batched over
// symmetric matrices of one size (n <= 1024): the feature Grams, FlashJoLT's B B^T, the slice
// Grams and the token Grams of short caches.
//
// Reading the trailing matrix from L2 once per column, in one workgroup per matrix, took 12 us a
// column at n = 256 and 16 us at n = 522 (one CU's L2 bandwidth, strided column reads and five
// barriers in a chain).  The chip's vector registers hold far more than these matrices, so each
// matrix is spread over the registers of TW wavefronts (one workgroup up to n = 256, TW / 8
// workgroups of eight waves above): wave rho keeps the rows TW j + rho, lane l of it the columns
// 64 c + l, and the rank-2 update of every column is applied at once, in place.
//
// Per column i every wave holds x = row i (column layout) and forms the reflector itself:
//   v = x scaled, tau, beta (norms summed in fp64; no barrier);
//   its rows' products (A v)_r, summed over lanes for four rows at a time by v_permlane swaps;
//   the products and row i + 1 go to all waves: through LDS inside one workgroup, or as 64-bit
//     words {value, column number} in memory between workgroups;
//   w = tau A v + K v, then A -= v w^T + w v^T, and row i + 1 likewise becomes the next x.
// The matrix takes two columns' updates at once (one rounding at its entries' size instead of
// two): at odd columns the products and row i + 1 lack the previous column's (vp, wp), which
// every wave adds itself, A v -= vp (wp . v) + wp (vp . v), while it waits for the exchange.
// So a column costs one exchange.  A reader of the words polls them until their column number is
// the one it needs: there is no flag to order against, no counter and no fence; both the words'
// stores and loads are relaxed agent-scope atomics (coherent across the XCDs).  The buffers
// alternate with the column's parity; a wave writes column i + 2's words only after its workgroup
// has read column i + 1's, which every workgroup published after reading column i's.  The words
// live in the strict upper triangle of the matrix (only the lower one is read), cleared before.
//
// Every wait is bounded; a workgroup that gives up leaves e[n-1] = NaN (otherwise 0), which the
// caller reports.  A matrix's workgroups have to run together: they are neighbours in the grid,
// which is dispatched in order, at most 32 per matrix, so the chip (256 workgroups at least)
// always holds whole matrices and the partial ones follow as those end.
// Whole spectrum of 4 cells, one workgroup per matrix with blocked updates -> this: T = 256 4.1 ->
// 2.5 ms, 522 10.7 -> 5.0 ms, 700 18.1 -> 6.9 ms; against the one-stage reduction of larger
// matrices T = 1001 21.1 -> 10.0 ms.  At n = 1300 the wave's registers spill and it loses (36 ms to
// 27), which ends its range.
#include <algorithm>

#include "common.h"
#include "kernels.h"

namespace {

constexpr int WORD_ROWS = 16;            // rows of A whose upper part holds the exchange words

// 64-bit word e of a matrix's exchange area
JOLT_DEV uint64_t *word_at(float *A, int n, int e) {
  const int per = (n - 20) / 2, r = e / per, k = e - r * per;
  const int64_t o = (int64_t)r * n + 17;                  // columns > r for every r < 16
  return reinterpret_cast<uint64_t *>(A + (o + ((reinterpret_cast<uintptr_t>(A) >> 2) + o) % 2)) + k;
}

JOLT_DEV void word_put(uint64_t *p, float v, uint32_t tag) {
  uint32_t u = __float_as_uint(v);
  asm volatile("" : "+v"(u));              // a copy: v itself stays a 32-bit register
  __hip_atomic_store(p, ((uint64_t)tag << 32) | u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// sums over the wave, in every lane
template <int CTRL>
JOLT_DEV double dpp_f64(double v) {
  const uint64_t b = (uint64_t)__double_as_longlong(v);
  const uint32_t lo = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)b, CTRL, 0xf, 0xf, false);
  const uint32_t hi = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)(b >> 32), CTRL, 0xf, 0xf, false);
  return __longlong_as_double((long long)(((uint64_t)hi << 32) | lo));
}
JOLT_DEV double lane_f64(double v, int l) {
  const uint64_t b = (uint64_t)__double_as_longlong(v);
  const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)b, l);
  const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(b >> 32), l);
  return __longlong_as_double((long long)(((uint64_t)hi << 32) | lo));
}
JOLT_DEV double wave_sum_dpp(double v) {
  v += dpp_f64<0x128>(v); v += dpp_f64<0x124>(v); v += dpp_f64<0x122>(v); v += dpp_f64<0x121>(v);
  return (lane_f64(v, 0) + lane_f64(v, 16)) + (lane_f64(v, 32) + lane_f64(v, 48));
}
JOLT_DEV float row_sum16(float v) {
  v += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x128, 0xf, 0xf, false));
  v += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x124, 0xf, 0xf, false));
  v += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x122, 0xf, 0xf, false));
  v += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x121, 0xf, 0xf, false));
  return v;
}
JOLT_DEV float lane_of(float x, int l) { return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(x), l)); }
JOLT_DEV float wave_sum_f32(float v) {
  v = row_sum16(v);
  return (lane_of(v, 0) + lane_of(v, 16)) + (lane_of(v, 32) + lane_of(v, 48));
}
// a in lanes 0 .. 31, b in lanes 32 .. 63, each summed with its other half
JOLT_DEV float fold32(float a, float b) {
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(a), __float_as_uint(b), false, false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}
// a in the even rows of 16 lanes, b in the odd ones, each summed with its neighbour row
JOLT_DEV float fold16(float a, float b) {
  const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(a), __float_as_uint(b), false, false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}

// CC: columns per lane (n <= 64 CC); TW: waves per matrix; RW: rows per wave (n <= TW RW);
// NW: waves per workgroup (TW / NW workgroups per matrix)
template <int CC, int TW, int RW, int NW>
__global__ void __launch_bounds__(NW * 64, 1) k_trd_reg(EigBatch b, int mat0, int spin_max) {
  constexpr int P = TW / NW, RP = (RW + 3) / 4 * 4;
  const int mat = mat0 + blockIdx.x / P, part = blockIdx.x % P, n = b.n;
  float *A = b.A + (int64_t)mat * b.mat_stride;
  double *dd = b.d + (int64_t)mat * n, *ee = b.e + (int64_t)mat * n;
  float *tau = b.tau + (int64_t)mat * n;
  const int tid = threadIdx.x, lane0 = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), rho = part * NW + wave;
  int lane = lane0;
  __shared__ float ex[2][2][64 * CC];    // [parity][products, row i + 1][column]
  __shared__ int give_up;
  if (tid == 0) give_up = 0;

  // rows TW j + rho; entries past n are zero
  float a[RW][CC], x[CC];
#pragma unroll
  for (int j = 0; j < RW; ++j) {
    const int r = TW * j + rho;
#pragma unroll
    for (int c = 0; c < CC; ++c) {
      const int col = 64 * c + lane, hi = max(r, col), lo = min(r, col);
      const float t = A[(uint32_t)(min(hi, n - 1) * n + min(lo, n - 1))];
      a[j][c] = hi < n ? t : 0.f;
      if (c % 8 == 7) __builtin_amdgcn_sched_barrier(0);      // bounds the addresses in flight
    }
    __builtin_amdgcn_sched_barrier(0);
  }
#pragma unroll
  for (int c = 0; c < CC; ++c) x[c] = 64 * c + lane < n ? A[(uint32_t)((64 * c + lane) * n)] : 0.f;
  __syncthreads();

  float vp[CC], wp[CC];                  // the previous column's update, pending at odd columns
#pragma unroll
  for (int c = 0; c < CC; ++c) { vp[c] = 0.f; wp[c] = 0.f; }
  // the workgroup's last row
  int last_row = 0;
  for (int u = 0; u < NW; ++u) {
    const int q = part * NW + u;
    if (q < n) last_row = max(last_row, (n - 1 - q) / TW * TW + q);
  }
  // entry of the wave's row j in a vector held by columns
  auto row_value = [&](const float (&u)[CC], int j) -> float {
    if constexpr (TW <= 64) {
      constexpr int per = TW <= 64 ? 64 / TW : 1;           // rows of the wave in 64 columns
      return lane_of(u[j / per], TW * (j % per) + rho);
    } else {
      constexpr int step = TW / 64;                          // it lies in chunk step j + rho / 64
      float t = u[min(step * j, CC - 1)];
#pragma unroll
      for (int k = 1; k < step; ++k) t = k == (rho >> 6) ? u[min(step * j + k, CC - 1)] : t;
      return lane_of(t, rho & 63);
    }
  };
  bool dead = false, leave = false;
  for (int i = 0; i < n - 1; ++i) {
    const int par = i & 1, i1 = i + 1, c1 = i1 >> 6, l1 = i1 & 63;
    // hides that the lane is the same in every iteration: addresses and masks are formed where
    // they are used instead of being kept in registers across the loop
    asm volatile("" : "+v"(lane));
    // ---- reflector from x
    double s2 = 0.0;
    float al = 0.f, di = 0.f;
#pragma unroll
    for (int c = 0; c < CC; ++c) {
      const int col = 64 * c + lane;
      if (col > i1) s2 = fma((double)x[c], (double)x[c], s2);
      if (c == c1) al = lane_of(x[c], l1);
      if (c == (i >> 6)) di = lane_of(x[c], i & 63);
    }
    const double sigma = wave_sum_dpp(s2), alpha = al;
    double beta = alpha, tv = 0.0, scal = 0.0;
    if (sigma != 0.0) {
      beta = -copysign(sqrt(fma(alpha, alpha, sigma)), alpha);
      tv = (beta - alpha) * recip2(beta);
      scal = recip2(alpha - beta);
    }
    float v[CC];
#pragma unroll
    for (int c = 0; c < CC; ++c) {
      const int col = 64 * c + lane;
      asm volatile("" : "+v"(x[c]));       // its fp64 value is formed again, not kept from the sum
      v[c] = col == i1 ? 1.f : (col > i1 ? (float)((double)x[c] * scal) : 0.f);
    }
    // ---- products of the wave's rows
    float s[RP];
#pragma unroll
    for (int j = 0; j < RP; ++j) s[j] = 0.f;
#pragma unroll
    for (int c = 0; c < CC; ++c)
      if (c >= c1) {                       // v is zero in the columns before
#pragma unroll
        for (int j = 0; j < RW; ++j) s[j] = fmaf(a[j][c], v[c], s[j]);
      }
    const uint32_t tag = (uint32_t)i1;
#pragma unroll
    for (int q = 0; q < RP / 4; ++q) {
      // rows q, q + RP/4, q + RP/2, q + 3 RP/4 end in lane rows 0, 1, 2, 3
      const float f = row_sum16(fold16(fold32(s[q], s[q + RP / 2]), fold32(s[q + RP / 4], s[q + 3 * RP / 4])));
      const int j = q + (RP / 4) * (lane >> 4), r = TW * j + rho;
      if ((lane & 15) == 0 && j < RW && r > i && r < n) {
        if constexpr (P == 1) ex[par][0][r] = f;
        else word_put(word_at(A, n, par * 2 * n + r), f, tag);
      }
    }
    if (rho == i1 % TW) {
#pragma unroll
      for (int j = 0; j < RW; ++j)
        if (j == i1 / TW) {
#pragma unroll
          for (int c = 0; c < CC; ++c) {
            const int col = 64 * c + lane;
            if (c >= c1 && col < n) {
              if constexpr (P == 1) ex[par][1][col] = a[j][c];
              else word_put(word_at(A, n, (par * 2 + 1) * n + col), a[j][c], tag);
            }
          }
        }
    }
    // ---- what the pending update adds to the products (0 at even columns)
    float pv = 0.f, pw = 0.f, vp1 = 0.f, wp1 = 0.f;
#pragma unroll
    for (int c = 0; c < CC; ++c) {
      pv = fmaf(vp[c], v[c], pv);
      pw = fmaf(wp[c], v[c], pw);
      if (c == c1) { vp1 = lane_of(vp[c], l1); wp1 = lane_of(wp[c], l1); }
    }
    pv = wave_sum_f32(pv);
    pw = wave_sum_f32(pw);
    if constexpr (P > 1) leave = last_row <= i1 && last_row != n - 1;
    if (P > 1 && !leave) {
      // the workgroup's waves share out the chunks of 64 words from column i + 1 on; a wave's
      // chunks are polled together
      constexpr int NQ = (2 * CC + NW - 1) / NW;
      uint64_t wd[NQ];
      bool ok[NQ];
#pragma unroll
      for (int k = 0; k < NQ; ++k) {
        const int q = wave + NW * k, col = 64 * (q >> 1) + lane;
        ok[k] = !(q < 2 * CC && col > i && col < n);
        wd[k] = 0;
      }
      for (int spins = 0;; ++spins) {
#pragma unroll
        for (int k = 0; k < NQ; ++k) {
          const int q = wave + NW * k, col = 64 * (q >> 1) + lane;
          if (!ok[k]) wd[k] = __hip_atomic_load(word_at(A, n, (par * 2 + (q & 1)) * n + col), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
        bool all = true;
#pragma unroll
        for (int k = 0; k < NQ; ++k) {
          ok[k] = ok[k] || (uint32_t)(wd[k] >> 32) == tag;
          all = all && ok[k];
        }
        if (__all(all)) break;
        if (spins >= spin_max) { give_up = 1; break; }
      }
#pragma unroll
      for (int k = 0; k < NQ; ++k) {
        const int q = wave + NW * k, col = 64 * (q >> 1) + lane;
        if (q < 2 * CC) ex[par][q & 1][col] = __uint_as_float((uint32_t)wd[k]);
      }
    }
    __syncthreads();
    if constexpr (P > 1) {
      dead = give_up != 0;
      if (dead) break;
    }
    // ---- outputs of the column, from the wave that owns row i + 1 (every wave has read its rows:
    // column 0's words have come from all of them)
    if (rho == i1 % TW) {
#pragma unroll
      for (int c = 0; c < CC; ++c) {
        const int col = 64 * c + lane;
        if (col > i && col < n) A[(uint32_t)(col * n + i)] = v[c];
      }
      if (lane == 0) { dd[i] = (double)di; ee[i] = beta; tau[i] = (float)tv; }
    }
    if (P > 1 && leave) return;
    // ---- w = tau A v + K v
    const float tf = (float)tv;
    float w[CC], y[CC];
    double vw = 0.0;
#pragma unroll
    for (int c = 0; c < CC; ++c) {
      w[c] = 0.f; y[c] = 0.f;
      if (c >= c1) {
        const int col = 64 * c + lane;
        const bool in = col > i && col < n;
        w[c] = in ? tf * (ex[par][0][col] - fmaf(vp[c], pw, wp[c] * pv)) : 0.f;
        y[c] = in ? ex[par][1][col] - fmaf(vp1, wp[c], wp1 * vp[c]) : 0.f;
        vw = fma((double)w[c], (double)v[c], vw);
      }
    }
    const float K = (float)(-0.5 * tv * wave_sum_dpp(vw));
    float w1 = 0.f;
#pragma unroll
    for (int c = 0; c < CC; ++c) {
      w[c] = fmaf(K, v[c], w[c]);
      if (c == c1) w1 = lane_of(w[c], l1);
    }
    // ---- the next x, and the rank-2 update of the wave's rows
#pragma unroll
    for (int c = 0; c < CC; ++c) x[c] = y[c] - fmaf(w1, v[c], w[c]);
    if (!(i & 1)) {
#pragma unroll
      for (int c = 0; c < CC; ++c) { vp[c] = v[c]; wp[c] = w[c]; }
      continue;
    }
#pragma unroll
    for (int j = 0; j < RW; ++j) {
      const float vr = row_value(v, j), wr = row_value(w, j), vpr = row_value(vp, j), wpr = row_value(wp, j);
#pragma unroll
      for (int c = 0; c < CC; ++c)
        if (c >= c1) a[j][c] -= fmaf(vr, w[c], fmaf(wr, v[c], fmaf(vpr, wp[c], wpr * vp[c])));
    }
#pragma unroll
    for (int c = 0; c < CC; ++c) { vp[c] = 0.f; wp[c] = 0.f; }
  }
  if (dead) {
    if (tid == 0) ee[n - 1] = __builtin_nan("");
    return;
  }
  if (rho == (n - 1) % TW) {
    float dl = 0.f;
#pragma unroll
    for (int c = 0; c < CC; ++c)
      if (c == (n - 1) >> 6) dl = lane_of(x[c], (n - 1) & 63);
    if (lane == 0) { dd[n - 1] = (double)dl; ee[n - 1] = 0.0; tau[n - 1] = 0.f; }
  }
}

// before: the exchange words cleared; after: the upper triangle, the diagonal and the last
// column zeroed (the dense V that the blocked back-transform multiplies by)
__global__ void k_trd_words_clear(EigBatch b) {
  float *A = b.A + (int64_t)blockIdx.y * b.mat_stride;
  for (int e = blockIdx.x * 256 + threadIdx.x; e < 4 * b.n; e += gridDim.x * 256)
    __hip_atomic_store(word_at(A, b.n, e), (uint64_t)0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__global__ void k_trd_clean(EigBatch b) {
  float *A = b.A + (int64_t)blockIdx.y * b.mat_stride;
  const int n = b.n;
  for (int r = blockIdx.x; r < n; r += gridDim.x)
    for (int c = threadIdx.x; c < n; c += 256)
      if (c >= r || c == n - 1) A[(int64_t)r * n + c] = 0.f;
}

template <int CC, int TW, int RW, int NW>
hipError_t launch_reg(const EigBatch &b, int spin_max, hipStream_t st) {
  static_assert(TW % NW == 0 && (TW / NW == 1 || TW >= 64), "waves per matrix");
  constexpr int P = TW / NW;
  if (b.n > 64 * CC || b.n > TW * RW) return hipErrorInvalidValue;
  if (P > 1) hipLaunchKernelGGL(k_trd_words_clear, dim3((4 * b.n + 255) / 256, b.n_mat), dim3(256), 0, st, b);
  hipLaunchKernelGGL((k_trd_reg<CC, TW, RW, NW>), dim3(b.n_mat * P), dim3(NW * 64), 0, st, b, 0, spin_max);
  hipLaunchKernelGGL(k_trd_clean, dim3(std::min(b.n, 256), b.n_mat), dim3(256), 0, st, b);
  return hipGetLastError();
}

}  // namespace

int trd_reg_workgroups(int n) { return n <= 256 ? 1 : n <= 576 ? 8 : n <= 768 ? 16 : 32; }

hipError_t launch_trd_reg(const EigBatch &b, int spin_max, hipStream_t st) {
  const int n = b.n, spin = std::max(spin_max, 0);
  if (n < 1 || n > TRD_REG_MAX) return hipErrorInvalidValue;
  // up to n = 256 one workgroup (an exchange between workgroups costs what its compute does)
  if (n <= 64) return launch_reg<1, 8, 8, 8>(b, spin, st);
  if (n <= 128) return launch_reg<2, 8, 16, 8>(b, spin, st);
  if (n <= 256) return launch_reg<4, 16, 16, 16>(b, spin, st);
  if (n <= 384) return launch_reg<6, 64, 6, 8>(b, spin, st);
  if (n <= 576) return launch_reg<9, 64, 9, 8>(b, spin, st);
  if (n <= 768) return launch_reg<12, 128, 6, 8>(b, spin, st);
  return launch_reg<16, 256, 4, 8>(b, spin, st);
}
