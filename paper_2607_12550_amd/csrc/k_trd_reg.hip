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
// A matrix is reduced in registers only once all its workgroups are running: they draw (matrix,
// part) from the launch's ticket, in order, count themselves in at the matrix's gather word, load
// their rows and wait until the count is complete.  From there on no wait depends on anything that
// is not running.  A workgroup whose gather wait runs out marks the matrix as left (only while the
// count is incomplete, so all its workgroups agree), nothing has been written yet, and the
// one-workgroup reduction behind this kernel takes it.  Kernels of other streams, contexts or
// processes that hold the chip can therefore delay a reduction but not stop it, however the
// workgroups are dispatched: by the ticket a launch has at most one incomplete matrix, whose up to
// 31 waiting workgroups give their places back.  (With (matrix, part) from the block index two
// launches could hold one XCD each with workgroups that waited for the other's; drawing them costs
// 0.2 of 6.9 ms at n = 1001, 0.2 of 4.6 ms for 16 matrices of order 700, nothing up to 576: the
// parts of a matrix are then spread less evenly over the XCDs.)  A second bound (spin_max) ends the
// exchange's own waits; a workgroup that gives up there marks its matrix in b.gave_up, which the
// caller reports.
// Whole spectrum of 4 cells, one workgroup per matrix with blocked updates -> this: T = 256 4.1 ->
// 2.5 ms, 522 10.7 -> 5.0 ms, 700 18.1 -> 6.9 ms; against the one-stage reduction of larger
// matrices T = 1001 21.1 -> 10.0 ms.  At n = 1300 the wave's registers spill and it loses (36 ms to
// 27), which ends its range.
#include <algorithm>

#include "common.h"
#include "kernels.h"

namespace {

// 64-bit word e of a matrix's exchange area, the upper part of its first 16 rows (8 n - 160 words or
// more, of which 4 n + 2 are used, n > 256)
JOLT_DEV uint64_t *word_at(float *A, int n, int e) {
  const int per = (n - 20) / 2, r = e / per, k = e - r * per;
  const int64_t o = (int64_t)r * n + 17;                  // columns > r for every r < 16
  return reinterpret_cast<uint64_t *>(A + (o + ((reinterpret_cast<uintptr_t>(A) >> 2) + o) % 2)) + k;
}

// the matrix's gather word: workgroups counted in, and whether it is left to one workgroup; the
// launch's ticket is a word of its first matrix
constexpr uint32_t TRD_LEFT = 1u << 16;
JOLT_DEV uint32_t *gather_word(float *A, int n) { return reinterpret_cast<uint32_t *>(word_at(A, n, 4 * n)); }
JOLT_DEV uint32_t *ticket_word(float *A, int n) { return reinterpret_cast<uint32_t *>(word_at(A, n, 4 * n + 1)); }

// waits until all `parts` workgroups of the matrix are counted in; false: the matrix is left.  A
// bound of 0 leaves every matrix (each workgroup marks it before it counts itself in).
JOLT_DEV bool gather_wait(uint32_t *word, int parts, int polls_max) {
  for (int polls = 0;; ++polls) {
    uint32_t w = __hip_atomic_load(word, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (w & TRD_LEFT) return false;
    if (w == (uint32_t)parts) return true;
    // fails, and the loop goes on, if another workgroup counted itself in meanwhile
    if (polls >= polls_max &&
        __hip_atomic_compare_exchange_strong(word, &w, w | TRD_LEFT, __ATOMIC_RELAXED, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT))
      return false;
    __builtin_amdgcn_s_sleep(8);
  }
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
__global__ void __launch_bounds__(NW * 64, 1) k_trd_reg(EigBatch b, int gather_max, int spin_max) {
  constexpr int P = TW / NW, RP = (RW + 3) / 4 * 4;
  const int tid = threadIdx.x, n = b.n;
  int job = blockIdx.x;
  __shared__ int head, give_up;          // head: the job drawn, then whether its matrix is left
  if (tid == 0) give_up = 0;
  if constexpr (P > 1) {
    if (tid == 0) {
      const int j = (int)__hip_atomic_fetch_add(ticket_word(b.A, n), 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      uint32_t *word = gather_word(b.A + (int64_t)(j / P) * b.mat_stride, n);
      if (gather_max == 0) __hip_atomic_fetch_or(word, TRD_LEFT, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      __hip_atomic_fetch_add(word, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      head = j;
    }
    __syncthreads();
    job = __builtin_amdgcn_readfirstlane(head);
  }
  const int mat = job / P, part = job % P;
  float *A = b.A + (int64_t)mat * b.mat_stride;
  double *dd = b.d + (int64_t)mat * n, *ee = b.e + (int64_t)mat * n;
  float *tau = b.tau + (int64_t)mat * n;
  const int lane0 = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), rho = part * NW + wave;
  int lane = lane0;
  __shared__ float ex[2][2][64 * CC];    // [parity][products, row i + 1][column]

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
  if constexpr (P > 1) {
    __syncthreads();                     // every wave has read the job
    if (tid == 0) head = gather_wait(gather_word(A, n), P, gather_max) ? 0 : 1;
  }
  __syncthreads();
  if constexpr (P > 1)
    if (head) return;

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
    if (tid == 0) b.gave_up[mat] = 1;
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

// before: the exchange, gather and ticket words cleared; after: the upper triangle, the diagonal and the last
// column zeroed (the dense V that the blocked back-transform multiplies by)
__global__ void k_trd_words_clear(EigBatch b) {
  float *A = b.A + (int64_t)blockIdx.y * b.mat_stride;
  if (blockIdx.x == 0 && threadIdx.x == 0) b.gave_up[blockIdx.y] = 0;
  for (int e = blockIdx.x * 256 + threadIdx.x; e < 4 * b.n + 2; e += gridDim.x * 256)
    __hip_atomic_store(word_at(A, b.n, e), (uint64_t)0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__global__ void k_trd_clean(EigBatch b) {
  float *A = b.A + (int64_t)blockIdx.y * b.mat_stride;
  const int n = b.n;
  for (int r = blockIdx.x; r < n; r += gridDim.x)
    for (int c = threadIdx.x; c < n; c += 256)
      if (c >= r || c == n - 1) A[(int64_t)r * n + c] = 0.f;
}

// Tridiagonalisation in one workgroup per matrix, the matrix in global memory (L2), for n <= 1024:
// large batches (both triangles of the input read), and what the register kernel leaves (left != 0:
// matrices marked in their gather word, of which only the lower triangle is read).  Writes d, e,
// tau and leaves v_i in column i of A (rows i+1..n-1, v_i(i+1) = 1) with zeros above, as the
// register kernel and the cleaning pass do.
//
// Blocked in panels of SB columns (the LAPACK latrd scheme inside one workgroup): the
// panel's reflectors V and the vectors W (A_i v_i corrected for the panel's earlier
// reflectors, then w += K v) are kept in LDS by absolute row.  Column i is brought up to
// date with the panel's earlier reflectors only when it becomes current; the mat-vec reads
// the trailing matrix as it was at the panel start and subtracts V (W^T v) + W (V^T v); the
// trailing matrix past the panel takes the rank-2 SB update once, at the panel end.  Each
// column then reads the trailing matrix once instead of three times (mat-vec, and the
// read and write of an immediate rank-2 update).
constexpr int SYTD2_THREADS = 1024;

// Workgroup sum with one barrier: successive calls alternate between two halves of red
// (2 x waves entries), so a call never overwrites values an earlier call is still reading.
JOLT_DEV double block_sum1(double v, double *red, int &flip) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, nw = blockDim.x >> 6;
  v = wave_sum(v);
  double *r = red + flip * nw;
  flip ^= 1;
  if (lane == 0) r[wave] = v;
  __syncthreads();
  double s = 0.0;
  for (int w = 0; w < nw; ++w) s += r[w];
  return s;
}

constexpr int SB = 16, SBL = SB + 1;     // panel width, LDS row stride of V and W

size_t sytd2_lds_bytes(int n) { return ((size_t)2 * n + (size_t)2 * n * SBL + 2 * SB) * sizeof(float); }

__global__ void __launch_bounds__(SYTD2_THREADS) k_sytd2(EigBatch b, int left) {
  const int mat = blockIdx.x, n = b.n;
  float *A = b.A + (int64_t)mat * b.mat_stride;
  if (left && !(*gather_word(A, n) & TRD_LEFT)) return;
  if (!left && threadIdx.x == 0) b.gave_up[mat] = 0;
  double *dd = b.d + (int64_t)mat * n, *ee = b.e + (int64_t)mat * n;
  float *tau = b.tau + (int64_t)mat * n;
  extern __shared__ float sh[];
  float *v = sh, *w = sh + n;
  float *Vp = w + n, *Wp = Vp + (size_t)n * SBL, *yv = Wp + (size_t)n * SBL;
  __shared__ double red[2 * (SYTD2_THREADS / 64)];
  __shared__ double s_alpha;                        // x[0] of the current column
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, nw = SYTD2_THREADS / 64;
  int flip = 0;
  if (left) {
    __syncthreads();                     // every thread has read the word
    for (int r = wave; r < n; r += nw)
      for (int c = lane; c < r; c += 64) A[(int64_t)c * n + r] = A[(int64_t)r * n + c];
    __syncthreads();
  }
  for (int k0 = 0; k0 < n - 1; k0 += SB) {
    const int jb = min(SB, n - 1 - k0);
    for (int q = tid; q < (n - k0) * SBL; q += SYTD2_THREADS) {
      Vp[(size_t)k0 * SBL + q] = 0.f;
      Wp[(size_t)k0 * SBL + q] = 0.f;
    }
    __syncthreads();
    for (int j = 0; j < jb; ++j) {
      const int i = k0 + j, L = n - 1 - i;
      // column i (rows i..n-1) brought up to date with reflectors k0 .. i-1; the squared
      // norm of x[1..] is accumulated on the way
      double part = 0.0;
      for (int r = i + tid; r < n; r += SYTD2_THREADS) {
        float a = A[(int64_t)r * n + i];
        for (int p = 0; p < j; ++p)
          a -= Vp[(size_t)r * SBL + p] * Wp[(size_t)i * SBL + p] + Wp[(size_t)r * SBL + p] * Vp[(size_t)i * SBL + p];
        if (r == i) A[(int64_t)i * n + i] = a;
        else v[r - i - 1] = a;
        if (r == i + 1) s_alpha = a;
        if (r > i + 1) part += (double)a * (double)a;
      }
      // its barrier also publishes v and x[0]; v[0] is overwritten below, so x[0] is read
      // from its own copy (rewritten only after two more barriers)
      const double sigma = block_sum1(part, red, flip);
      const double alpha = s_alpha;
      double beta, tv, scal;
      if (sigma == 0.0) {
        tv = 0.0; beta = alpha; scal = 0.0;
      } else {
        beta = -copysign(sqrt(alpha * alpha + sigma), alpha);
        tv = (beta - alpha) / beta;
        scal = 1.0 / (alpha - beta);
      }
      // v = x scaled (v[0] = 1); every entry has one owner in this loop
      for (int r = i + 1 + tid; r < n; r += SYTD2_THREADS) {
        const int t = r - i - 1;
        float vt = (t == 0) ? 1.f : (float)((double)v[t] * scal);
        if (tv == 0.0) vt = (t == 0) ? 1.f : 0.f;
        v[t] = vt;
        A[(int64_t)r * n + i] = vt;
        Vp[(size_t)r * SBL + j] = vt;
      }
      if (tid == 0) { ee[i] = beta; tau[i] = (float)tv; }
      __syncthreads();
      if (tv == 0.0) continue;                     // W column stays zero
      const float tf = (float)tv;
      // w' = A22 v over the trailing matrix as of the panel start: a wavefront takes four
      // rows at a time (rows r, r + nw, r + 2 nw, r + 3 nw) so that their loads are in
      // flight together; rows past L read row L - 1 and are not stored
      for (int r0 = wave; r0 < L; r0 += 4 * nw) {
        const float *row[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) row[u] = A + (int64_t)(i + 1 + min(r0 + u * nw, L - 1)) * n + (i + 1);
        float sacc[4] = {0.f, 0.f, 0.f, 0.f};
        for (int c = lane; c < L; c += 64) {
          float x[4];
#pragma unroll
          for (int u = 0; u < 4; ++u) x[u] = row[u][c];
          const float vc = v[c];
#pragma unroll
          for (int u = 0; u < 4; ++u) sacc[u] = fmaf(x[u], vc, sacc[u]);
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          const float su = wave_sum(sacc[u]);
          if (lane == 0 && r0 + u * nw < L) w[r0 + u * nw] = su;
        }
      }
      // yv = [W^T v ; V^T v] over rows i+1.. for the panel's earlier reflectors
      for (int q = wave; q < 2 * j; q += nw) {
        const float *col = (q < j ? Wp : Vp) + (q < j ? q : q - j);
        float sacc = 0.f;
        for (int t = lane; t < L; t += 64) sacc = fmaf(col[(size_t)(i + 1 + t) * SBL], v[t], sacc);
        sacc = wave_sum(sacc);
        if (lane == 0) yv[q < j ? q : SB + q - j] = sacc;
      }
      __syncthreads();
      // corrected w = tau (w' - V yv_W - W yv_V), kept in a register by the thread that owns
      // row t, and its dot with v for K
      part = 0.0;
      float wt[(1024 + SYTD2_THREADS - 1) / SYTD2_THREADS];
#pragma unroll
      for (int u = 0; u < (int)(sizeof(wt) / sizeof(float)); ++u) {
        const int t = tid + u * SYTD2_THREADS;
        wt[u] = 0.f;
        if (t < L) {
          float c = w[t];
          const size_t rr = (size_t)(i + 1 + t) * SBL;
          for (int p = 0; p < j; ++p) c -= Vp[rr + p] * yv[p] + Wp[rr + p] * yv[SB + p];
          wt[u] = tf * c;
          part += (double)wt[u] * (double)v[t];
        }
      }
      const float K = (float)(-0.5 * tv * block_sum1(part, red, flip));
#pragma unroll
      for (int u = 0; u < (int)(sizeof(wt) / sizeof(float)); ++u) {
        const int t = tid + u * SYTD2_THREADS;
        if (t < L) Wp[(size_t)(i + 1 + t) * SBL + j] = fmaf(K, v[t], wt[u]);
      }
      __syncthreads();
    }
    // trailing matrix past the panel: A -= V W^T + W V^T (both triangles)
    const int s0 = k0 + jb;
    for (int r = s0 + wave; r < n; r += nw) {
      float vr[SB], wr[SB];
#pragma unroll
      for (int p = 0; p < SB; ++p) { vr[p] = Vp[(size_t)r * SBL + p]; wr[p] = Wp[(size_t)r * SBL + p]; }
      float *row = A + (int64_t)r * n;
      for (int c = s0 + lane; c < n; c += 64) {
        float acc = 0.f;
#pragma unroll
        for (int p = 0; p < SB; ++p) acc = fmaf(vr[p], Wp[(size_t)c * SBL + p], fmaf(wr[p], Vp[(size_t)c * SBL + p], acc));
        row[c] -= acc;
      }
    }
    __syncthreads();
  }
  // diagonal of T, then zero the strictly upper part and diagonal of the reflector block
  for (int i = tid; i < n; i += SYTD2_THREADS) dd[i] = A[(int64_t)i * n + i];
  if (tid == 0) { ee[n - 1] = 0.0; tau[n - 1] = 0.f; }
  __syncthreads();
  for (int r = wave; r < n; r += nw) {
    float *row = A + (int64_t)r * n;
    for (int c = lane; c < n; c += 64)
      if (c >= r || c == n - 1) row[c] = 0.f;
  }
  if (n == 1 && tid == 0) A[0] = 0.f;
}

hipError_t launch_sytd2(const EigBatch &b, int left, hipStream_t st) {
  if (b.n > SYTD2_THREADS) return hipErrorInvalidValue;   // one corrected w entry per thread
  const size_t shm = sytd2_lds_bytes(b.n);
  if (shm > 65536) {
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(&k_sytd2),
                                       hipFuncAttributeMaxDynamicSharedMemorySize,
                                       (int)sytd2_lds_bytes(SYTD2_THREADS));
    if (e != hipSuccess) return e;
  }
  hipLaunchKernelGGL(k_sytd2, dim3(b.n_mat), dim3(SYTD2_THREADS), shm, st, b, left);
  return hipGetLastError();
}

template <int CC, int TW, int RW, int NW>
hipError_t launch_reg(const EigBatch &b, int gather_max, int spin_max, hipStream_t st) {
  static_assert(TW % NW == 0 && (TW / NW == 1 || TW >= 64), "waves per matrix");
  constexpr int P = TW / NW;
  if (b.n > 64 * CC || b.n > TW * RW) return hipErrorInvalidValue;
  if (P > 1) hipLaunchKernelGGL(k_trd_words_clear, dim3((4 * b.n + 257) / 256, b.n_mat), dim3(256), 0, st, b);
  hipLaunchKernelGGL((k_trd_reg<CC, TW, RW, NW>), dim3(b.n_mat * P), dim3(NW * 64), 0, st, b, gather_max, spin_max);
  if (P > 1) {
    const hipError_t e = launch_sytd2(b, 1, st);
    if (e != hipSuccess) return e;
  }
  hipLaunchKernelGGL(k_trd_clean, dim3(std::min(b.n, 256), b.n_mat), dim3(256), 0, st, b);
  return hipGetLastError();
}

}  // namespace

int trd_reg_workgroups(int n) { return n <= 256 ? 1 : n <= 576 ? 8 : n <= 768 ? 16 : 32; }

hipError_t launch_trd_reg(const EigBatch &b, int gather_max, int spin_max, hipStream_t st) {
  const int n = b.n, spin = std::max(spin_max, 0), gather = std::max(gather_max, 0);
  if (n < 1 || n > TRD_REG_MAX) return hipErrorInvalidValue;
  // up to n = 256 one workgroup (an exchange between workgroups costs what its compute does)
  if (n <= 64) return launch_reg<1, 8, 8, 8>(b, gather, spin, st);
  if (n <= 128) return launch_reg<2, 8, 16, 8>(b, gather, spin, st);
  if (n <= 256) return launch_reg<4, 16, 16, 16>(b, gather, spin, st);
  // A round is the workgroups that run at once (two a CU up to n = 384, else one).  Batches of more
  // rounds than n / 160 go to one workgroup per matrix, which takes 256 matrices a round; whole
  // spectrum in registers to one workgroup each, ms (at the line's two sides):
  //   n = 257: 64 matrices (1 round) 2.6 to 3.6, 96 (2) 3.9 to 3.8; 384: 128 (2) 6.1 to 7.2, 160 (3) 8.4 to 7.9;
  //   n = 385: 64 (2) 5.7 to 6.6, 96 (3) 8.0 to 7.1; 522: 96 (3) 11.4 to 13.7, 128 (4) 14.5 to 13.9;
  //   n = 577: 48 (3) 13.1 to 14.9, 64 (4) 16.8 to 15.5; 768: 64 (4) 22.2 to 30.0, 96 (6) 33.6 to 32.1
  const int64_t round = n <= 384 ? 512 : 256;
  if (n <= 768 && ((int64_t)b.n_mat * trd_reg_workgroups(n) + round - 1) / round > n / 160) return launch_sytd2(b, 0, st);
  if (n <= 384) return launch_reg<6, 64, 6, 8>(b, gather, spin, st);
  if (n <= 576) return launch_reg<9, 64, 9, 8>(b, gather, spin, st);
  if (n <= 768) return launch_reg<12, 128, 6, 8>(b, gather, spin, st);
  return launch_reg<16, 256, 4, 8>(b, gather, spin, st);
}
