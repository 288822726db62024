// Householder reduction of a symmetric fp64 matrix to tridiagonal form in one
// launch, the matrix held in registers across the compute units.
//
// A launch per step and column (eig.hip) costs two launches of 5 to 8 us per
// column, most of it launch gaps, load latency and re-reading the trailing
// rows: 1.0 ms at n = 128, 8.0 ms at 768 and 28.9 ms at 2048, against 0.27,
// 1.9 and 6.4 ms here.
// Here each of ceil(n / 8) workgroups keeps eight rows in registers for the
// whole reduction (n = 2048: 128 KiB on each of 256 compute units), applies
// every rank-2 update to them at once, and one exchange per column is all
// that crosses compute units.  With x = row i right of its diagonal, alpha =
// x_{i+1}, x' = x without that entry and the reflector v = (1, x' sc), sc =
// 1 / (alpha - beta), every workgroup publishes, for each of its rows r,
// q_r = A_r . x' and a_r = A[r][i+1], and reads everybody's.  A v = sc q + a
// and, by symmetry, a is the next column, so every workgroup forms by itself
//     p = sc q + a,   w = tau p - (tau^2 (p . v) / 2) v,   A -= v w^T + w v^T,
//     row i+1 of the updated matrix = a - v w_{i+1} - w v_{i+1}.
// beta and its divisions run while the exchange is under way.  What bounds it
// now is the exchange (a store and a load through the memory side, about a
// microsecond) and two sums over the workgroup per column.  Every word of
// the exchange is read once per workgroup: letting each wave read what it
// needs by itself (p . v as parts of the workgroups, one barrier less) made
// all waves of all compute units queue for the same lines (7.4 instead of
// 3.1 us per column at n = 2048).
//
// The exchange carries its own flags: the 128 bits of (q_r, a_r) travel as
// three 64-bit words of 43 payload bits and the step's number in the upper
// 21, each written and read by a relaxed device-scope atomic, so a reader
// polls the data itself and needs no ordering between words.  Two slots
// alternate, and a workgroup whose rows are done publishes its last words and
// leaves without reading anybody's: tridiag_steps.hpp has the rules and why two
// slots are enough.  All workgroups must be resident together: the launch is
// cooperative, and a reader gives up after poll_limit polls (*err; the caller
// then takes the other reduction), so every workgroup ends.
#include <algorithm>
#include <cmath>

#include "bitsmoe.h"
#include "common.hpp"
#include "eig_wave.hpp"
#include "internal.hpp"
#include "tridiag_steps.hpp"

namespace bitsmoe {
namespace {

constexpr int kRows = kTridiagRows;
constexpr int kMaxSize = 2048;  // largest n (thread t owns columns t, t + threads, ...)

constexpr uint64_t kMask43 = (uint64_t{1} << 43) - 1;

// Clears the exchange slots and the error flag.
__global__ __launch_bounds__(256) void tridiag_clear_kernel(uint64_t* __restrict__ ex, int words,
                                                            int* __restrict__ err) {
  const int i = static_cast<int>(blockIdx.x) * 256 + threadIdx.x;
  if (i < words) ex[i] = 0;
  if (i == 0) *err = 0;
}

__device__ __forceinline__ uint64_t load_word(const uint64_t* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void store_word(uint64_t* p, uint64_t v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// The double whose low 43 bits are in w0 and whose high 21 are in the low
// bits of w1, and the one in the upper 22 payload bits of w1 and in w2.
__device__ __forceinline__ double first_f64(uint64_t w0, uint64_t w1) {
  return __builtin_bit_cast(double, (w0 & kMask43) | (w1 << 43));
}
__device__ __forceinline__ double second_f64(uint64_t w1, uint64_t w2) {
  return __builtin_bit_cast(double, ((w1 & kMask43) >> 21) | (w2 << 22));
}

// d [n], e [n-1], tau [n-1] and the reflectors by rows: V[i][c] = 0 for
// c <= i, 1 at i + 1, v_c beyond (row n - 1 of V is not written right of its
// diagonal; it holds no reflector).  CPT kThreads >= n, gridDim.x =
// ceil(n / kRows).
template <int kThreads, int CPT>
__global__ __launch_bounds__(kThreads) void tridiag_kernel(
    const double* __restrict__ M, int n, double* __restrict__ V, double* __restrict__ dvec,
    double* __restrict__ evec, double* __restrict__ tau, uint64_t* __restrict__ ex,
    int* __restrict__ err, int poll_limit) {
  constexpr int W = kThreads / 64;
  // sums over the waves; this workgroup's products and column entries (the
  // latter by the step's parity: they are read while the next step's are
  // written); q, a at column i + 1 and q, a, v at column i + 2
  __shared__ __align__(16) double red_g[W], red_s[W], part[kRows][W], s_q[kRows], s_a[2][kRows], s_c[6];
  __shared__ int s_abort;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int r0 = static_cast<int>(blockIdx.x) * kRows;
  const bool last = blockIdx.x == gridDim.x - 1;
  static_assert((W == 4 || W == 8) && kRows == 8, "four or eight waves, eight rows");
  auto sumw = [](const double* q) {
    const double s = (q[0] + q[1]) + (q[2] + q[3]);
    return W == 4 ? s : s + ((q[W - 4] + q[W - 3]) + (q[W - 2] + q[W - 1]));
  };

  // The reflector v and vector w of the previous column (whose rank-2 update
  // is pending) and the current row x, at this thread's columns, and at this
  // workgroup's rows: lane q < kRows of every wave holds row r0 + q.
  double A[kRows][CPT], v[CPT], w[CPT], x[CPT], vl = 0.0, wl = 0.0, xl;
  const int rl = r0 + (lane & 7);
#pragma unroll
  for (int k = 0; k < CPT; ++k) {
    const int c = tid + kThreads * k;
    v[k] = w[k] = 0.0;
    x[k] = c > 0 && c < n ? M[c] : 0.0;  // row 0
#pragma unroll
    for (int q = 0; q < kRows; ++q)
      A[q][k] = r0 + q < n && c < n ? M[static_cast<int64_t>(r0 + q) * n + c] : 0.0;
  }
  xl = rl > 0 && rl < n ? M[rl] : 0.0;
#pragma unroll
  for (int q = 0; q < kRows; ++q) {
    const int r = r0 + q;
    if (r < n)
      for (int c = tid; c <= r; c += kThreads) V[static_cast<int64_t>(r) * n + c] = 0.0;
  }
  if (tid == 0) s_abort = 0;
  double dcur = M[0], alpha = M[1];
  __syncthreads();

  for (int i = 0; i + 1 < n; ++i) {
    const int kmin = (i + 1) / kThreads;  // columns below kmin kThreads are done
    const int to = (i + 1) % kThreads;    // thread (and k = kmin) of column i + 1
    double* sa = s_a[i & 1];
    // the pending rank-2 update, A x' and |x'|^2
    double acc[kRows], vr[kRows], wr[kRows], sg = 0.0;
#pragma unroll
    for (int q = 0; q < kRows; ++q) {
      vr[q] = readlane_f64(vl, q);
      wr[q] = readlane_f64(wl, q);
      acc[q] = 0.0;
    }
#pragma unroll
    for (int k = 0; k < CPT; ++k) {
      if (k < kmin) continue;
      const double xk = tid + kThreads * k > i + 1 ? x[k] : 0.0;
      sg = fma(xk, xk, sg);
#pragma unroll
      for (int q = 0; q < kRows; ++q) {
        A[q][k] = fma(-vr[q], w[k], fma(-wr[q], v[k], A[q][k]));
        acc[q] = fma(A[q][k], xk, acc[q]);
      }
      // column i + 1 of the workgroup's rows
      if (k == kmin && tid == to) {
#pragma unroll
        for (int q = 0; q < kRows; ++q) sa[q] = A[q][k];
      }
    }
    const double pw = wave_fold<kRows>(acc, lane);
    sg = wave_sum_dpp(sg);
    if ((lane & 7) == 0) part[lane >> 3][wave] = pw;
    if (lane == 0) red_g[wave] = sg;
    lds_barrier();
    const uint64_t epoch = static_cast<uint64_t>(i + 1) << 43;
    uint64_t* slot = ex + (i & 1) * 3 * n;
    if (wave == 0 && tridiag_exchanges(n, i)) {
      const double q = sumw(part[lane & 7]);
      const uint64_t P = __builtin_bit_cast(uint64_t, q);
      const uint64_t Q = __builtin_bit_cast(uint64_t, sa[lane & 7]);
      if (lane < kRows) {
        s_q[lane] = q;
        if (tridiag_word_live(n, i, rl)) {
          store_word(slot + rl, epoch | (P & kMask43));
          store_word(slot + n + rl, epoch | (P >> 43) | ((Q & ((uint64_t{1} << 22) - 1)) << 21));
          store_word(slot + 2 * n + rl, epoch | (Q >> 22));
        }
      }
    }
    // the reflector of row i
    const double sigma = sumw(red_g);
    double beta = alpha, t = 0.0, sc = 0.0;
    if (sigma != 0.0) {
      beta = -copysign(sqrt(fma(alpha, alpha, sigma)), alpha);
      t = (beta - alpha) / beta;
      sc = 1.0 / (alpha - beta);
    }
    vl = rl > i + 1 ? xl * sc : (rl == i + 1 ? 1.0 : 0.0);
    auto store_v = [&] {
      if (wave == 0 && lane < kRows && rl > i && rl < n) V[static_cast<int64_t>(i) * n + rl] = vl;
    };
    if (tridiag_leaves(n, i, r0)) {  // whole workgroup
      store_v();
      return;
    }
#pragma unroll
    for (int k = 0; k < CPT; ++k) {
      const int c = tid + kThreads * k;
      v[k] = c > i + 1 ? x[k] * sc : (c == i + 1 ? 1.0 : 0.0);
    }
    // everybody's products and column entries at this thread's columns
    uint64_t g[CPT][3];
    if (tridiag_exchanges(n, i)) {
      // (a poll that comes too early costs a whole further one)
      __builtin_amdgcn_s_sleep(8);
      for (int spin = 0;; ++spin) {
        bool all = true;
#pragma unroll
        for (int k = 0; k < CPT; ++k) {
          const int c = tid + kThreads * k;
          if (k < kmin || !tridiag_word_live(n, i, c)) continue;
#pragma unroll
          for (int h = 0; h < 3; ++h) g[k][h] = load_word(slot + h * n + c);
        }
#pragma unroll
        for (int k = 0; k < CPT; ++k) {
          const int c = tid + kThreads * k;
          if (k < kmin || !tridiag_word_live(n, i, c)) continue;
#pragma unroll
          for (int h = 0; h < 3; ++h) all &= (g[k][h] ^ epoch) <= kMask43;
        }
        if (all) break;
        if (spin >= poll_limit) {
          s_abort = 1;
          *err = 1;
          break;
        }
      }
    }
    // (these stores come after the polls, which would wait for them)
    store_v();
    if (last && tid == 0) {
      dvec[i] = dcur;
      evec[i] = beta;
      tau[i] = t;
    }
    if (!tridiag_exchanges(n, i)) {
      // x has a single entry: tau = 0, nothing is left to update
      if (last && tid == 0) dvec[n - 1] = sa[n - 1 - r0];
      return;
    }
    double p[CPT], a[CPT], sp = 0.0;
#pragma unroll
    for (int k = 0; k < CPT; ++k) {
      const int c = tid + kThreads * k;
      p[k] = a[k] = 0.0;
      if (k < kmin || !tridiag_word_live(n, i, c)) continue;
      a[k] = second_f64(g[k][1], g[k][2]);
      const double q = first_f64(g[k][0], g[k][1]);
      p[k] = fma(q, sc, a[k]);
      sp = fma(p[k], v[k], sp);
      if (c == i + 1) {
        s_c[0] = p[k];
        s_c[1] = a[k];
      }
      if (c == i + 2) {
        s_c[2] = p[k];
        s_c[3] = a[k];
        s_c[4] = v[k];
      }
    }
    sp = wave_sum_dpp(sp);
    if (lane == 0) red_s[wave] = sp;
    lds_barrier();
    if (s_abort) return;  // whole workgroup
    // w, and row i + 1 of the updated matrix
    const double K = 0.5 * t * t * sumw(red_s);
    const double w1 = t * s_c[0] - K;
#pragma unroll
    for (int k = 0; k < CPT; ++k) {
      w[k] = t * p[k] - K * v[k];
      x[k] = tid + kThreads * k > i + 1 ? a[k] - v[k] * w1 - w[k] : 0.0;
    }
    // (rows up to i, and lanes past kRows: values of no consequence)
    const double al = sa[lane & 7];
    wl = t * fma(s_q[lane & 7], sc, al) - K * vl;
    xl = al - vl * w1 - wl;
    alpha = s_c[3] - s_c[4] * w1 - (t * s_c[2] - K * s_c[4]);
    dcur = s_c[1] - 2.0 * w1;
  }
}

// The same reduction by one workgroup, for matrices that one compute unit's
// registers hold: the exchange through memory (1.9 us per column at n = 128)
// becomes one through LDS.  Wave v of W holds rows v, v + W, ..., lane l of
// it columns l, l + 64, ...  A x' is summed by columns (A is symmetric), so a
// wave needs no sums over its lanes: each forms its rows' share of every
// column, the shares meet in LDS, and after the one barrier of the column every
// wave forms p, w and the next row for all columns by itself.  One more wave
// has no rows: it forms the reflector (a sum, a square root and two divisions
// in series) while the others are at theirs.  Two sets of shares alternate.
// Bound by the serial chain of a column (0.96 us at n = 64, where the rows are
// few) and, from there on, the readlanes that spread x, v and w over a wave's
// rows: 164 us at n = 128, against 239 with workgroups of eight rows.  Eight
// waves are slower than four (209 us against 180, with the reflector in every
// wave: what all waves do costs more than fewer rows save), and so is this
// form beyond two columns a lane (2.9 us per column at 160).
template <int W, int CPT>
__global__ __launch_bounds__(64 * (W + 1)) void tridiag_small_kernel(
    const double* __restrict__ M, int n, double* __restrict__ V, double* __restrict__ dvec,
    double* __restrict__ evec, double* __restrict__ tau) {
  constexpr int RW = 64 * CPT / W;  // rows per wave
  constexpr int RG = 4;             // rows taken together
  static_assert(64 % W == 0 && RW % RG == 0 && CPT <= 2, "rows are dealt to the waves in turn");
  __shared__ double s_q[2][W][64 * CPT], s_a[2][64 * CPT], s_r[2][2];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x >> 6));
  double A[RW][CPT], v[CPT], w[CPT], x[CPT];
#pragma unroll
  for (int k = 0; k < CPT; ++k) {
    const int c = lane + 64 * k;
    v[k] = w[k] = 0.0;
    x[k] = c > 0 && c < n ? M[c] : 0.0;  // row 0
#pragma unroll
    for (int q = 0; q < RW; ++q) {
      const int r = wave + W * q;
      A[q][k] = wave < W && r < n && c < n ? M[static_cast<int64_t>(r) * n + c] : 0.0;
    }
  }
  // entry c of a vector over the columns, the same in every lane
  auto entry = [&](const double (&a)[CPT], int c) {
    double s = a[0];
#pragma unroll
    for (int k = 1; k < CPT; ++k) s = (c >> 6) == k ? a[k] : s;
    return readlane_f64(s, c & 63);
  };
  double dcur = M[0];
  for (int i = 0; i + 1 < n; ++i) {
    const int par = i & 1;
    double xp[CPT], acc[CPT];
#pragma unroll
    for (int k = 0; k < CPT; ++k) {
      xp[k] = lane + 64 * k > i + 1 ? x[k] : 0.0;
      acc[k] = 0.0;
    }
    if (wave < W) {
      // the pending rank-2 update, A x' over this wave's rows, and row i + 1.
      // Rows up to i and columns in blocks left of k0 are done: groups of rows
      // are skipped whole, the others' values there are of no consequence
      // (x', v and w are zero).
      auto rows = [&]<int K0>() {
#pragma unroll
        for (int g = 0; g < RW; g += RG) {
          if (wave + W * (g + RG - 1) <= i) continue;  // uniform
#pragma unroll
          for (int q = g; q < g + RG; ++q) {
            const int kr = W * q / 64, lr = wave + W * q % 64;
            const double vr = readlane_f64(v[kr], lr), wr = readlane_f64(w[kr], lr);
            const double xr = readlane_f64(xp[kr], lr);
#pragma unroll
            for (int k = K0; k < CPT; ++k) {
              A[q][k] = fma(-vr, w[k], fma(-wr, v[k], A[q][k]));
              acc[k] = fma(A[q][k], xr, acc[k]);
            }
          }
#pragma unroll
          for (int q = g; q < g + RG; ++q)
            if (wave + W * q == i + 1) {  // uniform
#pragma unroll
              for (int k = K0; k < CPT; ++k) s_a[par][lane + 64 * k] = A[q][k];
            }
        }
      };
      const int k0 = (i + 1) / 64;
      if constexpr (CPT >= 2) {
        if (k0 == 1) rows.template operator()<1>();
      }
      if (k0 == 0) rows.template operator()<0>();
#pragma unroll
      for (int k = 0; k < CPT; ++k) s_q[par][wave][lane + 64 * k] = acc[k];
    } else {
      // the reflector of row i
      const double alpha = entry(x, i + 1);
      double sg = 0.0;
#pragma unroll
      for (int k = 0; k < CPT; ++k) sg = fma(xp[k], xp[k], sg);
      const double sigma = wave_sum_dpp(sg);
      double beta = alpha, t = 0.0, sc = 0.0;
      if (sigma != 0.0) {
        beta = -copysign(sqrt(fma(alpha, alpha, sigma)), alpha);
        t = (beta - alpha) / beta;
        sc = 1.0 / (alpha - beta);
      }
      if (lane == 0) {
        s_r[par][0] = sc;
        s_r[par][1] = t;
        dvec[i] = dcur;
        evec[i] = beta;
        tau[i] = t;
      }
    }
    lds_barrier();
    const double sc = s_r[par][0], t = s_r[par][1];
#pragma unroll
    for (int k = 0; k < CPT; ++k) {
      const int c = lane + 64 * k;
      v[k] = c > i + 1 ? x[k] * sc : (c == i + 1 ? 1.0 : 0.0);
    }
    double p[CPT], a[CPT], sp = 0.0;
#pragma unroll
    for (int k = 0; k < CPT; ++k) {
      const int c = lane + 64 * k;
      double q = s_q[par][0][c];
#pragma unroll
      for (int u = 1; u < W; ++u) q += s_q[par][u][c];
      a[k] = c > i && c < n ? s_a[par][c] : 0.0;
      p[k] = c > i && c < n ? fma(q, sc, a[k]) : 0.0;
      sp = fma(p[k], v[k], sp);
    }
    // w, and row i + 1 of the updated matrix
    const double K = 0.5 * t * t * wave_sum_dpp(sp);
#pragma unroll
    for (int k = 0; k < CPT; ++k) w[k] = t * p[k] - K * v[k];
    const double w1 = entry(w, i + 1);
    if (wave == W) {
#pragma unroll
      for (int k = 0; k < CPT; ++k) {
        const int c = lane + 64 * k;
        if (c < n) V[static_cast<int64_t>(i) * n + c] = v[k];
      }
    }
    dcur = entry(a, i + 1) - 2.0 * w1;
#pragma unroll
    for (int k = 0; k < CPT; ++k)
      x[k] = lane + 64 * k > i + 1 ? a[k] - v[k] * w1 - w[k] : 0.0;
  }
  if (wave == 0) {
    if (lane == 0) dvec[n - 1] = dcur;
    for (int c = lane; c < n; c += 64) V[static_cast<int64_t>(n - 1) * n + c] = 0.0;
  }
}

}  // namespace

bool tridiag_small_fits(int64_t n) { return n >= 2 && n <= 128; }

void tridiag_small(const double* M, int64_t n64, double* V, double* dvec, double* evec, double* tau,
                   void* stream) {
  hipStream_t s = static_cast<hipStream_t>(stream);
  const int n = static_cast<int>(n64);
  if (n <= 64)
    hipLaunchKernelGGL((tridiag_small_kernel<4, 1>), dim3(1), dim3(320), 0, s, M, n, V, dvec, evec, tau);
  else
    hipLaunchKernelGGL((tridiag_small_kernel<4, 2>), dim3(1), dim3(320), 0, s, M, n, V, dvec, evec, tau);
}

bool tridiag_resident_fits(int64_t n) {
  return n >= 2 && n <= std::min<int64_t>(kMaxSize, static_cast<int64_t>(device_cus()) * kRows);
}

size_t tridiag_resident_bytes(int64_t n) {
  return n <= kMaxSize ? static_cast<size_t>(6 * n) * 8 : 0;
}

bool tridiag_resident(const double* M, int64_t n64, double* V, double* dvec, double* evec,
                      double* tau, void* work, int* err, int poll_limit, void* stream) {
  hipStream_t s = static_cast<hipStream_t>(stream);
  int n = static_cast<int>(n64);
  uint64_t* ex = static_cast<uint64_t*>(work);
  const int words = 2 * 3 * n;
  // Four waves up to n = 1024 (with eight, what every wave forms for itself
  // costs more than a second wave per SIMD hides: 768: 2.5 against 3.0 us per
  // column), eight above, where eight columns a lane no longer fit beside the
  // rest in one wave's vector registers (2048: 3.1 against 3.8 us).
  const int threads = n <= 1024 ? 256 : 512;
  const int cpt = (n + threads - 1) / threads;
  const void* fn = threads == 512 ? (cpt == 3 ? reinterpret_cast<const void*>(&tridiag_kernel<512, 3>)
                                              : reinterpret_cast<const void*>(&tridiag_kernel<512, 4>))
                   : cpt == 1     ? reinterpret_cast<const void*>(&tridiag_kernel<256, 1>)
                   : cpt == 2     ? reinterpret_cast<const void*>(&tridiag_kernel<256, 2>)
                   : cpt == 3     ? reinterpret_cast<const void*>(&tridiag_kernel<256, 3>)
                                  : reinterpret_cast<const void*>(&tridiag_kernel<256, 4>);
  hipLaunchKernelGGL(tridiag_clear_kernel, dim3(static_cast<unsigned>((words + 255) / 256)),
                     dim3(256), 0, s, ex, words, err);
  if (hipGetLastError() != hipSuccess) return false;
  void* args[] = {&M, &n, &V, &dvec, &evec, &tau, &ex, &err, &poll_limit};
  const hipError_t e = hipLaunchCooperativeKernel(
      fn, dim3(static_cast<unsigned>((n + kRows - 1) / kRows)), dim3(static_cast<unsigned>(threads)), args, 0, s);
  if (e != hipSuccess) {
    (void)hipGetLastError();  // refused (nothing ran): the caller takes the other reduction
    return false;
  }
  return true;
}

}  // namespace bitsmoe
