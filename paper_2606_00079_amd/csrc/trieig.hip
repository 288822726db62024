// Selected eigenpairs of a symmetric tridiagonal T (fp64): the r largest
// eigenvalues by multisection on Sturm counts, and their eigenvectors by
// twisted factorizations.
//
// Both rest on the three-term recurrence of T - x's leading minors,
//     p_j = (d_j - x) p_{j-1} - e_{j-1}^2 p_{j-2},
// whose ratios p_j / p_{j-1} are the pivots of the LDL^T factorization: one
// dependent fma per row where the pivots themselves take a division.  The
// computed ratios are the exact pivots of a T whose d and e^2 differ from the
// given ones by a few ulps (of |d - x| and of e^2), as for the quotient form,
// so counts and vectors carry the same error.  T is scaled to norm in [1/2, 1)
// by a power of two, p is rescaled by one every eight rows, and couplings
// below 1e-25 are raised to it: eight rows then move p by less than the
// exponent's range, and a zero p_j is followed by p_{j+1} = -e^2 p_{j-1} of
// the sign that counts it once.  (Beside a norm of 1/2 or more 1e-25 is far
// below an ulp; T = 0 has no norm to compare it with and is answered as such.)
//
// Before: counts by quotients (a division per row on the dependent chain:
// 2.39 ms at n = 2048, r = 1024; 0.70 ms at 768, r = 384) and three inverse
// iterations per vector, one thread each, through four work arrays in memory
// (8.48 and 2.58 ms).  Now 0.70 and 0.14 ms (0.16 and 0.04); both are bound by the
// serial chain over T's rows (one wave per SIMD).
#include <algorithm>
#include <cmath>

#include "bitsmoe.h"
#include "common.hpp"
#include "eig_wave.hpp"
#include "internal.hpp"

namespace bitsmoe {
namespace {

constexpr int kGroup = 8;          // rows between rescalings
constexpr double kMinE = 1e-25;    // smallest coupling of the scaled T
constexpr int64_t kVecLds = 3584;  // longest vector whose two recurrences stay in LDS

int64_t padded(int64_t n) { return (n + kGroup - 1) / kGroup * kGroup; }

// LDS (or scratch) index of row j: a double of padding every 32, so that lanes
// that walk chunks of rows do not share banks.
__host__ __device__ __forceinline__ int64_t row_at(int64_t j) { return j + (j >> 5); }

// Scales T and finds its bounds (one workgroup).  de[2j] = d_j, de[2j+1] =
// e_{j-1}^2 (0 for j = 0), rev the same for T read from its end, both padded
// to whole groups with rows that change no count; es[j] = e_j.  info: lo, hi
// (Gershgorin, widened), the norm of the scaled T, and of the given T its
// norm, max e^2, exponent of the scale and whether an entry is not finite.
__global__ __launch_bounds__(1024) void tri_prep_kernel(const double* __restrict__ d,
                                                        const double* __restrict__ e, int64_t n,
                                                        int64_t np, double* __restrict__ de,
                                                        double* __restrict__ rev,
                                                        double* __restrict__ es,
                                                        double* __restrict__ info) {
  __shared__ double s_lo[16], s_hi[16], s_nrm[16], s_e2[16];
  __shared__ int s_bad, s_ex;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  if (threadIdx.x == 0) s_bad = 0;
  __syncthreads();
  double lo = 1.7976931348623157e308, hi = -lo, nrm = 0.0, e2 = 0.0;
  for (int64_t j = threadIdx.x; j < n; j += 1024) {
    const double dj = d[j];
    const double el = j > 0 ? fabs(e[j - 1]) : 0.0, er = j + 1 < n ? fabs(e[j]) : 0.0;
    if (!(fabs(dj) + el + er <= 1.7976931348623157e308)) s_bad = 1;
    lo = fmin(lo, dj - el - er);
    hi = fmax(hi, dj + el + er);
    nrm = fmax(nrm, fabs(dj) + el + er);
    e2 = fmax(e2, er * er);
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    lo = fmin(lo, __shfl_xor(lo, o, 64));
    hi = fmax(hi, __shfl_xor(hi, o, 64));
    nrm = fmax(nrm, __shfl_xor(nrm, o, 64));
    e2 = fmax(e2, __shfl_xor(e2, o, 64));
  }
  if (lane == 0) {
    s_lo[wave] = lo;
    s_hi[wave] = hi;
    s_nrm[wave] = nrm;
    s_e2[wave] = e2;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int q = 1; q < 16; ++q) {
      lo = fmin(lo, s_lo[q]);
      hi = fmax(hi, s_hi[q]);
      nrm = fmax(nrm, s_nrm[q]);
      e2 = fmax(e2, s_e2[q]);
    }
    int ex = 0;
    if (nrm > 0.0 && !s_bad) (void)frexp(nrm, &ex);
    const double sn = ldexp(nrm, -ex), eps = 2.220446049250313e-16;
    s_ex = ex;
    info[0] = ldexp(lo, -ex) - 2.0 * eps * sn - kMinE;
    info[1] = ldexp(hi, -ex) + 2.0 * eps * sn + kMinE;
    info[2] = sn;
    info[3] = nrm;
    info[4] = e2;
    info[5] = ex;
    info[6] = s_bad;
  }
  __syncthreads();
  const int ex = s_ex;
  auto coupling = [&](int64_t j) {  // e_j of the scaled T
    const double v = ldexp(e[j], -ex);
    return fabs(v) >= kMinE ? v : kMinE;
  };
  for (int64_t j = threadIdx.x; j < np; j += 1024) {
    double a = 4.0, b = 0.0, ra = 4.0, rb = 0.0;  // padding: positive whatever x
    if (j < n) {
      const int64_t m = n - 1 - j;
      a = ldexp(d[j], -ex);
      ra = ldexp(d[m], -ex);
      if (j > 0) {
        const double f = coupling(j - 1), g = coupling(m);
        b = f * f;
        rb = g * g;
      }
      if (j + 1 < n) es[j] = coupling(j);
    }
    de[2 * j] = a;
    de[2 * j + 1] = b;
    rev[2 * j] = ra;
    rev[2 * j + 1] = rb;
  }
}

// One group of the recurrence: rescales (p1, p2) = (p_{j-1}, p_{j-2}) and
// advances them by kGroup rows, whose p go to out.
__device__ __forceinline__ void recur(const double (&de)[2 * kGroup], double x, double& p1,
                                      double& p2, double (&out)[kGroup]) {
  const int ex = __builtin_amdgcn_frexp_exp(fmax(fabs(p1), fabs(p2)));
  p1 = ldexp(p1, -ex);
  p2 = ldexp(p2, -ex);
#pragma unroll
  for (int u = 0; u < kGroup; ++u) {
    const double t = de[2 * u + 1] * p2;
    const double p = fma(de[2 * u] - x, p1, -t);
    out[u] = p;
    p2 = p1;
    p1 = p;
  }
}

// w[k] (and ws[k], of the scaled T) = eigenvalue n - r + k, ascending: one
// wave per eigenvalue splits [lo, hi] at 64 interior points per step (lane l
// counts at lo + (hi - lo)(l + 1)/65); the counts grow with x, so the lanes
// whose count is <= n - r + k form a prefix and the new interval is the gap
// after it.  Stops when the interval is two ulps of the norm wide or the
// points no longer fall strictly inside.
__global__ __launch_bounds__(64) void tri_bisect_kernel(const double* __restrict__ de, int64_t np,
                                                        int64_t t0, const double* __restrict__ info,
                                                        double* __restrict__ ws,
                                                        double* __restrict__ w) {
  const int lane = threadIdx.x;
  const int64_t t = t0 + blockIdx.x;
  if (info[2] == 0.0) {  // T = 0
    if (lane == 0) ws[blockIdx.x] = w[blockIdx.x] = 0.0;
    return;
  }
  double lo = info[0], hi = info[1];
  const double atol = 2.0 * 2.220446049250313e-16 * info[2];
  for (int it = 0; it < 64 && hi - lo > atol; ++it) {
    const double x = lo + (hi - lo) * (static_cast<double>(lane + 1) / 65.0);
    const bool inside = x > lo && x < hi;
    if (__ballot(inside) != ~0ull) break;  // the interval is a few ulps wide
    double p1 = 1.0, p2 = 0.0;
    uint32_t cnt = 0;
    double cur[2 * kGroup], nxt[2 * kGroup];
#pragma unroll
    for (int u = 0; u < 2 * kGroup; ++u) cur[u] = de[u];
    for (int64_t j = 0; j < np; j += kGroup) {
      const int64_t jn = j + kGroup < np ? j + kGroup : j;
#pragma unroll
      for (int u = 0; u < 2 * kGroup; ++u) nxt[u] = de[2 * jn + u];
      uint32_t prev = static_cast<uint32_t>(__builtin_bit_cast(uint64_t, p1) >> 32);
      double out[kGroup];
      recur(cur, x, p1, p2, out);
#pragma unroll
      for (int u = 0; u < kGroup; ++u) {
        const uint32_t h = static_cast<uint32_t>(__builtin_bit_cast(uint64_t, out[u]) >> 32);
        cnt += (h ^ prev) >> 31;
        prev = h;
      }
#pragma unroll
      for (int u = 0; u < 2 * kGroup; ++u) cur[u] = nxt[u];
    }
    const int p = __popcll(__ballot(static_cast<int64_t>(cnt) <= t));  // lanes 0..p-1
    const double xl = __shfl(x, p > 0 ? p - 1 : 0, 64);
    const double xh = __shfl(x, p < 64 ? p : 63, 64);
    lo = p > 0 ? xl : lo;
    hi = p < 64 ? xh : hi;
  }
  if (lane == 0) {
    const double v = 0.5 * (lo + hi);
    ws[blockIdx.x] = v;
    w[blockIdx.x] = ldexp(v, static_cast<int>(info[5]));
  }
}

// Row k = blockIdx.x of Zt: the eigenvector of ws[k].  One wave runs the
// recurrence from the top (p, pivots q+_j = p_j / p_{j-1}), the other from
// the bottom (q-); the twist is the row m with the smallest |gamma_m|, gamma =
// q+ + q- - (d - x), and (T - x) z = gamma_m e_m has z_m = 1,
// z_j = -(e_j / q+_j) z_{j+1} above and z_j = -(e_{j-1} / q-_j) z_{j-1} below:
// products, formed by chunks of rows per lane and a scan over the lanes.  The
// residual is that of one inverse iteration from the best unit vector, a few
// ulps of the norm.  bad[k] is set when the result is not finite.
// IN_LDS: both recurrences fit in LDS, else they use `work`
// (2 row_at(np) + 2 doubles per vector).
template <bool IN_LDS>
__global__ __launch_bounds__(128) void tri_vec_kernel(const double* __restrict__ de,
                                                      const double* __restrict__ rev,
                                                      const double* __restrict__ es, int64_t n,
                                                      int64_t np, const double* __restrict__ info,
                                                      const double* __restrict__ ws,
                                                      double* __restrict__ work,
                                                      double* __restrict__ Zt,
                                                      uint8_t* __restrict__ bad) {
  extern __shared__ double lds[];
  __shared__ double s_v[2];
  __shared__ int64_t s_i[2];
  if (info[2] == 0.0) {  // T = 0: unit vectors
    double* z = Zt + blockIdx.x * n;
    for (int64_t j = threadIdx.x; j < n; j += 128) z[j] = j == n - gridDim.x + blockIdx.x ? 1.0 : 0.0;
    if (threadIdx.x == 0) bad[blockIdx.x] = 0;
    return;
  }
  const int64_t len = row_at(np) + 1;
  double* pf = IN_LDS ? lds : work + blockIdx.x * 2 * len;  // rows from the top
  double* pb = pf + len;                                    // rows from the bottom
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const double x = ws[blockIdx.x];
  {
    const double* src = wave == 0 ? de : rev;
    double* dst = wave == 0 ? pf : pb;
    double p1 = 1.0, p2 = 0.0;
    double cur[2 * kGroup], nxt[2 * kGroup];
#pragma unroll
    for (int u = 0; u < 2 * kGroup; ++u) cur[u] = src[u];
    for (int64_t j = 0; j < np; j += kGroup) {
      const int64_t jn = j + kGroup < np ? j + kGroup : j;
#pragma unroll
      for (int u = 0; u < 2 * kGroup; ++u) nxt[u] = src[2 * jn + u];
      double out[kGroup];
      recur(cur, x, p1, p2, out);
      if (lane == 0) {  // (a group does not straddle the padding)
        double* o = dst + row_at(wave == 0 ? j : np - kGroup - j);
#pragma unroll
        for (int u = 0; u < kGroup; ++u) o[wave == 0 ? u : kGroup - 1 - u] = out[u];
      }
#pragma unroll
      for (int u = 0; u < 2 * kGroup; ++u) cur[u] = nxt[u];
    }
  }
  __syncthreads();
  // pf holds row j at j, pb row j at j + sh, so that both keep T's order
  const int64_t sh = np - n;
  auto p_of = [&](bool top, int64_t j) { return top ? pf[row_at(j)] : pb[row_at(np - 1 - j)]; };
  // pivot of row j of a recurrence (rows counted from its own end): p_j over
  // the p_{j-1} that it was formed from; a zero p stands for 2^-60 of its
  // predecessor, in its own pivot and in the next one
  auto before = [&](bool top, int64_t j) {  // the (rescaled) p_{j-1}
    if (j == 0) return 0.5;
    const double a = p_of(top, j - 1);
    if (j % kGroup != 0) return a;
    return ldexp(a, -__builtin_amdgcn_frexp_exp(fmax(fabs(a), fabs(p_of(top, j - 2)))));
  };
  auto pivot = [&](bool top, int64_t j) {
    double den = before(top, j), num = p_of(top, j);
    if (den == 0.0) {
      den = before(top, j - 1) * 8.673617379884035e-19;
      if (j % kGroup == 0) den = ldexp(den, -__builtin_amdgcn_frexp_exp(fabs(p_of(top, j - 2))));
    }
    if (num == 0.0) num = den * 8.673617379884035e-19;
    return num / den;
  };
  double best = 1.7976931348623157e308;
  int64_t m = n;
  for (int64_t j = threadIdx.x; j < n; j += 128) {
    const double g = fabs(pivot(true, j) + pivot(false, n - 1 - j) - (de[2 * j] - x));
    if (g < best || (m == n && g <= best)) {
      best = g;
      m = j;
    }
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    const double ob = __shfl_xor(best, o, 64);
    const int64_t om = __shfl_xor(m, o, 64);
    if (ob < best || (ob == best && om < m)) {
      best = ob;
      m = om;
    }
  }
  if (lane == 0) {
    s_v[wave] = best;
    s_i[wave] = m;
  }
  __syncthreads();
  m = s_v[1] < s_v[0] || (s_v[1] == s_v[0] && s_i[1] < s_i[0]) ? s_i[1] : s_i[0];
  const bool none = m >= n;  // no finite gamma
  if (none) m = 0;
  // the factors z_j / z_{j+1} above m go into pb's rows (which only serve
  // below it now), z_j / z_{j-1} below m into pf's
  auto above = [&](int64_t j) { return pb + row_at(j + sh); };
  auto below = [&](int64_t j) { return pf + row_at(j); };
  for (int64_t j = threadIdx.x; j < n; j += 128) {
    if (j < m) *above(j) = -(es[j] / pivot(true, j));
    if (j > m) *below(j) = -(es[j - 1] / pivot(false, n - 1 - j));
  }
  __syncthreads();
  const int64_t cnt = wave == 0 ? m : n - 1 - m;
  const int64_t chunk = (cnt + 63) / 64;
  const int64_t a = std::min<int64_t>(lane * chunk, cnt), b = std::min<int64_t>(a + chunk, cnt);
  auto at = [&](int64_t s) { return wave == 0 ? above(m - 1 - s) : below(m + 1 + s); };
  double prod = 1.0;
  for (int64_t s = a; s < b; ++s) prod *= *at(s);
  double incl = prod;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const double u = __shfl_up(incl, o, 64);
    if (lane >= o) incl *= u;
  }
  double run = __shfl_up(incl, 1, 64);
  if (lane == 0) run = 1.0;
  double ss = 0.0;
  for (int64_t s = a; s < b; ++s) {
    run *= *at(s);
    *at(s) = run;
    ss = fma(run, run, ss);
  }
  ss = wave_sum_dpp(ss);
  if (lane == 0) s_v[wave] = ss;
  __syncthreads();
  ss = 1.0 + s_v[0] + s_v[1];
  const double nrm = 1.0 / sqrt(ss);
  double* z = Zt + blockIdx.x * n;
  for (int64_t j = threadIdx.x; j < n; j += 128)
    z[j] = j == m ? nrm : (j < m ? *above(j) : *below(j)) * nrm;
  if (threadIdx.x == 0) bad[blockIdx.x] = none || !(ss <= 1e300);
}

}  // namespace

size_t tri_eigenpairs_bytes(int64_t n, int64_t r) {
  const int64_t np = padded(n);
  const int64_t work = np <= kVecLds ? 0 : 2 * (row_at(np) + 1) * r;
  return static_cast<size_t>(4 * np + n + r + work) * 8;
}

bitsmoe_status tri_eigenpairs(const double* d, const double* e, int64_t n, int64_t r, double* w,
                              double* Zt, double* info, uint8_t* bad, void* buf, void* stream) {
  hipStream_t s = static_cast<hipStream_t>(stream);
  const int64_t np = padded(n);
  double* de = static_cast<double*>(buf);
  double* rev = de + 2 * np;
  double* es = rev + 2 * np;
  double* ws = es + n;
  double* work = ws + r;
  hipLaunchKernelGGL(tri_prep_kernel, dim3(1), dim3(1024), 0, s, d, e, n, np, de, rev, es, info);
  hipLaunchKernelGGL(tri_bisect_kernel, dim3(static_cast<unsigned>(r)), dim3(64), 0, s, de, np, n - r,
                     info, ws, w);
  if (np <= kVecLds)
    hipLaunchKernelGGL(tri_vec_kernel<true>, dim3(static_cast<unsigned>(r)), dim3(128),
                       static_cast<size_t>(2 * (row_at(np) + 1)) * 8, s, de, rev, es, n, np, info, ws, work,
                       Zt, bad);
  else
    hipLaunchKernelGGL(tri_vec_kernel<false>, dim3(static_cast<unsigned>(r)), dim3(128), 0, s, de, rev,
                       es, n, np, info, ws, work, Zt, bad);
  BITSMOE_LAUNCH_CHECK("shared_basis_gpu: tridiagonal eigenpairs");
  return BITSMOE_OK;
}

}  // namespace bitsmoe
