// Back-transformation of the device eigensolver, U = H_0 H_1 ... H_{n-2} Z, in
// one launch, with the sign rule and the fp32 result.
//
// The reflectors act on every vector alike, so a workgroup takes NV vectors,
// keeps them in registers and applies all panels of eight reflectors from the
// last to the first in their compact form I - V T V^T (T 8 x 8, upper
// triangular): products with the panel's rows, a sum over the workgroup, the
// product with T, and the update.  The next panel's rows are loaded meanwhile.
// Nothing but V is read and there is one barrier per panel.
//
// Before: two launches per panel of 32 with the vectors in memory, 6.2 ms at
// n = 2048, r = 1024 and 1.47 ms at n = 768, r = 384, bound by one wave's walk
// over each row.  Now 0.96 and 0.16 ms; bound by the chain of a panel (sum, T, update),
// and at 2048 by reading V (16.8 MB per workgroup, from L2).
#include <algorithm>

#include "bitsmoe.h"
#include "common.hpp"
#include "eig_wave.hpp"
#include "internal.hpp"

namespace bitsmoe {
namespace {

constexpr int kPanel = 8;
constexpr int kMaxThreads = 512;
constexpr int kMaxCols = 4;  // columns per thread at most

// T of panel blockIdx.x (reflectors j0 .. j0 + 7, rows of V; zero past n - 2):
// T[c][c] = tau_c, T[r][c] = -tau_c sum_{k=r}^{c-1} T[r][k] (V_k . V_c).
__global__ __launch_bounds__(256) void panel_t_kernel(const double* __restrict__ V,
                                                      const double* __restrict__ tau, int64_t n,
                                                      double* __restrict__ Tall) {
  __shared__ double part[4][32], sG[32];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int64_t j0 = static_cast<int64_t>(blockIdx.x) * kPanel;
  const int nb = static_cast<int>(std::min<int64_t>(kPanel, n - 1 - j0));
  double acc[32];
#pragma unroll
  for (int q = 0; q < 32; ++q) acc[q] = 0.0;
  for (int64_t c = j0 + 1 + threadIdx.x; c < n; c += 256) {
    double v[kPanel];
#pragma unroll
    for (int a = 0; a < kPanel; ++a) v[a] = a < nb ? V[(j0 + a) * n + c] : 0.0;
    int q = 0;
#pragma unroll
    for (int a = 0; a < kPanel; ++a)
#pragma unroll
      for (int b = a + 1; b < kPanel; ++b) {
        acc[q] = fma(v[a], v[b], acc[q]);
        ++q;
      }
  }
  const double s = wave_fold<32>(acc, lane);
  if ((lane & 1) == 0) part[wave][lane >> 1] = s;
  __syncthreads();
  if (threadIdx.x < 32)
    sG[threadIdx.x] = (part[0][threadIdx.x] + part[1][threadIdx.x]) +
                      (part[2][threadIdx.x] + part[3][threadIdx.x]);
  __syncthreads();
  const int r = threadIdx.x;
  if (r >= kPanel) return;
  double t[kPanel];
  double* out = Tall + (static_cast<int64_t>(blockIdx.x) * kPanel + r) * kPanel;
#pragma unroll
  for (int c = 0; c < kPanel; ++c) {
    double v = 0.0;
#pragma unroll
    for (int k = 0; k < c; ++k)  // V_k . V_c is number k (15 - k) / 2 + c - k - 1
      if (k >= r) v = fma(t[k], sG[k * (15 - k) / 2 + c - k - 1], v);
    const double tc = c < nb ? tau[j0 + c] : 0.0;
    t[c] = c < r ? 0.0 : (c == r ? tc : -tc * v);
    out[c] = t[c];
  }
}

// Vectors NV blockIdx.x .. + NV - 1 (rows of Zt [r][n], ascending eigenvalues)
// through all reflectors; row r - 1 - k of Ut [r][n] gets vector k in fp32,
// signed so that its entry of largest magnitude is positive (lowest index on
// ties).  Thread t owns columns t, t + blockDim.x, ..., CPT blockDim.x >= n.
template <int NV, int CPT>
__global__ __launch_bounds__(kMaxThreads) void backtransform_kernel(
    const double* __restrict__ V, const double* __restrict__ Tall, const double* __restrict__ Zt,
    int n, int r, float* __restrict__ Ut) {
  constexpr int W = kMaxThreads / 64;
  constexpr int N = kPanel * NV;  // products per panel
  __shared__ __align__(16) double red[2][W][N], sx[W][N], sy[W][N];
  __shared__ double s_v[W][NV];
  __shared__ int s_i[W][NV];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int T = blockDim.x, nw = T >> 6;
  const int k0 = static_cast<int>(blockIdx.x) * NV;
  double z[NV][CPT];
#pragma unroll
  for (int k = 0; k < CPT; ++k) {
    const int c = tid + T * k;
#pragma unroll
    for (int u = 0; u < NV; ++u)
      z[u][k] = c < n && k0 + u < r ? Zt[static_cast<int64_t>(k0 + u) * n + c] : 0.0;
  }
  // (waves that were not launched: zeros)
  for (int q = tid; q < 2 * W * N; q += T) (&red[0][0][0])[q] = 0.0;
  __syncthreads();
  const int npan = (n - 1 + kPanel - 1) / kPanel;
  const int vl = lane % N;  // this lane's product: vector vl / 8, reflector vl % 8
  double cur[kPanel][CPT], nxt[kPanel][CPT];
  auto load = [&](int p, double (&v)[kPanel][CPT]) {
    const int j0 = p * kPanel;
#pragma unroll
    for (int a = 0; a < kPanel; ++a)
#pragma unroll
      for (int k = 0; k < CPT; ++k) {
        const int c = tid + T * k;
        v[a][k] = j0 + a < n - 1 && c > j0 && c < n ? V[static_cast<int64_t>(j0 + a) * n + c] : 0.0;
      }
  };
  if (npan > 0) load(npan - 1, cur);
  for (int p = npan - 1; p >= 0; --p) {
    const int kmin = (p * kPanel + 1) / T;  // columns below kmin T are untouched
    double acc[N], tc[kPanel];  // the products; row vl % 8 of T
#pragma unroll
    for (int a = 0; a < kPanel; ++a)
      tc[a] = Tall[(static_cast<int64_t>(p) * kPanel + (vl & 7)) * kPanel + a];
#pragma unroll
    for (int q = 0; q < N; ++q) acc[q] = 0.0;
#pragma unroll
    for (int k = 0; k < CPT; ++k) {
      if (k < kmin) continue;
#pragma unroll
      for (int u = 0; u < NV; ++u)
#pragma unroll
        for (int a = 0; a < kPanel; ++a)
          acc[u * kPanel + a] = fma(cur[a][k], z[u][k], acc[u * kPanel + a]);
    }
    const double s = wave_fold<N>(acc, lane);
    if (lane % (64 / N) == 0) red[p & 1][wave][lane / (64 / N)] = s;
    if (p > 0) load(p - 1, nxt);
    lds_barrier();
    {
      // every wave: the sums, and their product with T
      const double(*rd)[N] = red[p & 1];
      const double x = ((rd[0][vl] + rd[1][vl]) + (rd[2][vl] + rd[3][vl])) +
                       ((rd[4][vl] + rd[5][vl]) + (rd[6][vl] + rd[7][vl]));
      if (lane < N) sx[wave][lane] = x;
      __builtin_amdgcn_wave_barrier();
      double y0 = 0.0, y1 = 0.0;
#pragma unroll
      for (int a = 0; a < kPanel; a += 2) {
        y0 = fma(tc[a], sx[wave][(vl & ~7) + a], y0);
        y1 = fma(tc[a + 1], sx[wave][(vl & ~7) + a + 1], y1);
      }
      if (lane < N) sy[wave][lane] = y0 + y1;
      __builtin_amdgcn_wave_barrier();
    }
#pragma unroll
    for (int u = 0; u < NV; ++u)
#pragma unroll
      for (int a = 0; a < kPanel; ++a) {
        const double y = sy[wave][u * kPanel + a];
#pragma unroll
        for (int k = 0; k < CPT; ++k)
          z[u][k] = fma(-y, cur[a][k], z[u][k]);  // (cur is zero where untouched)
      }
    __builtin_amdgcn_wave_barrier();
#pragma unroll
    for (int a = 0; a < kPanel; ++a) {
#pragma unroll
      for (int k = 0; k < CPT; ++k) cur[a][k] = nxt[a][k];
    }
  }
  // order, sign, fp32
#pragma unroll
  for (int u = 0; u < NV; ++u) {
    double best = -1.0;
    int bi = n;
#pragma unroll
    for (int k = 0; k < CPT; ++k) {
      const int c = tid + T * k;
      if (c < n && fabs(z[u][k]) > best) {
        best = fabs(z[u][k]);
        bi = z[u][k] < 0.0 ? ~c : c;  // the sign rides along
      }
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
      const double ob = __shfl_xor(best, o, 64);
      const int oi = __shfl_xor(bi, o, 64);
      if (ob > best || (ob == best && (oi < 0 ? ~oi : oi) < (bi < 0 ? ~bi : bi))) {
        best = ob;
        bi = oi;
      }
    }
    if (lane == 0) {
      s_v[wave][u] = best;
      s_i[wave][u] = bi;
    }
  }
  __syncthreads();
#pragma unroll
  for (int u = 0; u < NV; ++u) {
    if (k0 + u >= r) continue;
    double best = s_v[0][u];
    int bi = s_i[0][u];
    for (int q = 1; q < nw; ++q) {
      const double ob = s_v[q][u];
      const int oi = s_i[q][u];
      if (ob > best || (ob == best && (oi < 0 ? ~oi : oi) < (bi < 0 ? ~bi : bi))) {
        best = ob;
        bi = oi;
      }
    }
    const double sg = bi < 0 ? -1.0 : 1.0;
#pragma unroll
    for (int k = 0; k < CPT; ++k) {
      const int c = tid + T * k;
      if (c < n)
        Ut[static_cast<int64_t>(r - 1 - (k0 + u)) * n + c] = static_cast<float>(sg * z[u][k]);
    }
  }
}

}  // namespace

bool backtransform_fits(int64_t n) { return n <= kMaxThreads * kMaxCols; }

size_t backtransform_bytes(int64_t n) {
  return static_cast<size_t>((n + kPanel - 1) / kPanel) * kPanel * kPanel * 8;
}

bitsmoe_status backtransform_panels(const double* V, const double* tau, int64_t n, double* T,
                                    void* stream) {
  const int64_t npan = (n - 1 + kPanel - 1) / kPanel;
  if (npan == 0) return BITSMOE_OK;
  hipLaunchKernelGGL(panel_t_kernel, dim3(static_cast<unsigned>(npan)), dim3(256), 0,
                     static_cast<hipStream_t>(stream), V, tau, n, T);
  BITSMOE_LAUNCH_CHECK("shared_basis_gpu: compact forms");
  return BITSMOE_OK;
}

bitsmoe_status backtransform(const double* V, const double* T, const double* Zt, int64_t n, int64_t r,
                             float* Ut, void* stream) {
  const int cpt = static_cast<int>((n + kMaxThreads - 1) / kMaxThreads);
  const int threads = static_cast<int>(((n + cpt - 1) / cpt + 63) / 64 * 64);
  // vectors per workgroup: more share a panel's rows, fewer fill the chip
  const int nv = r > 512 ? 4 : (r > 256 ? 2 : 1);
  const dim3 grid(static_cast<unsigned>((r + nv - 1) / nv)), block(static_cast<unsigned>(threads));
#define BITSMOE_BT(NV, CPT)                                                                     \
  hipLaunchKernelGGL((backtransform_kernel<NV, CPT>), grid, block, 0, static_cast<hipStream_t>(stream), \
                     V, T, Zt, static_cast<int>(n), static_cast<int>(r), Ut)
#define BITSMOE_BT_V(CPT) \
  if (nv == 4) BITSMOE_BT(4, CPT); else if (nv == 2) BITSMOE_BT(2, CPT); else BITSMOE_BT(1, CPT)
  if (cpt == 1) {
    BITSMOE_BT_V(1);
  } else if (cpt == 2) {
    BITSMOE_BT_V(2);
  } else if (cpt == 3) {
    BITSMOE_BT_V(3);
  } else {
    BITSMOE_BT_V(4);
  }
#undef BITSMOE_BT_V
#undef BITSMOE_BT
  BITSMOE_LAUNCH_CHECK("shared_basis_gpu: back-transformation");
  return BITSMOE_OK;
}

}  // namespace bitsmoe
