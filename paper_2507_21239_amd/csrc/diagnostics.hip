// diagnostics.hip -- sigma_d(m, r), the dust surface density per particle
// mass bin and radius (paper, Benchmark: the run's output is the dust surface
// density as a function of particle mass and distance from the star).
//
// Bins are half-open, r_edges[k] <= r < r_edges[k+1] and m_edges[l] <= m <
// m_edges[l+1], found by binary search on the edges (comparisons only, so a
// particle's bin does not depend on rounding).  Each active particle in range
// adds its swarm mass M to bin (k, l); each bin is then divided by its
// annulus area pi (r_edges[k+1]^2 - r_edges[k]^2) (1 in column mode, where M
// is per unit area).  Workgroups accumulate contiguous ranges of the particles
// in LDS and leave their bins in scratch, where a second launch adds them up;
// histograms that do not fit that add every particle to global memory by
// atomics.  The FP64 sums therefore follow the order of the atomics.
#include <algorithm>

#include "device_common.hpp"
#include "internal.hpp"

namespace mcd {

constexpr int kHistThreads = 1024;  // one workgroup per CU
constexpr int kHistLdsBins = 12800;  // 12 bytes each; with the edges within the 160 KB of LDS
constexpr int kHistLdsEdges = 1024;
constexpr int kHistParts = 4;
constexpr int kHistFewBins = 4096;  // in LDS for any number of particles and edges
static_assert(kHistLdsEdges * 8 + kHistLdsBins * 12 <= 160 * 1024, "one part fits");
static_assert((kHistFewBins + 3) * 8 + kHistFewBins * 12 <= 160 * 1024, "few bins in any shape fit");
constexpr int kHistUnroll = 4;

// bin of x by binary search: e[k] <= x < e[k+1], -1 outside the edges
__device__ inline int find_bin(const double *e, int n, double x) {
  if (!(x >= e[0]) || !(x < e[n])) return -1;
  int lo = 0, hi = n;  // e[lo] <= x < e[hi]
  while (hi - lo > 1) {
    const int mid = lo + (hi - lo) / 2;
    if (x < e[mid])
      hi = mid;
    else
      lo = mid;
  }
  return lo;
}

// the same with a guess for edges in geometric progression, which the edges
// either confirm or leave to the search: two reads of LDS instead of one per
// halving
struct Guess {
  float lo, scale;
};
__device__ inline Guess bin_guess(const double *e, int n) {
  const float a = __builtin_amdgcn_logf((float)e[0]), b = __builtin_amdgcn_logf((float)e[n]);
  return {a, (float)n / (b - a)};
}
__device__ inline int find_bin(const double *e, int n, double x, const Guess &q) {
  const float f = (__builtin_amdgcn_logf((float)x) - q.lo) * q.scale;
  const int g = (int)fminf(fmaxf(f, 0.0f), (float)(n - 1));  // 0 for a NaN
  if (x >= e[g] && x < e[g + 1]) return g;
  return find_bin(e, n, x);
}

__global__ __launch_bounds__(256) void k_hist_clear(double *sigma, uint32_t *count, int64_t nb) {
  for (int64_t b = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; b < nb;
       b += (int64_t)gridDim.x * blockDim.x) {
    sigma[b] = 0.0;
    if (count) count[b] = 0u;
  }
}

// Workgroup (w, p) takes the particles [w chunk, (w+1) chunk) and the bins of
// `rows` radial rows from p rows on; its sums and counts go to row w of the
// scratch (a lone workgroup's to the outputs, where counts may be unwanted).
// Bound by the one pass over the particles: at 2e6 particles in no radial order
// and 60 x 90 bins the call takes 21.7 us (10 us at the rate of a large copy;
// this launch 15, the next 7), by atomics on global memory, two a particle,
// 236 us.
__global__ __launch_bounds__(kHistThreads) void k_hist_lds(
    const double *__restrict__ r, const double *__restrict__ m, const double *__restrict__ M,
    const uint8_t *__restrict__ active, int64_t N, int64_t chunk, const double *__restrict__ re,
    int n_rb, const double *__restrict__ me, int n_mb, int rows, double *__restrict__ psum,
    uint32_t *__restrict__ pcount) {
  extern __shared__ __align__(16) char smem[];
  const int k0 = blockIdx.y * rows, k1 = min(k0 + rows, n_rb), nb = (k1 - k0) * n_mb;
  double *er = (double *)smem, *em = er + n_rb + 1, *ls = em + n_mb + 1;
  uint32_t *lc = (uint32_t *)(ls + rows * n_mb);
  for (int k = threadIdx.x; k <= n_rb; k += kHistThreads) er[k] = re[k];
  for (int k = threadIdx.x; k <= n_mb; k += kHistThreads) em[k] = me[k];
  for (int b = threadIdx.x; b < nb; b += kHistThreads) {
    ls[b] = 0.0;
    lc[b] = 0u;
  }
  __syncthreads();
  const Guess qr = bin_guess(er, n_rb), qm = bin_guess(em, n_mb);
  const int64_t i0 = (int64_t)blockIdx.x * chunk;
  const int64_t i1 = i0 + chunk < N ? i0 + chunk : N;
  for (int64_t i = i0 + threadIdx.x; i < i1; i += kHistUnroll * kHistThreads) {
    double x[kHistUnroll], y[kHistUnroll], w[kHistUnroll];
    bool on[kHistUnroll];
#pragma unroll
    for (int u = 0; u < kHistUnroll; ++u) {
      const int64_t j = i + u * kHistThreads, jc = j < i1 ? j : i;
      x[u] = r[jc];
      y[u] = m[jc];
      w[u] = M[jc];
      on[u] = active[jc] && j < i1;
    }
#pragma unroll
    for (int u = 0; u < kHistUnroll; ++u) {
      if (!on[u]) continue;
      const int k = find_bin(er, n_rb, x[u], qr);
      if (k < k0 || k >= k1) continue;
      const int l = find_bin(em, n_mb, y[u], qm);
      if (l < 0) continue;
      const int b = (k - k0) * n_mb + l;
      unsafeAtomicAdd(&ls[b], w[u]);
      atomicAdd(&lc[b], 1u);
    }
  }
  __syncthreads();
  const int64_t row = (int64_t)blockIdx.x * n_rb * n_mb + (int64_t)k0 * n_mb;
  for (int b = threadIdx.x; b < nb; b += kHistThreads) {
    psum[row + b] = ls[b];
    if (pcount) pcount[row + b] = lc[b];
  }
}

__device__ inline double bin_area(const double *re, int k, int column) {
  return column ? 1.0 : kPi * (re[k + 1] * re[k + 1] - re[k] * re[k]);
}

// 32 bins a workgroup, 32 slices of the scratch rows side by side
__global__ __launch_bounds__(1024) void k_hist_reduce(const double *__restrict__ psum,
                                                      const uint32_t *__restrict__ pcount,
                                                      int rows, const double *re, int n_rb,
                                                      int n_mb, int column, double *sigma,
                                                      uint32_t *count) {
  __shared__ double ls[32][33];
  __shared__ uint32_t lc[32][33];
  const int64_t nb = (int64_t)n_rb * n_mb;
  const int x = threadIdx.x & 31, y = threadIdx.x >> 5;
  const int64_t b = (int64_t)blockIdx.x * 32 + x;
  double s = 0.0;
  uint32_t c = 0;
  if (b < nb) {
#pragma unroll 8
    for (int w = y; w < rows; w += 32) {
      s += psum[w * nb + b];
      c += pcount[w * nb + b];
    }
  }
  ls[y][x] = s;
  lc[y][x] = c;
  __syncthreads();
  for (int h = 16; h > 0; h >>= 1) {
    if (y < h) {
      ls[y][x] += ls[y + h][x];
      lc[y][x] += lc[y + h][x];
    }
    __syncthreads();
  }
  if (y == 0 && b < nb) {
    sigma[b] = ls[0][x] / bin_area(re, (int)(b / n_mb), column);
    if (count) count[b] = lc[0][x];
  }
}

// Every particle adds to global memory; bound by the rate of the atomics.  A
// workgroup takes a contiguous range, so that in particles stored by radius the
// workgroups at work at one time fall on different bins (2e6 of them in 2000 x 4
// bins: 151 us, in strides over the whole grid 239).
__global__ __launch_bounds__(256) void k_hist_global(const double *__restrict__ r,
                                                     const double *__restrict__ m,
                                                     const double *__restrict__ M,
                                                     const uint8_t *__restrict__ active, int64_t N,
                                                     int64_t chunk, const double *re, int n_rb,
                                                     const double *me, int n_mb,
                                                     double *sigma, uint32_t *count) {
  __shared__ double le[kHistLdsEdges];
  if (n_rb + n_mb + 2 <= kHistLdsEdges) {
    for (int k = threadIdx.x; k <= n_rb; k += blockDim.x) le[k] = re[k];
    for (int k = threadIdx.x; k <= n_mb; k += blockDim.x) le[n_rb + 1 + k] = me[k];
    __syncthreads();
    re = le;
    me = le + n_rb + 1;
  }
  const int64_t i0 = (int64_t)blockIdx.x * chunk;
  const int64_t i1 = i0 + chunk < N ? i0 + chunk : N;
  for (int64_t i = i0 + threadIdx.x; i < i1; i += blockDim.x) {
    if (!active[i]) continue;
    const int k = find_bin(re, n_rb, r[i]);
    const int l = find_bin(me, n_mb, m[i]);
    if (k < 0 || l < 0) continue;
    const int64_t b = (int64_t)k * n_mb + l;
    unsafeAtomicAdd(&sigma[b], M[i]);
    if (count) atomicAdd(&count[b], 1u);
  }
}

__global__ __launch_bounds__(256) void k_hist_area(double *sigma, const double *re, int n_rb,
                                                   int n_mb, int column) {
  const int64_t b = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (b >= (int64_t)n_rb * n_mb) return;
  sigma[b] /= bin_area(re, (int)(b / n_mb), column);
}

// one edge a thread, from the launch's arguments
__global__ __launch_bounds__(kArgEdges) void k_put_edges(EdgeArgs a, int n, double *dst) {
  const int k = threadIdx.x;
  if (k < n) dst[k] = a.e[k];
}

hipError_t launch_put_edges(const double *host, int n, double *dst, hipStream_t s) {
  EdgeArgs a{};
  for (int k = 0; k < n; ++k) a.e[k] = host[k];
  k_put_edges<<<1, kArgEdges, 0, s>>>(a, n, dst);
  return hipGetLastError();
}

hipError_t launch_sigma_hist(const double *r, const double *m, const double *M,
                             const uint8_t *active, int64_t N, const double *re, int n_rb,
                             const double *me, int n_mb, int column, double *sigma,
                             uint32_t *count, int cus, void *scratch, size_t scratch_bytes,
                             hipStream_t s) {
  const int64_t nb = (int64_t)n_rb * n_mb;
  const int rows = std::min(n_rb, kHistLdsBins / n_mb);  // radial rows per workgroup
  const int parts = rows > 0 ? (n_rb + rows - 1) / rows : kHistParts + 1;
  const int ne = n_rb + n_mb + 2;
  // workgroups: one per CU, each with a full round of particles and a row of
  // scratch.  Below 5 particles a bin clearing and adding up the rows takes
  // longer than the atomics (120 x 140 bins: at 4.5e4 particles 31.6 against
  // 27.0 us, at 8e4 30.5 against 30.7; 60 x 90 bins, 3e4: 23.0 against 25.7; all
  // with 12 us of host work that the call no longer has).  Few bins are in LDS
  // for any number of particles and edges: 16 against 19 us, and where the
  // particles share bins, whose atomics wait for one another, 17 against 275
  // (20479 in one of 64 x 64 bins)
  int64_t gw = std::min<int64_t>(std::max(1, cus / parts), (N + kHistThreads - 1) / kHistThreads);
  gw = std::min<int64_t>(gw, (int64_t)(scratch_bytes / ((size_t)nb * 12)));
  const bool few = nb <= kHistFewBins;
  if (few || (N >= 5 * nb && gw >= 1 && parts <= kHistParts && ne <= kHistLdsEdges)) {
    const bool alone = gw < 1;  // too few particles for a row of scratch: one workgroup
    gw = std::max<int64_t>(gw, 1);
    const int64_t chunk = (N + gw - 1) / gw;
    const size_t lds = (size_t)ne * 8 + (size_t)rows * n_mb * 12;
    hipError_t e = hipSuccess;
    if (lds > 64 * 1024)
      e = hipFuncSetAttribute((const void *)k_hist_lds, hipFuncAttributeMaxDynamicSharedMemorySize,
                              (int)lds);
    if (e != hipSuccess) return e;
    double *psum = alone ? sigma : (double *)scratch;
    uint32_t *pcount = alone ? count : (uint32_t *)(psum + gw * nb);
    k_hist_lds<<<dim3((unsigned)gw, (unsigned)parts), kHistThreads, lds, s>>>(
        r, m, M, active, N, chunk, re, n_rb, me, n_mb, rows, psum, pcount);
    if (alone) {
      k_hist_area<<<(unsigned)((nb + 255) / 256), 256, 0, s>>>(sigma, re, n_rb, n_mb, column);
      return hipGetLastError();
    }
    k_hist_reduce<<<(unsigned)((nb + 31) / 32), 1024, 0, s>>>(psum, pcount, (int)gw, re, n_rb, n_mb,
                                                              column, sigma, count);
    return hipGetLastError();
  }
  const unsigned gb = (unsigned)std::min<int64_t>((nb + 255) / 256, 4096);
  k_hist_clear<<<gb, 256, 0, s>>>(sigma, count, nb);
  const int64_t gp = std::max<int64_t>(1, std::min<int64_t>((N + 255) / 256, 4 * (int64_t)cus));
  const int64_t chunk = (N + gp - 1) / gp;
  k_hist_global<<<(unsigned)gp, 256, 0, s>>>(r, m, M, active, N, chunk, re, n_rb, me, n_mb, sigma,
                                             count);
  k_hist_area<<<(unsigned)((nb + 255) / 256), 256, 0, s>>>(sigma, re, n_rb, n_mb, column);
  return hipGetLastError();
}

}  // namespace mcd
