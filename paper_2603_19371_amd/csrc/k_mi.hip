// Mutual-information similarity of one LM attempt (Sec. 2.2: minimise
// (log2 B - MI)^2), from a B x B joint histogram with cubic B-spline Parzen
// windows.  Each image's values are mapped to bin coordinates
// 1 + (B - 3)(v - lo)/(hi - lo) ([lo, hi] its range over the volume, the
// moving range extended to 0, the value outside the volume), so every
// window's four bins lie inside [0, B).
//
//   k_mi_range   per-block minima and maxima of F and M; k_mi_range_final
//                turns them into the two affine maps (order-free: min/max)
//   k_mi_hist    per-block joint histograms of the window products (FP64),
//                summed
//                exactly as fixed-point integers (2^-32 per unit), so the
//                result does not depend on the order of the additions
//   k_mi_fold    sums the block histograms in groups of kMiFold (exact)
//   k_mi_reduce  one block: the exact sums of the groups, p, the marginals,
//                MI (FP64, fixed order) and the table log2(p_ab / p_b) of the
//                gradient; then the decision on L = -MI
//   k_mi_bwd     g = N dr/du = -(sum_ab w_a(F) w'_b(Mw) s_M log2(p_ab/p_b)) dMw
#include <algorithm>

#include "decide.h"
#include "lmr_internal.h"

namespace lmr {

namespace {

constexpr int kMiThreads = 256;
constexpr int kMiHistThreads = 1024;
constexpr double kFix = 4294967296.0;  // 2^32

// The windows and bin coordinates are evaluated in FP64: the gradient of MI
// sums products of windows and log-ratios that vary quickly with the bin
// coordinate, and FP32 coordinates (2^-24 of up to B) would move the step
// by ~1e-5 of its size.
// The four windows of bin coordinate c: bins k0 .. k0+3, k0 = floor(c) - 1.
// Their distances lie in [1, 2), [0, 1), (0, 1] and (1, 2], so each window
// has one polynomial and no branch (at distance 1 the two pieces agree, at 2
// the outer one is 0).  A coordinate that is not a number has no window.
__device__ __forceinline__ int windows(double c, double w[4]) {
  const double fl = floor(c);
  const int k0 = static_cast<int>(fl) - 1;
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const double a = fabs(c - static_cast<double>(k0 + j));
    double v;
    if (j == 0 || j == 3) {
      const double b = 2.0 - a;
      v = b * b * b * (1.0 / 6.0);
    } else {
      v = 2.0 / 3.0 - a * a + 0.5 * a * a * a;
    }
    w[j] = a < 2.0 ? v : 0.0;
  }
  return k0;
}
// Their derivatives with respect to c.
__device__ __forceinline__ int dwindows(double c, double w[4]) {
  const double fl = floor(c);
  const int k0 = static_cast<int>(fl) - 1;
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const double a = fabs(c - static_cast<double>(k0 + j));
    const double sgn = j < 2 ? 1.0 : -1.0;
    double v;
    if (j == 0 || j == 3) {
      const double b = 2.0 - a;
      v = -sgn * 0.5 * b * b;
    } else {
      v = sgn * (-2.0 * a + 1.5 * a * a);
    }
    w[j] = a < 2.0 ? v : 0.0;
  }
  return k0;
}

template <typename T>
__global__ void __launch_bounds__(kMiThreads)
    k_mi_range(const T* __restrict__ F, const T* __restrict__ M, long long N,
               float* __restrict__ part) {
  float fl = INFINITY, fh = -INFINITY, ml = INFINITY, mh = -INFINITY;
  for (long long i = blockIdx.x * (long long)kMiThreads + threadIdx.x; i < N;
       i += (long long)gridDim.x * kMiThreads) {
    const float f = ldf(F, static_cast<int>(i)), m = ldf(M, static_cast<int>(i));
    fl = fminf(fl, f);
    fh = fmaxf(fh, f);
    ml = fminf(ml, m);
    mh = fmaxf(mh, m);
  }
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) {
    fl = fminf(fl, __shfl_xor(fl, off, 64));
    fh = fmaxf(fh, __shfl_xor(fh, off, 64));
    ml = fminf(ml, __shfl_xor(ml, off, 64));
    mh = fmaxf(mh, __shfl_xor(mh, off, 64));
  }
  __shared__ float red[4][kMiThreads / 64];
  const int wv = threadIdx.x >> 6;
  if ((threadIdx.x & 63) == 0) {
    red[0][wv] = fl;
    red[1][wv] = fh;
    red[2][wv] = ml;
    red[3][wv] = mh;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int k = 1; k < kMiThreads / 64; ++k) {
      red[0][0] = fminf(red[0][0], red[0][k]);
      red[1][0] = fmaxf(red[1][0], red[1][k]);
      red[2][0] = fminf(red[2][0], red[2][k]);
      red[3][0] = fmaxf(red[3][0], red[3][k]);
    }
#pragma unroll
    for (int q = 0; q < 4; ++q) part[4 * blockIdx.x + q] = red[q][0];
  }
}

// map[0..3] = (lo_F, s_F, lo_M, s_M) with s = (B - 3) / (hi - lo) (FP64).
// One wave: a lane takes every 64th block's ranges (min and max do not depend
// on the order; one thread over 256 blocks took 27 us).
__global__ void __launch_bounds__(64)
    k_mi_range_final(const float* __restrict__ part, int nblocks, int bins,
                     double* __restrict__ map) {
  float fl = INFINITY, fh = -INFINITY, ml = INFINITY, mh = -INFINITY;
  for (int b = threadIdx.x; b < nblocks; b += 64) {
    const float4 q = reinterpret_cast<const float4*>(part)[b];
    fl = fminf(fl, q.x);
    fh = fmaxf(fh, q.y);
    ml = fminf(ml, q.z);
    mh = fmaxf(mh, q.w);
  }
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) {
    fl = fminf(fl, __shfl_xor(fl, off, 64));
    fh = fmaxf(fh, __shfl_xor(fh, off, 64));
    ml = fminf(ml, __shfl_xor(ml, off, 64));
    mh = fmaxf(mh, __shfl_xor(mh, off, 64));
  }
  if (threadIdx.x != 0) return;
  ml = fminf(ml, 0.0f);
  mh = fmaxf(mh, 0.0f);
  double df = static_cast<double>(fh) - fl, dm = static_cast<double>(mh) - ml;
  if (!(df > 0.0)) df = 1.0;
  if (!(dm > 0.0)) dm = 1.0;
  map[0] = fl;
  map[1] = (bins - 3) / df;
  map[2] = ml;
  map[3] = (bins - 3) / dm;
}

// A block keeps kMiCopies copies of the histogram in LDS, entry k of copy q
// at k * kMiCopies + q, and lane l adds to copy l % kMiCopies.  Most voxels
// of an image share a few bins (the background), so with one copy per wave
// nearly every lane of an addition hits the same entry and they are served
// one after another; here at most 64 / kMiCopies do, and the copies of an
// entry lie on different banks (96x80x96, 32 bins: 38 -> 12.5 us).  A product
// of two windows is below 4/9, so its fixed-point form fits 32 bits.
constexpr int kMiCopies = 16;
template <typename T>
__global__ void __launch_bounds__(kMiHistThreads)
    k_mi_hist(const T* __restrict__ F, const float* __restrict__ Mw, long long N, int bins,
              const double* __restrict__ map, unsigned long long* __restrict__ part,
              const DevState* __restrict__ st) {
  if (st && st->stalled) return;
  extern __shared__ unsigned long long h[];  // [bins * bins][kMiCopies]
  const int BB = bins * bins;
  for (int k = threadIdx.x; k < kMiCopies * BB; k += kMiHistThreads) h[k] = 0ull;
  __syncthreads();
  const double flo = map[0], sf = map[1], mlo = map[2], sm = map[3];
  unsigned long long* hq = h + threadIdx.x % kMiCopies;
  for (long long i = blockIdx.x * (long long)kMiHistThreads + threadIdx.x; i < N;
       i += (long long)gridDim.x * kMiHistThreads) {
    double wa[4], wb[4];
    const int a0 = windows(1.0 + (static_cast<double>(ldf(F, static_cast<int>(i))) - flo) * sf,
                           wa);
    const int b0 = windows(1.0 + (static_cast<double>(Mw[i]) - mlo) * sm, wb);
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int a = a0 + j;
      if (a < 0 || a >= bins || wa[j] == 0.0) continue;
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const int b = b0 + k;
        if (b < 0 || b >= bins || wb[k] == 0.0) continue;
        atomicAdd(&hq[(a * bins + b) * kMiCopies],
                  static_cast<unsigned long long>(
                      static_cast<unsigned>(wa[j] * wb[k] * kFix + 0.5)));
      }
    }
  }
  __syncthreads();
  // consecutive threads start at different copies of an entry: 16 reads on
  // distinct banks
  for (int k = threadIdx.x; k < BB; k += kMiHistThreads) {
    unsigned long long s = 0ull;
#pragma unroll
    for (int q = 0; q < kMiCopies; ++q) s += h[k * kMiCopies + (q + k) % kMiCopies];
    part[(long long)blockIdx.x * BB + k] = s;
  }
}

// fold[g] = the sum of block histograms kMiFold g .. kMiFold g + kMiFold - 1.
// The block histograms are 2 MB at 32 bins: one block alone reads them at the
// rate of one compute unit (66 us with the reduction; 4.5 + 9 us in two steps).
__global__ void __launch_bounds__(kMiThreads)
    k_mi_fold(const unsigned long long* __restrict__ part, int nblocks, int BB,
              unsigned long long* __restrict__ fold, const DevState* __restrict__ st) {
  if (st && st->stalled) return;
  const int k = blockIdx.x * kMiThreads + threadIdx.x, b0 = blockIdx.y * kMiFold;
  if (k >= BB) return;
  unsigned long long s = 0ull;
#pragma unroll
  for (int j = 0; j < kMiFold; ++j)
    if (b0 + j < nblocks) s += part[(long long)(b0 + j) * BB + k];
  fold[(long long)blockIdx.y * BB + k] = s;
}

constexpr int kMiReduceThreads = 1024;
constexpr int kMiMaxBins = 32;

// One block.  tab (FP64 [B*B], log2(p_ab / p_b), 0 where p_ab = 0) for the
// gradient, MI and the decision on it: MI is one number, so a launch of its
// own for the decision would only wait for it (5 us).  A frozen pair is left
// as it is but for the record that nothing was accepted.
__global__ void __launch_bounds__(kMiReduceThreads)
    k_mi_reduce(const unsigned long long* __restrict__ fold, int ngroups, int bins,
                long long N, double* __restrict__ tab, DevState* st, MiDecision md) {
  DevState cur{};
  if (md.mode == 0) {
    cur = *st;
    if (cur.stalled) {
      if (threadIdx.x == 0) st->accepted = 0;
      return;
    }
  }
  const int BB = bins * bins;
  const double inv = 1.0 / (static_cast<double>(N) * kFix);
  __shared__ double p[kMiMaxBins * (kMiMaxBins + 1)];  // rows of bins + 1
  const int t = threadIdx.x, a = t / bins, b = t % bins;
  if (t < BB) {
    unsigned long long s = 0ull;
#pragma unroll 8
    for (int g = 0; g < ngroups; ++g) s += fold[(long long)g * BB + t];
    p[a * (bins + 1) + b] = static_cast<double>(s) * inv;
  }
  __syncthreads();
  __shared__ double pa[kMiMaxBins], pb[kMiMaxBins];
  if (t < bins) {
    double sa = 0.0, sb = 0.0;
    for (int j = 0; j < bins; ++j) {
      sa += p[t * (bins + 1) + j];
      sb += p[j * (bins + 1) + t];
    }
    pa[t] = sa;
    pb[t] = sb;
  }
  __syncthreads();
  double mi = 0.0;
  if (t < BB) {
    const double v = p[a * (bins + 1) + b];
    if (v > 0.0) {
      mi = v * log2(v / (pa[a] * pb[b]));
      tab[t] = log2(v / pb[b]);
    } else {
      tab[t] = 0.0;
    }
  }
  // fixed-order block sum of the per-thread terms
  __shared__ double red[kMiReduceThreads];
  red[threadIdx.x] = mi;
  __syncthreads();
  for (int w = kMiReduceThreads / 2; w > 0; w >>= 1) {
    if (threadIdx.x < w) red[threadIdx.x] += red[threadIdx.x + w];
    __syncthreads();
  }
  if (threadIdx.x == 0)
    decide_write(st, cur, -(red[0] * static_cast<double>(N)) / static_cast<double>(N), md.dp,
                 md.mode, md.force, md.lambda0, md.probe);
}

template <typename T>
__global__ void __launch_bounds__(kMiThreads)
    k_mi_bwd(const T* __restrict__ F, const float* __restrict__ Mw, const float* dMw,
             long long N, int bins, const double* __restrict__ map,
             const double* __restrict__ tab, const DevState* __restrict__ st, float* graw) {
  if (st && (st->stalled || !st->accepted)) return;
  // the table in LDS: a voxel reads 16 of its entries
  __shared__ double s_tab[kMiMaxBins * kMiMaxBins];
  for (int k = threadIdx.x; k < bins * bins; k += kMiThreads) s_tab[k] = tab[k];
  __syncthreads();
  const double flo = map[0], sf = map[1], mlo = map[2], sm = map[3];
  for (long long i = blockIdx.x * (long long)kMiThreads + threadIdx.x; i < N;
       i += (long long)gridDim.x * kMiThreads) {
    double wa[4], wb[4];
    const int a0 = windows(1.0 + (static_cast<double>(ldf(F, static_cast<int>(i))) - flo) * sf,
                           wa);
    const int b0 = dwindows(1.0 + (static_cast<double>(Mw[i]) - mlo) * sm, wb);
    double s = 0.0;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int a = a0 + j;
      if (a < 0 || a >= bins) continue;
      double t = 0.0;
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const int b = b0 + k;
        if (b < 0 || b >= bins) continue;
        t += wb[k] * s_tab[a * bins + b];
      }
      s += wa[j] * t;
    }
    const float d = static_cast<float>(-s * sm);  // -dMI/dMw (times N)
    const float n0 = dMw[i], n1 = dMw[N + i], n2 = dMw[2 * N + i];
    graw[i] = d * n0;
    graw[N + i] = d * n1;
    graw[2 * N + i] = d * n2;
  }
}

unsigned mi_blocks(long long N) {
  long long b = (N + kMiHistThreads * 2 - 1) / (kMiHistThreads * 2);
  if (b > kMiBlocks) b = kMiBlocks;
  return static_cast<unsigned>(b < 1 ? 1 : b);
}

}  // namespace

hipError_t launch_mi_range(const void* F, const void* M, lmr_dtype t, const Geom& g, int bins,
                           float* part, double* map, hipStream_t s) {
  const unsigned nb = mi_blocks(g.N);
  if (t == LMR_BF16)
    hipLaunchKernelGGL(k_mi_range<uint16_t>, dim3(nb), dim3(kMiThreads), 0, s,
                       static_cast<const uint16_t*>(F), static_cast<const uint16_t*>(M), g.N,
                       part);
  else
    hipLaunchKernelGGL(k_mi_range<float>, dim3(nb), dim3(kMiThreads), 0, s,
                       static_cast<const float*>(F), static_cast<const float*>(M), g.N, part);
  hipLaunchKernelGGL(k_mi_range_final, dim3(1), dim3(64), 0, s, part, static_cast<int>(nb),
                     bins, map);
  return hipGetLastError();
}

hipError_t launch_mi_fwd(const void* F, lmr_dtype t, const float* Mw, const Geom& g, int bins,
                         const double* map, unsigned long long* hpart, double* tab,
                         DevState* state, const MiDecision& md, hipStream_t s) {
  const DevState* st = md.mode == 0 ? state : nullptr;  // attempts skip a frozen pair
  if (bins < 1 || bins > kMiMaxBins) return hipErrorInvalidValue;
  const unsigned nb = mi_blocks(g.N), ngroups = (nb + kMiFold - 1) / kMiFold;
  const int BB = bins * bins;
  const size_t lds = sizeof(unsigned long long) * kMiCopies * BB;
  unsigned long long* fold = hpart + static_cast<size_t>(kMiBlocks) * BB;
  if (t == LMR_BF16)
    hipLaunchKernelGGL(k_mi_hist<uint16_t>, dim3(nb), dim3(kMiHistThreads), lds, s,
                       static_cast<const uint16_t*>(F), Mw, g.N, bins, map, hpart, st);
  else
    hipLaunchKernelGGL(k_mi_hist<float>, dim3(nb), dim3(kMiHistThreads), lds, s,
                       static_cast<const float*>(F), Mw, g.N, bins, map, hpart, st);
  hipLaunchKernelGGL(k_mi_fold, dim3((BB + kMiThreads - 1) / kMiThreads, ngroups),
                     dim3(kMiThreads), 0, s, hpart, static_cast<int>(nb), BB, fold, st);
  hipLaunchKernelGGL(k_mi_reduce, dim3(1), dim3(kMiReduceThreads), 0, s, fold,
                     static_cast<int>(ngroups), bins, g.N, tab, state, md);
  return hipGetLastError();
}

hipError_t launch_mi_bwd(const void* F, lmr_dtype t, const float* Mw, const float* dMw,
                         const Geom& g, int bins, const double* map, const double* tab,
                         const DevState* st, float* graw, hipStream_t s) {
  const unsigned nb = static_cast<unsigned>(std::min<long long>((g.N + 255) / 256, 4096));
  if (t == LMR_BF16)
    hipLaunchKernelGGL(k_mi_bwd<uint16_t>, dim3(nb), dim3(kMiThreads), 0, s,
                       static_cast<const uint16_t*>(F), Mw, dMw, g.N, bins, map, tab, st,
                       graw);
  else
    hipLaunchKernelGGL(k_mi_bwd<float>, dim3(nb), dim3(kMiThreads), 0, s,
                       static_cast<const float*>(F), Mw, dMw, g.N, bins, map, tab, st, graw);
  return hipGetLastError();
}

}  // namespace lmr
