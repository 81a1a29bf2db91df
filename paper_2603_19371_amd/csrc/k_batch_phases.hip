// Batched form without the persistent kernel: each phase of an attempt is one
// launch over the work items of all pairs (one item per block), so the
// kernel boundaries order the phases instead of grid barriers, and every
// phase kernel has the registers, and so the occupancy, of its own work
// (batch_attempt.h holds the items).  A phase whose pairs run on both forms
// is launched once per form, each launch skipping the other form's items.
#include "batch_attempt.h"

namespace lmr {

namespace {

template <typename T>
__global__ void __launch_bounds__(kNT) k_bp_update(const BatchPair* __restrict__ pairs,
                                                   int npairs) {
  __shared__ StagedLds lds;
  update_item<T>(pairs, npairs, blockIdx.x, lds);
}

// BEGIN: the state of a pair on bricks at the identity.
template <bool BEGIN>
__global__ void __launch_bounds__(kNT) k_bp_decide(const BatchPair* __restrict__ pairs,
                                                   DecideParams dp) {
  const BatchPair& P = pairs[blockIdx.x];
  if (BEGIN && !P.bricks) return;
  decide_pair(P, dp, BEGIN);
}

// The begin of the pairs on bricks: U0 = 0, the image warped by it and its
// derivative, on the columns of the update's work items (256 threads write 28
// bytes a voxel; bound by those stores).  The state is set by k_bp_decide
// once there is a loss; the forward pass before it only asks whether the
// pair is frozen.
template <typename T>
__global__ void __launch_bounds__(kNT) k_bp_start(const BatchPair* __restrict__ pairs,
                                                  int npairs) {
  const BatchPair& P = pairs[owner(pairs, npairs, blockIdx.x, &BatchPair::utile0)];
  if (!P.bricks) return;
  const int local = blockIdx.x - P.utile0;
  if (local == 0 && threadIdx.x == 0) P.st->stalled = 0;
  const int tx = (P.g.nx + kBatchUpdateTX - 1) / kBatchUpdateTX,
            ty = (P.g.ny + kBatchUpdateTY - 1) / kBatchUpdateTY;
  const int x = (local % tx) * kBatchUpdateTX + static_cast<int>(threadIdx.x) % kBatchUpdateTX;
  const int y =
      ((local / tx) % ty) * kBatchUpdateTY + static_cast<int>(threadIdx.x) / kBatchUpdateTX;
  const int z0 = (local / (tx * ty)) * P.ucz, z1 = min(z0 + P.ucz, P.g.nz);
  if (x >= P.g.nx || y >= P.g.ny) return;
  const int N = static_cast<int>(P.g.N);
  const RBuf bm = make_rbuf_n(static_cast<const T*>(P.M), N);
  for (int z = z0; z < z1; ++z) {
    const int i = (z * P.g.ny + y) * P.g.nx + x;
    const BCell c = make_bcell(P.g, x, y, z, 0.0f, 0.0f, 0.0f);
    float v[8], d[3];
    bcorners<T>(bm, P.g, c, v);
    P.Mw[i] = binterp(c, v, d);
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      P.U0[k * N + i] = 0.0f;
      P.graw[k * N + i] = d[k];
    }
  }
}

// The stencil phases of the marching pairs, one tile per block.
template <int RB, typename T, typename Acc>
__global__ void __launch_bounds__(kNT) k_bp_fwd(const BatchPair* __restrict__ pairs,
                                                int npairs) {
  __shared__ StencilLds<RB, kTY, FwdPol<T, kNT, Acc>> lds;
  char none;
  fwd_item<RB, T, Acc, 0>(pairs, npairs, blockIdx.x, lds, none);
}

template <int RB, typename T, typename Acc>
__global__ void __launch_bounds__(kNT) k_bp_bwd(const BatchPair* __restrict__ pairs,
                                                int npairs) {
  __shared__ StencilLds<RB, kTY, BwdPol<T, Acc>> lds;
  char none;
  bwd_item<RB, T, Acc, 0>(pairs, npairs, blockIdx.x, lds, none);
}

template <int RG>
__global__ void __launch_bounds__(kNT) k_bp_smooth(const BatchPair* __restrict__ pairs,
                                                   int npairs) {
  __shared__ StencilLds<RG, kTY, SmoothPol<RG>> lds;
  char none;
  smooth_item<RG, 0>(pairs, npairs, blockIdx.x, lds, none);
}

// And of the pairs on bricks, one brick per block: wide ones (32 pairs of
// about 48^3 on small bricks, then wide ones: forward 82 -> 68 us, backward of
// accepted pairs 125 -> 95, smoothing 68 -> 50), but small ones where all
// pairs together have fewer than kWideItems wide ones (attempts: with 24 to 90
// wide ones small 11 to 19 % faster; 96 to 192, nine batches, either up to 7 %;
// from 300 on wide 5 to 27 % faster but for pairs that pad them, 64 of 16x20x24:
// 70 us, small 63, and for one pair of 64x64x72, 320 of them: 53, 49).
constexpr int kWideItems = 96;

template <int R, bool WIDE, class Pol>
using BatchBrickLds = BrickLds<R, Pol, WIDE ? kWide : kT3>;
template <bool WIDE>
constexpr int kBrickThreads = WIDE ? kWideThreads : kCubeThreads;

template <bool WIDE>
__device__ __forceinline__ const BatchPair& brick_pair(const BatchPair* __restrict__ pairs,
                                                       int npairs, int& local) {
  const BatchPair& P = pairs[owner(pairs, npairs, blockIdx.x,
                                   WIDE ? &BatchPair::wide0 : &BatchPair::tile0)];
  local = blockIdx.x - (WIDE ? P.wide0 : P.tile0);
  return P;
}

template <int R, bool WIDE, class Pol>
__device__ __forceinline__ void brick_item(const Pol& pol, const BatchPair& P, int local,
                                           BatchBrickLds<R, WIDE, Pol>& lds) {
  int x0, y0, z0;
  auto loc = pol.begin_block(nullptr);
  if constexpr (WIDE) {
    brick_origin<kWide>(P.g, local, x0, y0, z0);
    WideFetch<R, Pol> f;
    wide_fetch<R>(pol, P.g, x0, y0, z0, loc, f);
    stencil_wide<R>(pol, P.g, x0, y0, z0, loc, f, lds, true, 0);
  } else {
    brick_origin<kT3>(P.g, local, x0, y0, z0);
    stencil_cube<R>(pol, P.g, x0, y0, z0, loc, lds);
    pol.end_tile(loc, local);
  }
}

template <int RB, bool WIDE, typename T, typename Acc>
__global__ void __launch_bounds__(kBrickThreads<WIDE>)
    k_bp_fstat_bricks(const BatchPair* __restrict__ pairs, int npairs) {
  __shared__ BatchBrickLds<RB, WIDE, FStatPol<T, Acc>> lds;
  int local;
  const BatchPair& P = brick_pair<WIDE>(pairs, npairs, local);
  if (!P.bricks) return;
  FStatPol<T, Acc> pol;
  pol.F = static_cast<const T*>(P.F);
  pol.fstat = P.fstat;
  pol.N = static_cast<int>(P.g.N);
  pol.inv_n = P.inv_n;
  brick_item<RB, WIDE>(pol, P, local, lds);
}

template <int RB, bool WIDE, typename T, typename Acc>
__global__ void __launch_bounds__(kBrickThreads<WIDE>)
    k_bp_fwd_bricks(const BatchPair* __restrict__ pairs, int npairs) {
  __shared__ BatchBrickLds<RB, WIDE, FwdPol<T, kNT, Acc>> lds;
  int local;
  const BatchPair& P = brick_pair<WIDE>(pairs, npairs, local);
  if (!P.bricks || P.st->stalled) return;
  brick_item<RB, WIDE>(fwd_policy<T, Acc>(P), P, local, lds);
}

template <int RB, bool WIDE, typename T, typename Acc>
__global__ void __launch_bounds__(kBrickThreads<WIDE>)
    k_bp_bwd_bricks(const BatchPair* __restrict__ pairs, int npairs) {
  __shared__ BatchBrickLds<RB, WIDE, BwdPol<T, Acc>> lds;
  int local;
  const BatchPair& P = brick_pair<WIDE>(pairs, npairs, local);
  if (!P.bricks || P.st->stalled || !P.st->accepted) return;
  brick_item<RB, WIDE>(bwd_policy<T, Acc>(P), P, local, lds);
}

template <int RG, bool WIDE>
__global__ void __launch_bounds__(kBrickThreads<WIDE>)
    k_bp_smooth_bricks(const BatchPair* __restrict__ pairs, int npairs) {
  __shared__ BatchBrickLds<RG, WIDE, SmoothPol<RG>> lds;
  int local;
  const BatchPair& P = brick_pair<WIDE>(pairs, npairs, local);
  if (!P.bricks || P.st->stalled || !P.st->accepted) return;
  brick_item<RG, WIDE>(smooth_policy<RG>(P), P, local, lds);
}

struct PhaseLaunch {
  const BatchPair* pairs;
  int npairs, n_update_items, n_tiles, n_wide;
  bool march;
  hipStream_t s;
};

enum class Box { kStat, kFwd, kBwd };

template <int RB, bool WIDE, typename T, typename Acc>
void launch_box_bricks(const PhaseLaunch& L, Box what) {
  const dim3 grid(WIDE ? L.n_wide : L.n_tiles), blk(kBrickThreads<WIDE>);
  if (what == Box::kStat)
    hipLaunchKernelGGL((k_bp_fstat_bricks<RB, WIDE, T, Acc>), grid, blk, 0, L.s, L.pairs,
                       L.npairs);
  else if (what == Box::kFwd)
    hipLaunchKernelGGL((k_bp_fwd_bricks<RB, WIDE, T, Acc>), grid, blk, 0, L.s, L.pairs,
                       L.npairs);
  else
    hipLaunchKernelGGL((k_bp_bwd_bricks<RB, WIDE, T, Acc>), grid, blk, 0, L.s, L.pairs,
                       L.npairs);
}

template <int RB, typename T, typename Acc>
void launch_box(const PhaseLaunch& L, Box what) {
  if (L.march) {
    const dim3 grid(L.n_tiles), blk(kNT);
    if (what == Box::kFwd)
      hipLaunchKernelGGL((k_bp_fwd<RB, T, Acc>), grid, blk, 0, L.s, L.pairs, L.npairs);
    else
      hipLaunchKernelGGL((k_bp_bwd<RB, T, Acc>), grid, blk, 0, L.s, L.pairs, L.npairs);
  }
  if (L.n_wide >= kWideItems)
    launch_box_bricks<RB, true, T, Acc>(L, what);
  else if (L.n_wide)
    launch_box_bricks<RB, false, T, Acc>(L, what);
}

template <int RG>
void launch_smooth_forms(const PhaseLaunch& L) {
  if (L.march)
    hipLaunchKernelGGL((k_bp_smooth<RG>), dim3(L.n_tiles), dim3(kNT), 0, L.s, L.pairs,
                       L.npairs);
  if (L.n_wide >= kWideItems)
    hipLaunchKernelGGL((k_bp_smooth_bricks<RG, true>), dim3(L.n_wide),
                       dim3(kBrickThreads<true>), 0, L.s, L.pairs, L.npairs);
  else if (L.n_wide)
    hipLaunchKernelGGL((k_bp_smooth_bricks<RG, false>), dim3(L.n_tiles),
                       dim3(kBrickThreads<false>), 0, L.s, L.pairs, L.npairs);
}

// One attempt, or the begin of the pairs on bricks.
template <bool BEGIN, typename T, typename Acc>
hipError_t phases_t(const PhaseLaunch& L, int rb, int rg, const DecideParams& dp) {
  auto box = [&](Box what) {
    switch (rb) {
      case 1: launch_box<1, T, Acc>(L, what); break;
      case 2: launch_box<2, T, Acc>(L, what); break;
      case 3: launch_box<3, T, Acc>(L, what); break;
      case 4: launch_box<4, T, Acc>(L, what); break;
    }
  };
  if (rb < 1 || rb > 4 || rg < 0 || rg > 4) return hipErrorInvalidValue;
  if constexpr (BEGIN) {
    hipLaunchKernelGGL(k_bp_start<T>, dim3(L.n_update_items), dim3(kNT), 0, L.s, L.pairs,
                       L.npairs);
    box(Box::kStat);
  } else {
    hipLaunchKernelGGL(k_bp_update<T>, dim3(L.n_update_items), dim3(kNT), 0, L.s, L.pairs,
                       L.npairs);
  }
  box(Box::kFwd);
  hipLaunchKernelGGL(k_bp_decide<BEGIN>, dim3(L.npairs), dim3(kNT), 0, L.s, L.pairs, dp);
  box(Box::kBwd);
  switch (rg) {
    case 0: launch_smooth_forms<0>(L); break;
    case 1: launch_smooth_forms<1>(L); break;
    case 2: launch_smooth_forms<2>(L); break;
    case 3: launch_smooth_forms<3>(L); break;
    case 4: launch_smooth_forms<4>(L); break;
  }
  return hipGetLastError();
}

}  // namespace

namespace {

template <bool BEGIN>
hipError_t phases(const PhaseLaunch& L, lmr_dtype t, lmr_accum accum, int rb, int rg,
                  const DecideParams& dp) {
  if (accum == LMR_ACC_F32C)
    return t == LMR_BF16 ? phases_t<BEGIN, uint16_t, F32C>(L, rb, rg, dp)
                         : phases_t<BEGIN, float, F32C>(L, rb, rg, dp);
  return t == LMR_BF16 ? phases_t<BEGIN, uint16_t, double>(L, rb, rg, dp)
                       : phases_t<BEGIN, float, double>(L, rb, rg, dp);
}

}  // namespace

hipError_t launch_batch_phases(lmr_dtype t, lmr_accum accum, int box_radius,
                               int gauss_radius, bool march, const BatchPair* pairs,
                               int npairs, int n_update_items, int n_tiles, int n_wide,
                               const DecideParams& dp, hipStream_t s) {
  return phases<false>(PhaseLaunch{pairs, npairs, n_update_items, n_tiles, n_wide, march, s}, t,
                       accum, box_radius, gauss_radius, dp);
}

hipError_t launch_batch_begin(lmr_dtype t, lmr_accum accum, int box_radius, int gauss_radius,
                              const BatchPair* pairs, int npairs, int n_update_items,
                              int n_tiles, int n_wide, const DecideParams& dp,
                              hipStream_t s) {
  return phases<true>(PhaseLaunch{pairs, npairs, n_update_items, n_tiles, n_wide, false, s}, t,
                      accum, box_radius, gauss_radius, dp);
}

}  // namespace lmr
