// Per-pair launches of the three stencils of an LM attempt (stencil.h):
// LNCC forward (P2), LNCC + warp backward (P4) and Gaussian smoothing (P5).
// A block per brick, or per one or two tiles of the march; block ids are
// remapped so that each XCD receives a contiguous range of tiles and shares
// their halos in its L2.
#include <algorithm>

#include "decide.h"
#include "pass_decision.h"
#include "stencil.h"

namespace lmr {

namespace {

// The tiling (and with it the chunks, and the partial sums of the forward
// pass) is in 32 x kTY tiles, as in the batched form; a block runs one, or two
// of them, one above the other, on two waves per SIMD, and two such blocks
// share a CU (at most 128 VGPRs a thread).
constexpr int kTY = 8, kMarchTY = 2 * kTY;
__host__ __device__ inline int march_rows(const Tiling& t) {
  return t.pairs ? (t.tiles_y + 1) / 2 : t.tiles_y;
}

// The decision of the attempt inside a pass of NT threads (pass_decision.h):
// every block reduces the partials and decides on the pair state st; block 0
// stores the result in pd.next.  Returns the decided state, in LDS.
template <int NT>
__device__ const DevState* decide_in_pass(const DevState* st, const PassDecision& pd) {
  constexpr int kSumThreads = 256;  // the decision kernel's order of the sum
  __shared__ double sh[kSumThreads];
  __shared__ DevState s_next;
  DevState cur;
  if (threadIdx.x == 0) cur = *st;
  const double S = reduce_partials<kSumThreads, NT>([&](int k) { return pd.partials[k]; },
                                                    pd.nparts, sh);
  if (threadIdx.x == 0) {
    const DevState n = decide_next(cur, -S / static_cast<double>(pd.N), pd.dp, pd.force);
    if (blockIdx.x == 0) *pd.next = n;
    s_next = n;
  }
  __syncthreads();
  return &s_next;
}

// Whether a block of a pass runs, and the state it runs on (rs; null without
// a pair state).  need: 0 always run, 1 skip a frozen pair, 2 run only after
// an acceptance.  DEC: the pass takes the decision first and runs on the
// decided state.  pd.commit: block 0 first stores st there.
template <int NT, bool DEC>
__device__ __forceinline__ bool pass_state(const DevState* st, int need,
                                           const PassDecision& pd, const DevState*& rs) {
  if constexpr (DEC) {
    rs = decide_in_pass<NT>(st, pd);
    return rs->accepted != 0;
  } else {
    rs = st;
    if (pd.commit && blockIdx.x == 0 && threadIdx.x == 0) *pd.commit = *st;
    if (st && need) {
      if (st->stalled) return false;
      if (need == 2 && !st->accepted) return false;
    }
    return true;
  }
}

// Sums of one double per thread over the halves of a block of NT threads, each
// in the order of block_sum_to over a block of NT / 2.
template <int NT>
__device__ __forceinline__ void half_sums_to(double v, double* lower, double* upper) {
  constexpr int kWaves = NT / 64;
  __shared__ double red[kWaves];
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
  __syncthreads();
  if (threadIdx.x % (NT / 2) == 0) {
    const int w0 = threadIdx.x >> 6;
    double s = 0.0;
#pragma unroll
    for (int k = 0; k < kWaves / 2; ++k) s += red[w0 + k];
    double* out = threadIdx.x == 0 ? lower : upper;
    if (out) *out = s;
  }
}

template <int R, int TY, class P, bool DEC>
__global__ void __launch_bounds__(kTX* TY)
    __attribute__((amdgpu_waves_per_eu(TY == kMarchTY ? 4 : 2)))
    k_stencil(const P pol, Geom g, Tiling t, const DevState* st, int need, PassDecision pd) {
  const DevState* rs;
  if (!pass_state<kTX * TY, DEC>(st, need, pd, rs)) return;
  __shared__ StencilLds<R, TY, P> sm[TY == kMarchTY ? 2 : 1];
  const int b = xcd_remap(blockIdx.x, gridDim.x);
  const int rows = TY == kMarchTY ? (t.tiles_y + 1) / 2 : t.tiles_y;  // march_rows(t)
  const int tx = b % t.tiles_x, row = (b / t.tiles_x) % rows, chunk = b / (t.tiles_x * rows);
  const int z0 = chunk * t.cz;
  typename P::Local loc = pol.begin_block(rs);
  const int z1 = min(z0 + t.cz, g.nz);
  // partials in tile order, as in the batched form
  if constexpr (TY == kTY) {
    stencil_tile<R, TY>(pol, g, tx * kTX, row * TY, z0, z1, loc, sm[0]);
    pol.end_tile(loc, b);
    return;
  } else {
    stencil_march<R, TY>(pol, g, tx * kTX, row * TY, z0, z1, loc, sm);
  }
  if constexpr (TY == kMarchTY && P::kSum) {
    double* lower = pol.partials + (chunk * t.tiles_y + 2 * row) * t.tiles_x + tx;
    half_sums_to<kTX * TY>(loc.sum, lower,
                           2 * row + 1 < t.tiles_y ? lower + t.tiles_x : nullptr);
  }
}

// The partial of a deep brick: the sums over its halves, each in the order of
// block_sum_to over a small brick's block, added.
__device__ __forceinline__ void deep_sum_to(double lower, double upper, double* out) {
  constexpr int kWaves = kCubeThreads / 64;
  __shared__ double red[2][kWaves];
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) {
    lower += __shfl_xor(lower, off, 64);
    upper += __shfl_xor(upper, off, 64);
  }
  if ((threadIdx.x & 63) == 0) {
    red[0][threadIdx.x >> 6] = lower;
    red[1][threadIdx.x >> 6] = upper;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    double s[2] = {0.0, 0.0};
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
      for (int k = 0; k < kWaves; ++k) s[h] += red[h][k];
    *out = s[0] + s[1];
  }
}

// The same stencil on small or deep bricks (stencil.h).
template <int R, class P, int DEPTH, bool DEC>
__global__ void __launch_bounds__(kCubeThreads)
    __attribute__((amdgpu_waves_per_eu(DEC ? 4 : 1)))
    k_cube(const P pol, Geom g, const DevState* st, int need, PassDecision pd) {
  const DevState* rs;
  if (!pass_state<kCubeThreads, DEC>(st, need, pd, rs)) return;
  __shared__ BrickLds<R, P, kT3, DEPTH> sm;
  const int b = xcd_remap(blockIdx.x, gridDim.x);
  int x0, y0, z0;
  brick_origin<kT3, DEPTH>(g, b, x0, y0, z0);
  typename P::Local loc = pol.begin_block(rs);
  const double others = stencil_cube<R>(pol, g, x0, y0, z0, loc, sm);
  if constexpr (P::kSum && DEPTH > kBrickZ)
    deep_sum_to(loc.sum, others, pol.partials + b);
  else
    pol.end_tile(loc, b);
}

// And on wide bricks.
template <int R, class P>
__global__ void __launch_bounds__(kWideThreads)
    k_wide(const P pol, Geom g, const DevState* st, int need, PassDecision pd) {
  const DevState* rs;
  if (!pass_state<kWideThreads, false>(st, need, pd, rs)) return;
  __shared__ BrickLds<R, P, kWide> sm;
  const int b = xcd_remap(blockIdx.x, gridDim.x);
  int x0, y0, z0;
  brick_origin<kWide>(g, b, x0, y0, z0);
  typename P::Local loc = pol.begin_block(rs);
  WideFetch<R, P> f;
  wide_fetch<R>(pol, g, x0, y0, z0, loc, f);
  stencil_wide<R>(pol, g, x0, y0, z0, loc, f, sm, false, b);
}

}  // namespace

namespace {

// Chunk length of the march for tiling t.  A launch runs its blocks in rounds
// of as many as are co-resident (two per CU that run two tiles, four that run
// one), and each block of a round marches its chunk plus the 2R halo planes,
// so a launch lasts about rounds x (cz + 2R) plane steps.  Among the chunk
// lengths not below make_tiling's floor, take the one that minimises this (the
// longer chunk on a tie).  Returns the planes that the fullest CU marches,
// counted in tiles.
long long set_chunks(Tiling& t, const Geom& g, int R) {
  const long long cols = (long long)t.tiles_x * march_rows(t);
  const long long cus = device_cus(), cap = (t.pairs ? 2 : 4) * cus;
  const int floor_cz =
      std::min(march_floor_cz((long long)t.tiles_x * t.tiles_y, g.nz), g.nz);
  long long best = -1;
  for (int n = 1; n <= g.nz; ++n) {
    const int cz = (g.nz + n - 1) / n;
    if (cz < floor_cz) break;
    const int chunks = (g.nz + cz - 1) / cz;
    if (chunks != n) continue;  // the same chunk length as a smaller n
    const long long cost = ((cols * chunks + cap - 1) / cap) * (cz + 2 * R);
    if (best < 0 || cost < best) {
      best = cost;
      t.cz = cz;
      t.nchunks = chunks;
    }
  }
  return (t.pairs ? 2 : 1) * ((cols * t.nchunks + cus - 1) / cus) * (t.cz + 2 * R);
}

}  // namespace

// Two tiles per block read a plane's halo rows once for both and have half the
// barriers, so a tile's plane costs them some 3 R percent less than a block of
// one; but an odd row of tiles leaves half of a block idle, and the blocks are
// the coarser load for the CUs.  So they are taken where the fullest CU has at
// most that share of planes more then (attempt, window 7: 160x72x160, 56
// planes either way: one tile 94.9 us, two 91.3; 300x24x300, 60 and 72: 90.2,
// 95.6; 512x8x512, 56 and 88: 84.8, 104.1; 130x70x130, 45 and 60: 81.5, 84.4;
// window 5, 256x40x256, 60 and 68: 93.8, 96.0).  The tiling does not depend on
// the kernel: a box sum's rounding depends on where its chunk starts, and the
// batched form (blocks of one tile) reproduces a pair's run by using the same
// tiling for all passes.
Tiling march_tiling(const Geom& g, int R) {
  Tiling one = make_tiling(g.nz, g.ny, g.nx, kTY), two = one;
  two.pairs = 1;
  const long long c1 = set_chunks(one, g, R), c2 = set_chunks(two, g, R);
  return 100 * c2 <= (100 + 3 * R) * c1 ? two : one;
}

namespace {

// The forward policy's block reduction is sized for its block: one policy
// type serves both forms, so both forms launch blocks of the same size.
static_assert(kTX * kTY == kCubeThreads, "marching tiles and cubes share FwdPol<T, 256>");

// Volumes of at most this many voxels run on cubes under LMR_STENCIL_AUTO
// (the half- and quarter-resolution levels of a brain-sized pair).
constexpr long long kCubeMaxVoxels = 1LL << 20;

// Asked for bricks, a volume marches all the same where they would be more than
// a launch holds (2^32 threads; a slab one voxel thick of half a billion).
constexpr long long kMaxBricks = (1LL << 32) / kWideThreads;

bool use_cubes(const Geom& g, const lmr_params& p) {
  return (p.stencil == LMR_STENCIL_CUBE && bricks_of(g, kT3, kBrickZ) < kMaxBricks) ||
         (p.stencil == LMR_STENCIL_AUTO && g.N <= kCubeMaxVoxels);
}

// The bricks of a pass.  Blocks are spread over the CUs, so a pass takes about
// as long as its fullest CU: ceil(blocks / CUs) deep or wide bricks; small ones
// are short enough that their number over the CUs describes them.  Times of a
// deep and a wide brick in hundredths of a small one's, each with a constant,
// from attempts of 28 shapes of 2.2e5 to 1e6 voxels (cubes to needles and
// slabs) in every form of the box passes and of the Gaussian.  Up to
// kPassDecisionMaxParts small bricks there is no other: the backward pass takes
// the decision on those.
struct BrickTimes {
  int deep, deep0, wide, wide0;
};
Brick fastest_brick(const Geom& g, const BrickTimes& t) {
  const long long small = bricks_of(g, kT3, kBrickZ), deep = bricks_of(g, kT3, kDeepZ),
                  wide = bricks_of(g, kWide, kBrickZ), cus = device_cus();
  if (small <= kPassDecisionMaxParts) return Brick::kSmall;
  const long long s = 100 * small, d = cus * (t.deep * ((deep + cus - 1) / cus) + t.deep0),
                  w = cus * (t.wide * ((wide + cus - 1) / cus) + t.wide0);
  return w <= s && w <= d ? Brick::kWide : d < s ? Brick::kDeep : Brick::kSmall;
}

// The Gaussian (attempt, window 7, box passes wide: 80x96x112, small 52.6 us,
// deep 51.4, wide 50.8; 300x5x400 56.7, 56.3, 57.3; 2000x20x20 76.9, 74.9,
// 77.2).
Brick gauss_brick(const Geom& g) { return fastest_brick(g, {125, 120, 200, 26}); }

template <class P, int R, bool DEC = false>
hipError_t run(const P& pol, const Geom& g, bool cubes, const DevState* st, int need,
               hipStream_t s, const PassDecision& pd = PassDecision{}) {
  if constexpr (DEC && R > kPassDecisionMaxRadius) {
    return hipErrorInvalidValue;  // wider windows keep the decision kernel
  } else {
    if (cubes) {
      const Brick form = P::kBox ? box_brick(g, R) : gauss_brick(g);
      const dim3 grid(brick_blocks(g, form));
      if (form == Brick::kSmall)
        hipLaunchKernelGGL((k_cube<R, P, kBrickZ, DEC>), grid, dim3(kCubeThreads), 0, s, pol, g,
                           st, need, pd);
      else if constexpr (DEC)
        return hipErrorInvalidValue;  // the others keep the decision kernel
      else if (form == Brick::kWide)
        hipLaunchKernelGGL((k_wide<R, P>), grid, dim3(kWideThreads), 0, s, pol, g, st, need, pd);
      else if constexpr (!P::kBox || R <= 2)
        hipLaunchKernelGGL((k_cube<R, P, kDeepZ, false>), grid, dim3(kCubeThreads), 0, s, pol, g,
                           st, need, pd);
      else
        return hipErrorInvalidValue;
      return hipGetLastError();
    }
    const Tiling t = march_tiling(g, R);
    const dim3 grid(t.tiles_x * march_rows(t) * t.nchunks);
    if (t.pairs)
      hipLaunchKernelGGL((k_stencil<R, kMarchTY, P, DEC>), grid, dim3(kTX * kMarchTY), 0, s, pol,
                         g, t, st, need, pd);
    else
      hipLaunchKernelGGL((k_stencil<R, kTY, P, DEC>), grid, dim3(kTX * kTY), 0, s, pol, g, t, st,
                         need, pd);
    return hipGetLastError();
  }
}

template <class P, bool DEC = false>
hipError_t run_box(const P& pol, int window, const Geom& g, bool cubes, const DevState* st,
                   int need, hipStream_t s, const PassDecision& pd = PassDecision{}) {
  switch (window / 2) {
    case 1: return run<P, 1, DEC>(pol, g, cubes, st, need, s, pd);
    case 2: return run<P, 2, DEC>(pol, g, cubes, st, need, s, pd);
    case 3: return run<P, 3, DEC>(pol, g, cubes, st, need, s, pd);
    case 4: return run<P, 4, DEC>(pol, g, cubes, st, need, s, pd);
    default: return hipErrorInvalidValue;
  }
}

template <typename T, typename Acc>
hipError_t fstat_t(const T* F, const Geom& g, const lmr_params& p, double* fstat,
                   hipStream_t s) {
  FStatPol<T, Acc> pol;
  pol.F = F;
  pol.fstat = fstat;
  pol.N = static_cast<int>(g.N);
  pol.inv_n = 1.0 / ((double)p.window * p.window * p.window);
  return run_box(pol, p.window, g, use_cubes(g, p), nullptr, 0, s);
}

template <typename T, typename Acc>
hipError_t fwd_t(const T* F, const float* Mw, const double* fstat, const Geom& g,
                 const lmr_params& p, const DevState* st, float* maps, double* partials,
                 int nparts, float* cc, hipStream_t s) {
  if (fwd_num_blocks(g, p) != nparts) return hipErrorInvalidValue;
  FwdPol<T, kTX * kTY, Acc> pol;
  pol.F = F;
  pol.Mw = Mw;
  pol.fstat = fstat;
  pol.maps = maps;
  pol.cc = cc;
  pol.partials = partials;
  pol.N = static_cast<int>(g.N);
  pol.inv_n = 1.0 / ((double)p.window * p.window * p.window);
  pol.eps = p.cc_eps;
  return run_box(pol, p.window, g, use_cubes(g, p), st, 1, s);
}

template <typename T, typename Acc>
hipError_t bwd_t(const T* F, const float* Mw, const float* maps, const Geom& g,
                 const lmr_params& p, const DevState* st, const float* dMw, float* graw,
                 hipStream_t s, const PassDecision* pd = nullptr) {
  BwdPol<T, Acc> pol;
  pol.F = F;
  pol.Mw = Mw;
  pol.maps = maps;
  pol.dMw = dMw;
  pol.graw = graw;
  pol.g = g;
  pol.inv_n = 1.0 / ((double)p.window * p.window * p.window);
  if (pd) return run_box<BwdPol<T, Acc>, true>(pol, p.window, g, use_cubes(g, p), st, 2, s, *pd);
  return run_box(pol, p.window, g, use_cubes(g, p), st, 2, s);
}

template <int R>
hipError_t smooth_r(const float* in, float* out, const Geom& g, const lmr_params& p,
                    const DevState* st, hipStream_t s, DevState* commit = nullptr) {
  SmoothPol<R> pol;
  pol.in = in;
  pol.out = out;
  pol.N = static_cast<int>(g.N);
  gauss_taps<R>(p.grad_sigma, pol.w);
  PassDecision pd{};
  pd.commit = commit;
  return run<SmoothPol<R>, R>(pol, g, use_cubes(g, p), st, 2, s, pd);
}

}  // namespace

bool batch_bricks(const Geom& g, const lmr_params& p) {
  return use_cubes(g, p) && g.N <= kBatchBrickMaxVoxels;
}

int brick_blocks(const Geom& g, Brick form) {
  return bricks_of(g, form == Brick::kWide ? kWide : kT3,
                   form == Brick::kDeep ? kDeepZ : kBrickZ);
}

// Attempts, Gaussian wide, small / deep / wide: window 3, 80x96x112 46.8, 45.4,
// 46.4 us, 2000x20x20 60.2, 57.6, 65.7, 80x49x57 24.4, 25.3, 26.7; window 5,
// 80x96x112 50.1, 48.7, 48.3, 65x89x77 37.2, 38.9, 36.2, 300x5x400 46.8, 46.7,
// 51.7; window 7, 80x96x112 55.5, 55.9, 50.8, 102x56x81 41.5, 42.1, 42.3,
// 300x5x400 51.6, 53.7, 57.3; window 9 as 7.  Deep ones are not built for radii
// above 2.
Brick box_brick(const Geom& g, int R) {
  constexpr BrickTimes kTimes[3] = {
      {143, 160, 283, 175}, {170, 65, 274, 89}, {1000, 0, 240, 63}};
  return fastest_brick(g, kTimes[std::min(R, 3) - 1]);
}

int fwd_num_blocks(const Geom& g, const lmr_params& p) {
  return use_cubes(g, p) ? brick_blocks(g, box_brick(g, p.window / 2))
                         : march_tiling(g, p.window / 2).tiles();
}

int gauss_radius(double sigma) {
  if (!(sigma > 0.0)) return 0;
  return (int)ceil(3.0 * sigma - 1e-12);
}

// The box sums accumulate in FP64 (LMR_ACC_F64) or in compensated FP32
// (LMR_ACC_F32C); the image type picks the loads.
hipError_t launch_fstat(const void* F, lmr_dtype t, const Geom& g, const lmr_params& p,
                        double* fstat, hipStream_t s) {
  if (t == LMR_BF16) {
    const uint16_t* f = static_cast<const uint16_t*>(F);
    return p.accum == LMR_ACC_F32C ? fstat_t<uint16_t, F32C>(f, g, p, fstat, s)
                                   : fstat_t<uint16_t, double>(f, g, p, fstat, s);
  }
  const float* f = static_cast<const float*>(F);
  return p.accum == LMR_ACC_F32C ? fstat_t<float, F32C>(f, g, p, fstat, s)
                                 : fstat_t<float, double>(f, g, p, fstat, s);
}

hipError_t launch_fwd(const void* F, lmr_dtype t, const float* Mw, const double* fstat,
                      const Geom& g, const lmr_params& p, const DevState* st, float* maps,
                      double* partials, int nparts, float* cc_map, hipStream_t s) {
  if (t == LMR_BF16) {
    const uint16_t* f = static_cast<const uint16_t*>(F);
    return p.accum == LMR_ACC_F32C
               ? fwd_t<uint16_t, F32C>(f, Mw, fstat, g, p, st, maps, partials, nparts, cc_map,
                                       s)
               : fwd_t<uint16_t, double>(f, Mw, fstat, g, p, st, maps, partials, nparts,
                                         cc_map, s);
  }
  const float* f = static_cast<const float*>(F);
  return p.accum == LMR_ACC_F32C
             ? fwd_t<float, F32C>(f, Mw, fstat, g, p, st, maps, partials, nparts, cc_map, s)
             : fwd_t<float, double>(f, Mw, fstat, g, p, st, maps, partials, nparts, cc_map,
                                    s);
}

hipError_t launch_bwd(const void* F, lmr_dtype t, const float* Mw, const float* maps,
                      const Geom& g, const lmr_params& p, const DevState* st,
                      const float* dMw, float* graw, hipStream_t s) {
  if (t == LMR_BF16) {
    const uint16_t* f = static_cast<const uint16_t*>(F);
    return p.accum == LMR_ACC_F32C
               ? bwd_t<uint16_t, F32C>(f, Mw, maps, g, p, st, dMw, graw, s)
               : bwd_t<uint16_t, double>(f, Mw, maps, g, p, st, dMw, graw, s);
  }
  const float* f = static_cast<const float*>(F);
  return p.accum == LMR_ACC_F32C ? bwd_t<float, F32C>(f, Mw, maps, g, p, st, dMw, graw, s)
                                 : bwd_t<float, double>(f, Mw, maps, g, p, st, dMw, graw, s);
}

hipError_t launch_smooth(const float* graw, const Geom& g, const lmr_params& p,
                         const DevState* st, float* out, hipStream_t s) {
  switch (gauss_radius(p.grad_sigma)) {
    case 0: return smooth_r<0>(graw, out, g, p, st, s);
    case 1: return smooth_r<1>(graw, out, g, p, st, s);
    case 2: return smooth_r<2>(graw, out, g, p, st, s);
    case 3: return smooth_r<3>(graw, out, g, p, st, s);
    case 4: return smooth_r<4>(graw, out, g, p, st, s);
    case 5: return smooth_r<5>(graw, out, g, p, st, s);
    case 6: return smooth_r<6>(graw, out, g, p, st, s);
    default: return hipErrorInvalidValue;
  }
}

bool bwd_takes_decision(const Geom& g, const lmr_params& p, int nparts) {
  return nparts <= kPassDecisionMaxParts && p.window / 2 <= kPassDecisionMaxRadius &&
         !(use_cubes(g, p) && box_brick(g, p.window / 2) != Brick::kSmall);
}

hipError_t launch_bwd_decide(const void* F, lmr_dtype t, const float* Mw, const float* maps,
                             const Geom& g, const lmr_params& p, const DevState* st,
                             const float* dMw, float* graw, const PassDecision& pd,
                             hipStream_t s) {
  if (!st || !pd.partials || !pd.next || !bwd_takes_decision(g, p, pd.nparts))
    return hipErrorInvalidValue;
  if (t == LMR_BF16) {
    const uint16_t* f = static_cast<const uint16_t*>(F);
    return p.accum == LMR_ACC_F32C
               ? bwd_t<uint16_t, F32C>(f, Mw, maps, g, p, st, dMw, graw, s, &pd)
               : bwd_t<uint16_t, double>(f, Mw, maps, g, p, st, dMw, graw, s, &pd);
  }
  const float* f = static_cast<const float*>(F);
  return p.accum == LMR_ACC_F32C
             ? bwd_t<float, F32C>(f, Mw, maps, g, p, st, dMw, graw, s, &pd)
             : bwd_t<float, double>(f, Mw, maps, g, p, st, dMw, graw, s, &pd);
}

hipError_t launch_smooth_commit(const float* graw, const Geom& g, const lmr_params& p,
                                const DevState* next, DevState* st, float* out,
                                hipStream_t s) {
  if (!next || !st) return hipErrorInvalidValue;
  switch (gauss_radius(p.grad_sigma)) {
    case 0: return smooth_r<0>(graw, out, g, p, next, s, st);
    case 1: return smooth_r<1>(graw, out, g, p, next, s, st);
    case 2: return smooth_r<2>(graw, out, g, p, next, s, st);
    case 3: return smooth_r<3>(graw, out, g, p, next, s, st);
    case 4: return smooth_r<4>(graw, out, g, p, next, s, st);
    case 5: return smooth_r<5>(graw, out, g, p, next, s, st);
    case 6: return smooth_r<6>(graw, out, g, p, next, s, st);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace lmr
