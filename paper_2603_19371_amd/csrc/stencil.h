// Separable 3D stencils of one LM attempt on a shared 2.5D framework, as
// device functions used by the per-pair kernels (k_stencil.hip) and by the
// batched persistent kernel (k_batch.hip).
//
//   FStatPol  window mean and variance of F, once per pair.
//   FwdPol    LNCC forward: box sums of Mw, Mw^2, F Mw over the w^3 window
//             (zero padding, divisor w^3), cc = s_FM^2/(s_FF s_MM + eps),
//             adjoint maps alpha = 2 s_FM/D, alpha mu_F, beta = -s_FM^2 s_FF/D^2,
//             beta mu_M, and one FP64 partial sum of cc per tile.
//   BwdPol    LNCC backward: box sums of the four maps give
//             d(sum cc)/dMw_j = (F_j B(alpha) - B(alpha mu_F) + 2 Mw_j B(beta)
//                                - 2 B(beta mu_M)) / w^3,
//             times the trilinear derivative of M at x + u(x) (warp backward);
//             the result is g = N dL/du with L = -mean cc.
//   SmoothPol Gaussian of the raw gradient (Eulerian descent, Sec. 2.1).
//
// A tile is a 32 x TY column of outputs over a chunk of z planes.  For each
// input plane the block stages a (TY+2R) x (32+2R) halo tile of the raw FP32
// inputs in LDS (the next plane is already in flight in registers while the
// current one is reduced), reduces along y (expanding the raw inputs into the
// accumulated channels: for the forward pass the exact products F^2, Mw^2,
// F Mw in FP64) and then along x, and keeps the last 2R+1 plane sums in a
// register ring.  Box sums run a running sum through the ring; the Gaussian
// sums it with its taps.
#pragma once

#include <type_traits>

#include "lmr_internal.h"

namespace lmr {

constexpr int kTX = 32;

// Compensated FP32 accumulator (the LMR_ACC_F32C box sums): an unevaluated
// sum hi + lo of two floats, accumulated by cascaded summation.  The high
// parts add with Knuth's TwoSum, whose exact rounding error joins the low
// parts, which add plainly; a product of two floats enters exactly through
// the FMA remainder.  No renormalisation between additions.  The y- and
// x-passes take 2R+1 additions each; the running z-sum of a tile takes two
// per plane of its march (the entering plane and the leaving one), i.e.
// 2 (cz + 2R) of them, about 200 on a 96-plane chunk.  Every TwoSum error is
// at most half an ulp of the running hi, so after k additions |lo| is at
// most about k/2 ulp(hi), and the plain additions of lo add an error of at
// most k^2/4 * 2^-24 ulp(hi): below 0.01 ulp(hi) for k = 200.  hi + lo
// therefore keeps about twice FP32's significand over a whole chunk.  With
// contraction off the sequences run as written.
struct F32C {
  float hi, lo;
  F32C() = default;  // trivial, so LDS arrays may hold it; F32C() value-initialises to 0
  __host__ __device__ explicit F32C(float v) : hi(v), lo(0.0f) {}
  __device__ static F32C product(float a, float b) {
    F32C r{};
    r.hi = a * b;
    r.lo = fmaf(a, b, -r.hi);
    return r;
  }
  __device__ friend F32C operator+(const F32C& a, const F32C& b) {
    F32C r{};
    r.hi = a.hi + b.hi;
    const float bb = r.hi - a.hi;
    const float e = (a.hi - (r.hi - bb)) + (b.hi - bb);
    r.lo = (a.lo + b.lo) + e;
    return r;
  }
  __device__ friend F32C operator-(const F32C& a, const F32C& b) {
    F32C nb{};
    nb.hi = -b.hi;
    nb.lo = -b.lo;
    return a + nb;
  }
  __device__ F32C& operator+=(const F32C& b) { return *this = *this + b; }
};
__device__ __forceinline__ double to_f64(double v) { return v; }
__device__ __forceinline__ double to_f64(const F32C& v) {
  return static_cast<double>(v.hi) + static_cast<double>(v.lo);
}

struct Tiling {
  int ty, tiles_x, tiles_y, nchunks, cz;
  int pairs;  // 1: a stand-alone context's blocks run two tiles (march_tiling)
  __host__ __device__ int tiles() const { return tiles_x * tiles_y * nchunks; }
};

constexpr int kMinTiles = 256;  // one tile per CU

// Floor on the chunk length: 8 planes while that still gives every CU a tile
// (the 2R halo planes stay a moderate share), else 4, else 2 when 4 would
// leave CUs without a tile (small pyramid levels: the march of a chunk is
// their latency).
__host__ __device__ inline int march_floor_cz(long long cols, int nz) {
  return cols * ((nz + 7) / 8) >= kMinTiles   ? 8
         : cols * ((nz + 3) / 4) >= kMinTiles ? 4
                                              : 2;
}

// z-chunk: long enough that the 2R halo planes of a chunk stay a small
// fraction when the volume is large, short enough that small volumes still
// give a few hundred tiles.  target_tiles and min_cz are tuning knobs.
__host__ __device__ inline Tiling make_tiling(int nz, int ny, int nx, int ty,
                                              int target_tiles = 2048, int min_cz = 16) {
  Tiling t;
  t.ty = ty;
  t.pairs = 0;
  t.tiles_x = (nx + kTX - 1) / kTX;
  t.tiles_y = (ny + ty - 1) / ty;
  const int cols = t.tiles_x * t.tiles_y;
  const int want = (target_tiles + cols - 1) / cols;
  int cz = (nz + want - 1) / want;
  if (cols * ((nz + min_cz - 1) / min_cz) >= target_tiles / 2 && cz < min_cz) cz = min_cz;
  const int floor_cz = march_floor_cz(cols, nz);
  if (cz < floor_cz) cz = floor_cz;
  if (cz > nz) cz = nz;
  t.cz = cz;
  t.nchunks = (nz + cz - 1) / cz;
  return t;
}

// Whether a pair of a batch runs on bricks: where a stand-alone context does,
// up to kBatchBrickMaxVoxels (larger pairs fill the GPU together and march as
// fast: 16 of 64x64x72 on bricks 303 us per attempt, marching 360; 4 of
// 96x96x96 198 and 180); the bricks of that context's box passes, and so of its
// partial sums of cc (k_stencil.hip); and the number of bricks of a volume.
constexpr long long kBatchBrickMaxVoxels = 1LL << 19;
bool batch_bricks(const Geom& g, const lmr_params& p);
enum class Brick : int { kSmall, kDeep, kWide };
Brick box_brick(const Geom& g, int R);
__host__ __device__ inline int bricks_of(const Geom& g, int side, int depth) {
  return ((g.nx + side - 1) / side) * ((g.ny + side - 1) / side) * ((g.nz + depth - 1) / depth);
}
int brick_blocks(const Geom& g, Brick form);

// The march's tiling of a volume for stencil radius R on the current device
// (k_stencil.hip): every pass of a per-pair attempt, and by default each pair
// of the batched form.
Tiling march_tiling(const Geom& g, int R);

// LDS of one stencil tile: the staged raw inputs and the y-pass sums.
template <int R, int TY, class P>
struct StencilLds {
  float in[P::NRAW][TY + 2 * R][kTX + 2 * R];
  typename P::Acc y[P::NCH][TY][kTX + 2 * R];
};

// The march of a tile (x0, y0, z0..z1) by a block of kTX x TY threads.  No
// vector memory operation of a step sits in a branch: a position outside the
// volume, a plane past the chunk and an output that does not exist use
// kFarIndex, which loads 0 and stores nothing.  The compiler then knows how
// many operations follow a load and waits for just that load; with branches it
// waits for everything in flight, stores included (160x192x224, window 7, BF16
// images: forward pass 96 -> 77 us; FP32 images: forward 81 -> 79, backward
// 108 -> 104).
template <int R, int TY, class P>
struct March {
  using A = typename P::Acc;
  static constexpr int NR = P::NRAW, NC = P::NCH, W = 2 * R + 1;
  static constexpr int LX = kTX + 2 * R, LY = TY + 2 * R, NT = kTX * TY;
  static constexpr int NPOS = LX * LY, PER = (NPOS + NT - 1) / NT;

  const P& pol;
  const Geom& g;
  const int z0, zend, plane, lx, ly, col;
  const bool own;
  int pidx[PER];  // positions of the halo tile this thread stages
  bool pin[PER];
  float pre[PER][NR];  // the plane in flight
  A ring[W][NC], run[NC];

  __device__ __forceinline__ March(const P& p, const Geom& geom, int x0, int y0, int z0_, int z1)
      : pol(p), g(geom), z0(z0_), zend(z1 + R), plane(geom.ny * geom.nx),
        lx(threadIdx.x % kTX), ly(threadIdx.x / kTX), col((y0 + ly) * geom.nx + x0 + lx),
        own(x0 + lx < geom.nx && y0 + ly < geom.ny) {
#pragma unroll
    for (int q = 0; q < PER; ++q) {
      const int i = threadIdx.x + q * NT;
      const int yy = i / LX, xx = i - yy * LX;
      const int gyy = y0 - R + yy, gxx = x0 - R + xx;
      pin[q] = i < NPOS && (unsigned)gyy < (unsigned)g.ny && (unsigned)gxx < (unsigned)g.nx;
      pidx[q] = pin[q] ? gyy * g.nx + gxx : 0;
    }
#pragma unroll
    for (int c = 0; c < NC; ++c) {
      run[c] = A();
#pragma unroll
      for (int k = 0; k < W; ++k) ring[k][c] = A();
    }
  }
  __device__ __forceinline__ void fetch(const typename P::Local& loc, int zi) {
    const bool zin = (unsigned)zi < (unsigned)g.nz && zi < zend;
    const unsigned zoff = zin ? static_cast<unsigned>(zi * plane) : 0u;
#pragma unroll
    for (int q = 0; q < PER; ++q)
      pol.load(loc, (zin && pin[q]) ? zoff + static_cast<unsigned>(pidx[q]) : kFarIndex,
               pre[q]);
  }
  __device__ __forceinline__ void commit(StencilLds<R, TY, P>& sm) const {
#pragma unroll
    for (int q = 0; q < PER; ++q) {
      const int i = threadIdx.x + q * NT;
      if (i < NPOS) {
        const int yy = i / LX, xx = i - yy * LX;
#pragma unroll
        for (int c = 0; c < NR; ++c) sm.in[c][yy][xx] = pre[q][c];
      }
    }
  }
  // kFarIndex where the plane zo holds no output of this thread
  __device__ __forceinline__ unsigned out_index(int zo) const {
    return zo >= z0 && own ? static_cast<unsigned>(zo * plane + col) : kFarIndex;
  }
  __device__ __forceinline__ void operands(unsigned io, typename P::Pre& q) const {
    pol.pre(io != kFarIndex ? io : 0u, q);
  }
  // fence > 0: at most that many taps of the window in flight (see below)
  template <int FENCE>
  __device__ __forceinline__ void ypass(StencilLds<R, TY, P>& sm) const {
    for (int i = threadIdx.x; i < TY * LX; i += NT) {
      const int yy = i / LX, xx = i - yy * LX;
      A a[NC];
#pragma unroll
      for (int c = 0; c < NC; ++c) a[c] = A();
#pragma unroll
      for (int k = 0; k < W; ++k) {
        float r[NR];
#pragma unroll
        for (int c = 0; c < NR; ++c) r[c] = sm.in[c][yy + k][xx];
        pol.accum(a, r, k);
        if constexpr (FENCE > 0)
          if (k % FENCE == FENCE - 1) __builtin_amdgcn_sched_barrier(0);
      }
#pragma unroll
      for (int c = 0; c < NC; ++c) sm.y[c][yy][xx] = a[c];
    }
  }
  // the window sums of the plane whose y pass is in sm; S: its ring slot
  template <int S, int FENCE>
  __device__ __forceinline__ void xpass(const StencilLds<R, TY, P>& sm, A (&o)[NC]) {
    A pl[NC];
#pragma unroll
    for (int c = 0; c < NC; ++c) pl[c] = A();
#pragma unroll
    for (int k = 0; k < W; ++k) {
#pragma unroll
      for (int c = 0; c < NC; ++c) {
        if constexpr (P::kBox)
          pl[c] += sm.y[c][ly][lx + k];
        else
          pl[c] = fma(A(pol.wt(k)), sm.y[c][ly][lx + k], pl[c]);
      }
      if constexpr (FENCE > 0)
        if (k % FENCE == FENCE - 1) __builtin_amdgcn_sched_barrier(0);
    }
    if constexpr (P::kBox) {
      // ring[S] holds the plane that entered W steps ago
#pragma unroll
      for (int c = 0; c < NC; ++c) {
        run[c] += pl[c] - ring[S][c];
        ring[S][c] = pl[c];
        o[c] = run[c];
      }
    } else {
#pragma unroll
      for (int c = 0; c < NC; ++c) {
        ring[S][c] = pl[c];
        o[c] = A(0);
      }
      // planes zi-2R .. zi sit in slots S+1 .. S+W (mod W)
#pragma unroll
      for (int k = 0; k < W; ++k)
#pragma unroll
        for (int c = 0; c < NC; ++c)
          o[c] = fma(A(pol.wt(k)), ring[(S + 1 + k) % W][c], o[c]);
    }
  }
};

// One step of stencil_tile: plane zi, in ring slot S.
template <int S, bool FENCE, int R, int TY, class P>
__device__ __forceinline__ void tile_step(March<R, TY, P>& m, int zi, typename P::Local& loc,
                                          StencilLds<R, TY, P>& sm) {
  // with FP64 sums the operands of this step's output are requested before the
  // next plane, so that they arrive during the y pass (read at their use, a
  // block waits a memory round trip per plane; forward pass at 160x192x224,
  // w 7: 90.5 -> 85.5 us).  The compensated sums have no registers to hold
  // them (121x145x119, w 9: 346 -> 351 us).
  constexpr bool kEarly = !std::is_same<typename P::Acc, F32C>::value;
  // and their windows from radius 3 on are fenced (stencil_march), which keeps
  // the backward pass at 117 registers and four waves per SIMD (left alone 164
  // and three; attempt at 160x72x160, window 7: 100.3 -> 94.9 us); compensated
  // sums are a percent faster without.  (FENCE: not in the persistent kernel
  // that also runs bricks: 166 registers for 213 let a third of its blocks onto
  // a CU, and its grid barriers wait for all of them: 32^3, 60 -> 75 us.)
  constexpr bool kFenced = FENCE && P::kBox && kEarly && R >= 3;
  m.commit(sm);
  const unsigned io = m.out_index(zi - R);
  typename P::Pre q;
  if (kEarly) m.operands(io, q);
  m.fetch(loc, zi + 1);
  __syncthreads();
  m.template ypass<kFenced ? 4 : 0>(sm);
  __syncthreads();
  typename P::Acc o[P::NCH];
  m.template xpass<S, kFenced ? 1 : 0>(sm, o);
  if (!kEarly) m.operands(io, q);
  m.pol.emit(loc, io, q, o);
}

// Calls f(slot) for the slots 0 .. W-1 in turn, until it returns true.
template <int S, int W, class F>
__device__ __forceinline__ bool each_slot(F&& f) {
  if constexpr (S < W) {
    if (f(std::integral_constant<int, S>{})) return true;
    return each_slot<S + 1, W>(f);
  } else {
    return false;
  }
}

// The stencil over a tile, two barriers per plane, in the LDS `sm`: where a
// stand-alone context's blocks run one tile (march_tiling), and in the batch.
// (The persistent kernel's phases overlay their LDS; those of one launch per
// phase have their own and could run stencil_march.)
template <int R, int TY, bool FENCE = true, class P>
__device__ __forceinline__ void stencil_tile(const P& pol, const Geom& g, int x0, int y0,
                                             int z0, int z1, typename P::Local& loc,
                                             StencilLds<R, TY, P>& sm) {
  March<R, TY, P> m(pol, g, x0, y0, z0, z1);
  int zi = z0 - R;
  m.fetch(loc, zi);
  while (!each_slot<0, 2 * R + 1>([&](auto s) {
    tile_step<decltype(s)::value, FENCE>(m, zi, loc, sm);
    return ++zi == m.zend;
  })) {
  }
}

// The stencil over a tile with one barrier per plane, on two copies of the
// LDS: after the barrier of plane zi a block runs the y pass of that plane,
// stages the next one into the other copy and runs the x pass of plane zi - 1
// from there, so the LDS reads of one overlap the sums of the other.  With
// 32 x 16 tiles two blocks share a CU and a plane's halo rows are read 22 times
// for 16 rows of outputs, not 14 for 8 (what bounds the passes is how fast
// halo lines come from the caches: loads and stores alone take 90 of the
// backward pass's 104 us on 32 x 8 tiles, 81 on 32 x 16).  kFence keeps the
// compiler from requesting all taps of a window at once, whose registers it
// would spill: 160x192x224, window 7, FP64 sums, forward 73 us either way,
// backward 102 -> 89 (window 9: 190 -> 127).  The smoothing pass has the
// registers (57 us; 61 with fences).  Against the two-barrier form on 32 x 8
// tiles: forward 79 -> 72 us, backward 104 -> 89, smoothing 62 -> 57; with
// compensated FP32 sums and window 9 forward 223 -> 147, backward 256 -> 190.
template <int R, int TY, class P>
__device__ __forceinline__ void stencil_march(const P& pol, const Geom& g, int x0, int y0,
                                              int z0, int z1, typename P::Local& loc,
                                              StencilLds<R, TY, P> (&sm)[2]) {
  constexpr int kFenceY = P::kBox ? 4 : 0, kFenceX = P::kBox ? 1 : 0;
  March<R, TY, P> m(pol, g, x0, y0, z0, z1);
  int zi = z0 - R, b = 1;
  m.fetch(loc, zi);
  m.commit(sm[0]);
  m.fetch(loc, zi + 1);
  __syncthreads();
  m.template ypass<kFenceY>(sm[0]);
  m.commit(sm[1]);
  m.fetch(loc, zi + 2);
  while (!each_slot<0, 2 * R + 1>([&](auto s) {
    __syncthreads();
    const unsigned io = m.out_index(zi - R);
    typename P::Pre q;
    m.operands(io, q);
    m.template ypass<kFenceY>(sm[b]);  // plane zi + 1
    m.commit(sm[b ^ 1]);               // plane zi + 2: sm[b ^ 1].in was read a step ago
    m.fetch(loc, zi + 3);
    typename P::Acc o[P::NCH];
    m.template xpass<decltype(s)::value, kFenceX>(sm[b ^ 1], o);
    pol.emit(loc, io, q, o);
    b ^= 1;
    return ++zi == m.zend;
  })) {
  }
}

// ------------------------------------------------------------- 3D tiles
// Small volumes (coarse pyramid levels) have too few 32 x TY columns to fill
// the GPU, and the plane-serial march of a short chunk is their latency.
// There a block owns a brick of kBrickZ planes instead: each thread reads one
// (y, x) column of the halo straight from memory (all its loads in flight at
// once, in wide bricks the operands of its outputs with them) and reduces
// along z; then the block reduces along y and along x in LDS and emits.  Three
// steps instead of a march.
//
// Three sizes (fastest_brick in k_stencil.hip).  Small bricks, kT3 x kT3
// columns, where few blocks are the limit (40x48x56: 420 of them); deep bricks,
// the same columns of kDeepZ planes; and wide bricks, kWide x kWide columns, for
// larger volumes: what bounds a pass there is the cache lines its halo rows
// touch (loads and stores alone take 14 of the forward pass's 18 us on 8 x 8
// x 8 bricks at 80x96x112, whose 14-voxel rows use 56 bytes of one or two
// 128-byte lines), and a 22-voxel row serves twice the outputs (15 us; the
// backward pass 23 -> 19, the Gaussian 13.6 -> 11).
//
// Every output is the sum of its terms in ascending y, then x, of z sums: those
// of its column in ascending z or, for compensated sums from radius 2 on,
// running sums that start where kBrickZ divides z.  So it does not depend on
// the brick that computes it.
constexpr int kT3 = 8, kWide = 16, kBrickZ = 4, kDeepZ = 8;
constexpr int kCubeThreads = 256, kWideThreads = 512;

// The z sums of the halo columns of a brick of SIDE x SIDE columns.  The y
// pass reads them, keeps its own (fewer) results in registers and, after a
// barrier, writes them over the z sums, so one array serves both passes and
// more blocks fit on a CU.
template <int R, class P, int SIDE, int DEPTH = kBrickZ>
struct BrickLds {
  using A = typename P::Acc;
  static constexpr int L = SIDE + 2 * R;
  A z[P::NCH][DEPTH][L][L];
  __device__ __forceinline__ A (&y())[P::NCH][DEPTH][SIDE][L] {
    return *reinterpret_cast<A(*)[P::NCH][DEPTH][SIDE][L]>(&z[0][0][0][0]);
  }
};

// KO consecutive outputs of one channel along an axis from the KO + 2R values
// they share, each summed in order.
template <int R, int KO, class P>
__device__ __forceinline__ void window_outputs(const P& pol,
                                               const typename P::Acc (&v)[KO + 2 * R],
                                               typename P::Acc (&o)[KO]) {
  using A = typename P::Acc;
#pragma unroll
  for (int j = 0; j < KO; ++j) {
    o[j] = A();
#pragma unroll
    for (int k = 0; k <= 2 * R; ++k) {
      if constexpr (P::kBox)
        o[j] += v[j + k];
      else
        o[j] = fma(A(pol.wt(k)), v[j + k], o[j]);
    }
  }
}

// Halo column `col` of the brick at (x0, y0, z0).
template <int R, int SIDE, int DEPTH = kBrickZ, class P>
__device__ __forceinline__ void brick_column(const P& pol, const Geom& g, int x0, int y0,
                                             int z0, const typename P::Local& loc, int col,
                                             float (&r)[DEPTH + 2 * R][P::NRAW]) {
  constexpr int L = SIDE + 2 * R;
  const int yy = col / L, xx = col - yy * L;
  const int gy = y0 - R + yy, gx = x0 - R + xx;
  const bool in = (unsigned)gy < (unsigned)g.ny && (unsigned)gx < (unsigned)g.nx;
#pragma unroll
  for (int k = 0; k < DEPTH + 2 * R; ++k) {
    const int gz = z0 - R + k;
    const unsigned i = (in && (unsigned)gz < (unsigned)g.nz)
                           ? static_cast<unsigned>((gz * g.ny + gy) * g.nx + gx)
                           : kFarIndex;
    pol.load(loc, i, r[k]);
  }
}

// Its z sums into LDS, the raw inputs expanded into the accumulated channels.
template <int R, int SIDE, int DEPTH = kBrickZ, class P>
__device__ __forceinline__ void brick_zsum(const P& pol, const Geom& g, int x0, int y0, int z0,
                                           const typename P::Local& loc,
                                           const float (&r)[DEPTH + 2 * R][P::NRAW], int col,
                                           BrickLds<R, P, SIDE, DEPTH>& sm) {
  using A = typename P::Acc;
  constexpr int NC = P::NCH, L = SIDE + 2 * R;
  const int yy = col / L, xx = col - yy * L;
  auto write = [&](int oz, const A (&a)[NC]) {
#pragma unroll
    for (int c = 0; c < NC; ++c) sm.z[c][oz][yy][xx] = a[c];
  };
  auto sum = [&](int oz, A (&a)[NC]) {
#pragma unroll
    for (int c = 0; c < NC; ++c) a[c] = A();
#pragma unroll
    for (int k = 0; k <= 2 * R; ++k) pol.accum(a, r[oz + k], k);
  };
  A a[NC];
#pragma unroll
  for (int z = 0; z < DEPTH; z += kBrickZ) {
    sum(z, a);
    write(z, a);
    if constexpr (std::is_same<A, F32C>::value && R >= 2) {
      // the entering position's terms added, the leaving one's (formed again)
      // subtracted: an addition of compensated sums is eight operations, and
      // from radius 2 on this takes fewer of them than every sum by itself (19
      // instead of 28 a channel at radius 3: attempts 3 to 6 % faster; radius
      // 2, 1 to 3 %; with FP64 sums nothing)
#pragma unroll
      for (int oz = z + 1; oz < z + kBrickZ; ++oz) {
        A enter[NC], leave[NC];
#pragma unroll
        for (int c = 0; c < NC; ++c) enter[c] = leave[c] = A();
        pol.accum(enter, r[oz + 2 * R], 0);
        pol.accum(leave, r[oz - 1], 0);
#pragma unroll
        for (int c = 0; c < NC; ++c) a[c] += enter[c] - leave[c];
        write(oz, a);
      }
      // a term that is not finite does not leave a sum again: there every sum by
      // itself, its terms loaded again (kept in r they take 20 registers and a
      // third of a CU's wide bricks: attempts of 24 batches 2 % slower, 16 of
      // 64x64x60 287 us, 300; loaded again, no slower)
      bool lost = false;
#pragma unroll
      for (int c = 0; c < NC; ++c) lost |= a[c].lo != a[c].lo;
      if (lost) {
#pragma unroll 1
        for (int oz = z + 1; oz < z + kBrickZ; ++oz) {
#pragma unroll
          for (int c = 0; c < NC; ++c) a[c] = A();
#pragma unroll 1
          for (int k = oz; k <= oz + 2 * R; ++k) {
            const int gx = x0 - R + xx, gy = y0 - R + yy, gz = z0 - R + k;
            float v[P::NRAW];
            if ((unsigned)gx < (unsigned)g.nx && (unsigned)gy < (unsigned)g.ny &&
                (unsigned)gz < (unsigned)g.nz) {
              pol.load(loc, (gz * g.ny + gy) * g.nx + gx, v);
              pol.accum(a, v, 0);
            }
          }
          write(oz, a);
        }
      }
    } else {
#pragma unroll
      for (int oz = z + 1; oz < z + kBrickZ; ++oz) {
        sum(oz, a);
        write(oz, a);
      }
    }
  }
}

// The y pass of a brick by NT threads, KY outputs per item.
template <int R, int SIDE, int NT, int KY, int DEPTH, class P>
__device__ __forceinline__ void brick_ypass(const P& pol, BrickLds<R, P, SIDE, DEPTH>& sm) {
  using A = typename P::Acc;
  constexpr int NC = P::NCH, L = SIDE + 2 * R, NY = DEPTH * (SIDE / KY) * L,
                PY = (NY + NT - 1) / NT;
  A ay[PY][NC][KY];
#pragma unroll
  for (int j = 0; j < PY; ++j) {
    const int it = threadIdx.x + j * NT;
    if (NY % NT == 0 || it < NY) {
      const int xx = it % L, row = it / L;
      const int oy = (row % (SIDE / KY)) * KY, oz = row / (SIDE / KY);
#pragma unroll
      for (int c = 0; c < NC; ++c) {
        A v[KY + 2 * R];
#pragma unroll
        for (int k = 0; k < KY + 2 * R; ++k) v[k] = sm.z[c][oz][oy + k][xx];
        window_outputs<R, KY>(pol, v, ay[j][c]);
      }
    }
  }
  __syncthreads();
  auto& sy = sm.y();
#pragma unroll
  for (int j = 0; j < PY; ++j) {
    const int it = threadIdx.x + j * NT;
    if (NY % NT == 0 || it < NY) {
      const int xx = it % L, row = it / L;
      const int oy = (row % (SIDE / KY)) * KY, oz = row / (SIDE / KY);
#pragma unroll
      for (int c = 0; c < NC; ++c)
#pragma unroll
        for (int k = 0; k < KY; ++k) sy[c][oz][oy + k][xx] = ay[j][c][k];
    }
  }
}

// A small or deep brick by kCubeThreads threads, an output per kBrickZ planes
// each.  Summing policies: loc.sum receives that of the first kBrickZ planes,
// the return value is that of a deep brick's others.
template <int R, int DEPTH, class P>
__device__ __forceinline__ double stencil_cube(const P& pol, const Geom& g, int x0, int y0,
                                             int z0, typename P::Local& loc,
                                             BrickLds<R, P, kT3, DEPTH>& sm) {
  using A = typename P::Acc;
  constexpr int NC = P::NCH, L = kT3 + 2 * R, NT = kCubeThreads;
  static_assert(kBrickZ * kT3 * kT3 == NT, "one output per thread and kBrickZ planes");
  for (int col = threadIdx.x; col < L * L; col += NT) {
    float r[DEPTH + 2 * R][P::NRAW];
    brick_column<R, kT3, DEPTH>(pol, g, x0, y0, z0, loc, col, r);
    brick_zsum<R, kT3, DEPTH>(pol, g, x0, y0, z0, loc, r, col, sm);
  }
  __syncthreads();
  brick_ypass<R, kT3, NT, 1>(pol, sm);
  __syncthreads();
  auto& sy = sm.y();
  const int oy = (threadIdx.x / kT3) % kT3, ox = threadIdx.x % kT3;
  const int gx = x0 + ox, gy = y0 + oy;
  double first = 0.0, others = 0.0;
#pragma unroll
  for (int j = 0; j < DEPTH; j += kBrickZ) {
    const int oz = threadIdx.x / (kT3 * kT3) + j, gz = z0 + oz;
    A a[NC];
#pragma unroll
    for (int c = 0; c < NC; ++c) {
      A v[1 + 2 * R], o[1];
#pragma unroll
      for (int k = 0; k <= 2 * R; ++k) v[k] = sy[c][oz][oy][ox + k];
      window_outputs<R, 1>(pol, v, o);
      a[c] = o[0];
    }
    if (gx < g.nx && gy < g.ny && gz < g.nz) {
      const int i = (gz * g.ny + gy) * g.nx + gx;
      typename P::Pre q;
      pol.pre(i, q);
      pol.emit(loc, i, q, a);
    }
    if constexpr (P::kSum && DEPTH > kBrickZ) {
      (j == 0 ? first : others) = loc.sum;
      loc.sum = j == 0 ? 0.0 : first;
    }
  }
  return others;
}

// ---- wide bricks: kWideThreads threads, two outputs adjacent in x each
template <int R, class P>
struct WideFetch {
  float r[kBrickZ + 2 * R][P::NRAW];  // the thread's halo column
  typename P::Pre q[2];               // the operands of its outputs
  int i;                              // its first output
  bool ok0, ok1;                      // which of them exist
};

template <int R, class P>
__device__ __forceinline__ void wide_fetch(const P& pol, const Geom& g, int x0, int y0, int z0,
                                           const typename P::Local& loc, WideFetch<R, P>& f) {
  constexpr int L = kWide + 2 * R;
  static_assert(kBrickZ * kWide * kWide == 2 * kWideThreads, "two outputs per thread");
  if (L * L >= kWideThreads || threadIdx.x < L * L)
    brick_column<R, kWide>(pol, g, x0, y0, z0, loc, threadIdx.x, f.r);
  const int gx = x0 + (threadIdx.x % 8) * 2, gy = y0 + (threadIdx.x / 8) % 16,
            gz = z0 + threadIdx.x / 128;
  f.ok0 = gx < g.nx && gy < g.ny && gz < g.nz;
  f.ok1 = f.ok0 && gx + 1 < g.nx;
  f.i = (gz * g.ny + gy) * g.nx + gx;
  if (f.ok0) pol.pre(f.i, f.q[0]);
  if (f.ok1) pol.pre(f.i + 1, f.q[1]);
}

// The passes over a fetched brick.  cc (summing policies): what each of the
// thread's outputs added to loc.sum.
template <int R, class P>
__device__ __forceinline__ void wide_passes(const P& pol, const Geom& g, int x0, int y0, int z0,
                                            typename P::Local& loc, WideFetch<R, P>& f,
                                            BrickLds<R, P, kWide>& sm, double (&cc)[2]) {
  using A = typename P::Acc;
  constexpr int NC = P::NCH, L = kWide + 2 * R, NT = kWideThreads;
  if (L * L >= NT || threadIdx.x < L * L)
    brick_zsum<R, kWide>(pol, g, x0, y0, z0, loc, f.r, threadIdx.x, sm);
  for (int col = threadIdx.x + NT; col < L * L; col += NT) {  // R > 3
    float r[kBrickZ + 2 * R][P::NRAW];
    brick_column<R, kWide>(pol, g, x0, y0, z0, loc, col, r);
    brick_zsum<R, kWide>(pol, g, x0, y0, z0, loc, r, col, sm);
  }
  __syncthreads();
  brick_ypass<R, kWide, NT, 4>(pol, sm);
  __syncthreads();
  auto& sy = sm.y();
  cc[0] = cc[1] = 0.0;
  if (!f.ok0) return;
  const int ox = (threadIdx.x % 8) * 2, oy = (threadIdx.x / 8) % 16, oz = threadIdx.x / 128;
  A a[2][NC];
#pragma unroll
  for (int c = 0; c < NC; ++c) {
    A v[2 + 2 * R], o[2];
#pragma unroll
    for (int k = 0; k < 2 + 2 * R; ++k) v[k] = sy[c][oz][oy][ox + k];
    window_outputs<R, 2>(pol, v, o);
    a[0][c] = o[0];
    a[1][c] = o[1];
  }
#pragma unroll
  for (int j = 0; j < 2; ++j) {
    if (j == 1 && !f.ok1) break;
    pol.emit(loc, f.i + j, f.q[j], a[j]);
    if constexpr (P::kSum) {
      cc[j] = loc.sum;
      loc.sum = 0.0;
    }
  }
}

// The partial sums of a wide brick.  Its 2 x 2 small bricks are summed in the
// order of block_sum_to over a small brick's block (there lane 8 oy + ox of
// wave oz; here the outputs 2 j and 2 j + 1 of a row share a lane, so the last
// step of the tree is inside it).  sub: one partial per small brick, at its
// number in the volume, else their sum to partials[slot].
__device__ __forceinline__ void wide_partials(const double (&cc)[2], const Geom& g, int x0,
                                              int y0, int z0, bool sub, int slot,
                                              double* partials) {
  __shared__ double red[kBrickZ][2][2];  // plane, half along y, half along x
  __shared__ double quad[4];
  double e = cc[0], o = cc[1];
#pragma unroll
  for (int off : {32, 16, 8, 2, 1}) {
    e += __shfl_xor(e, off, 64);
    o += __shfl_xor(o, off, 64);
  }
  const int lane = threadIdx.x & 63;
  if ((lane & ~4) == 0) red[threadIdx.x / 128][(threadIdx.x / 64) % 2][lane / 4] = e + o;
  __syncthreads();
  if (threadIdx.x < 4) {
    const int px = threadIdx.x & 1, py = threadIdx.x >> 1;
    double s = 0.0;
#pragma unroll
    for (int k = 0; k < kBrickZ; ++k) s += red[k][py][px];
    if (sub) {
      const int cx = (g.nx + kT3 - 1) / kT3, cy = (g.ny + kT3 - 1) / kT3;
      const int bx = x0 / kT3 + px, by = y0 / kT3 + py;
      if (bx < cx && by < cy) partials[((z0 / kBrickZ) * cy + by) * cx + bx] = s;
    } else {
      quad[threadIdx.x] = s;
    }
  }
  if (sub) return;
  __syncthreads();
  if (threadIdx.x == 0) partials[slot] = ((quad[0] + quad[1]) + quad[2]) + quad[3];
}

// A wide brick from fetch to partials.
template <int R, class P>
__device__ __forceinline__ void stencil_wide(const P& pol, const Geom& g, int x0, int y0, int z0,
                                             typename P::Local& loc, WideFetch<R, P>& f,
                                             BrickLds<R, P, kWide>& sm, bool sub, int slot) {
  double cc[2];
  wide_passes<R>(pol, g, x0, y0, z0, loc, f, sm, cc);
  if constexpr (P::kSum) wide_partials(cc, g, x0, y0, z0, sub, slot, pol.partials);
}

// Origin of brick b of a volume (x fastest, then y, then z).
template <int SIDE, int DEPTH = kBrickZ>
__device__ __forceinline__ void brick_origin(const Geom& g, int b, int& x0, int& y0, int& z0) {
  const int cx = (g.nx + SIDE - 1) / SIDE, cy = (g.ny + SIDE - 1) / SIDE;
  x0 = (b % cx) * SIDE;
  y0 = ((b / cx) % cy) * SIDE;
  z0 = (b / (cx * cy)) * DEPTH;
}

// Block sum of one double per thread; thread 0 writes it to *out.
template <int NT>
__device__ __forceinline__ void block_sum_to(double v, double* out) {
  __shared__ double red[NT / 64];
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  if (lane == 0) red[wv] = v;
  __syncthreads();
  if (threadIdx.x == 0) {
    double s = 0.0;
#pragma unroll
    for (int k = 0; k < NT / 64; ++k) s += red[k];
    *out = s;
  }
  __syncthreads();
}

// ------------------------------------------------- statistics of F (once)
// The window mean and variance of the fixed image do not change between
// attempts: they are box-summed once per pair (at begin) and stored in FP64
// as mu_F and sigma_FF, from sums of the exact products F^2.
template <typename T, typename AccT = double>
struct FStatPol {
  using Acc = AccT;
  static constexpr int NRAW = 1, NCH = 2;
  static constexpr bool kBox = true, kSum = false;
  const T* __restrict__ F;
  double* __restrict__ fstat;  // [2][N]: mu_F, sigma_FF
  int N;
  double inv_n;
  struct Local {
    RBuf bF;
  };
  struct Pre {};

  __device__ static constexpr double wt(int) { return 1.0; }
  __device__ Local begin_block(const DevState*) const { return Local{make_rbuf_n(F, N)}; }
  __device__ void load(const Local& l, unsigned i, float v[1]) const { v[0] = bld<T>(l.bF, i); }
  __device__ void accum(Acc a[2], const float r[1], int) const {
    if constexpr (std::is_same<Acc, F32C>::value) {
      a[0] += F32C(r[0]);
      a[1] += F32C::product(r[0], r[0]);
    } else {
      const double f = r[0];
      a[0] += f;
      a[1] = fma(f, f, a[1]);
    }
  }
  __device__ void pre(unsigned, Pre&) const {}
  __device__ void emit(Local&, unsigned i, const Pre&, const Acc S[2]) const {
    if (i == kFarIndex) return;
    const double muF = to_f64(S[0]) * inv_n;
    fstat[i] = muF;
    fstat[N + i] = to_f64(S[1]) * inv_n - muF * muF;
  }
  __device__ void end_tile(Local&, int) const {}
};

// ------------------------------------------------------------- forward (P2)
// Box sums of Mw, Mw^2 and F Mw (exact products in FP64); mu_F and sigma_FF
// come from FStatPol's pass over the same F.
template <typename T, int NT, typename AccT = double>
struct FwdPol {
  using Acc = AccT;
  static constexpr int NRAW = 2, NCH = 3;
  static constexpr bool kBox = true, kSum = true;
  const T* __restrict__ F;
  const float* __restrict__ Mw;
  const double* __restrict__ fstat;
  float* __restrict__ maps;
  float* __restrict__ cc;
  double* __restrict__ partials;
  int N;
  double inv_n, eps;
  struct Local {
    double sum;
    RBuf bF, bM, out[4];
  };
  struct Pre {
    double muF, sff;
  };

  __device__ static constexpr double wt(int) { return 1.0; }
  __device__ Local begin_block(const DevState*) const {
    Local l{0.0, make_rbuf_n(F, N), make_rbuf_n(Mw, N), {}};
#pragma unroll
    for (int c = 0; c < 4; ++c) l.out[c] = make_rbuf_n(maps + (size_t)c * N, N);
    return l;
  }
  __device__ void load(const Local& l, unsigned i, float v[2]) const {
    v[0] = bld<T>(l.bF, i);
    v[1] = bld<float>(l.bM, i);
  }
  __device__ void accum(Acc a[3], const float r[2], int) const {
    if constexpr (std::is_same<Acc, F32C>::value) {
      a[0] += F32C(r[1]);
      a[1] += F32C::product(r[1], r[1]);
      a[2] += F32C::product(r[0], r[1]);
    } else {
      const double f = r[0], m = r[1];
      a[0] += m;
      a[1] = fma(m, m, a[1]);
      a[2] = fma(f, m, a[2]);
    }
  }
  __device__ void pre(unsigned i, Pre& q) const {
    q.muF = fstat[i];
    q.sff = fstat[N + i];
  }
  __device__ void emit(Local& loc, unsigned i, const Pre& q, const Acc S[3]) const {
    const double muF = q.muF, sff = q.sff;
    const double muM = to_f64(S[0]) * inv_n;
    const double sfm = to_f64(S[2]) * inv_n - muF * muM;
    const double smm = to_f64(S[1]) * inv_n - muM * muM;
    const double iD = 1.0 / (sff * smm + eps);
    const double c = sfm * sfm * iD;
    const double alpha = 2.0 * sfm * iD;
    const double beta = -c * sff * iD;
    bst(loc.out[0], i, static_cast<float>(alpha));
    bst(loc.out[1], i, static_cast<float>(alpha * muF));
    bst(loc.out[2], i, static_cast<float>(beta));
    bst(loc.out[3], i, static_cast<float>(beta * muM));
    if (cc && i != kFarIndex) cc[i] = static_cast<float>(c);
    loc.sum += i != kFarIndex ? c : 0.0;
  }
  // partial sum of cc of the tile just processed, to partials[slot]
  __device__ void end_tile(Local& loc, int slot) const {
    block_sum_to<NT>(loc.sum, partials + slot);
    loc.sum = 0.0;
  }
};

// ------------------------------------------------------------ backward (P4)
template <typename T, typename AccT = double>
struct BwdPol {
  using Acc = AccT;
  static constexpr int NRAW = 4, NCH = 4;
  static constexpr bool kBox = true, kSum = false;
  const T* __restrict__ F;
  const float* __restrict__ Mw;
  const float* __restrict__ maps;
  // derivative of M at x + u(x), stored by the kernel that warped M (P1 or
  // k_warp): gathered here it costs the pass a dependent read of the field
  // and eight corner loads (160x192x224 traced: gathered 152 us; stored 117 us
  // and 14 us more in the warp).  May alias graw (read, then overwritten, by the
  // thread of the same voxel).
  const float* dMw;
  float* graw;
  Geom g;
  double inv_n;
  struct Local {
    RBuf bmap[4], out[3];
  };
  struct Pre {
    float f, m, d[3];
  };

  __device__ static constexpr double wt(int) { return 1.0; }
  __device__ Local begin_block(const DevState*) const {
    const long long N = g.N;
    Local l;
#pragma unroll
    for (int c = 0; c < 4; ++c) l.bmap[c] = make_rbuf_n(maps + c * N, N);
#pragma unroll
    for (int c = 0; c < 3; ++c) l.out[c] = make_rbuf_n(graw + c * N, N);
    return l;
  }
  __device__ void load(const Local& l, unsigned i, float v[4]) const {
#pragma unroll
    for (int c = 0; c < 4; ++c) v[c] = bld<float>(l.bmap[c], i);
  }
  __device__ void accum(Acc a[4], const float r[4], int) const {
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      if constexpr (std::is_same<Acc, F32C>::value)
        a[c] += F32C(r[c]);
      else
        a[c] += static_cast<double>(r[c]);
    }
  }
  __device__ void pre(unsigned i, Pre& q) const {
    const long long N = g.N;
    q.f = ldf(F, i);
    q.m = Mw[i];
#pragma unroll
    for (int c = 0; c < 3; ++c) q.d[c] = (dMw + c * N)[i];
  }
  __device__ void emit(const Local& l, unsigned i, const Pre& q, const Acc Bs[4]) const {
    const double fj = q.f, mj = q.m;
    const double B[4] = {to_f64(Bs[0]), to_f64(Bs[1]), to_f64(Bs[2]), to_f64(Bs[3])};
    const double dS = (fj * B[0] - B[1] + 2.0 * mj * B[2] - 2.0 * B[3]) * inv_n;
    const float d = static_cast<float>(dS);
#pragma unroll
    for (int c = 0; c < 3; ++c) bst(l.out[c], i, -d * q.d[c]);
  }
  __device__ void end_tile(Local&, int) const {}
};

// ----------------------------------------------------------- smoothing (P5)
template <int R>
struct SmoothPol {
  using Acc = float;
  static constexpr int NRAW = 3, NCH = 3;
  static constexpr bool kBox = false, kSum = false;
  const float* __restrict__ in;
  float* __restrict__ out;
  int N;
  float w[2 * R + 1];
  struct Local {
    RBuf b[3], out[3];
  };
  struct Pre {};

  __device__ float wt(int k) const { return w[k]; }
  __device__ Local begin_block(const DevState*) const {
    Local l;
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      l.b[c] = make_rbuf_n(in + (size_t)c * N, N);
      l.out[c] = make_rbuf_n(out + (size_t)c * N, N);
    }
    return l;
  }
  __device__ void load(const Local& l, unsigned i, float v[3]) const {
#pragma unroll
    for (int c = 0; c < 3; ++c) v[c] = bld<float>(l.b[c], i);
  }
  __device__ void accum(float a[3], const float r[3], int k) const {
#pragma unroll
    for (int c = 0; c < 3; ++c) a[c] = fmaf(w[k], r[c], a[c]);
  }
  __device__ void pre(unsigned, Pre&) const {}
  __device__ void emit(Local& l, unsigned i, const Pre&, const float S[3]) const {
#pragma unroll
    for (int c = 0; c < 3; ++c) bst(l.out[c], i, S[c]);
  }
  __device__ void end_tile(Local&, int) const {}
};

// Normalised Gaussian taps k in [-R, R] (host side).
template <int R>
inline void gauss_taps(double sigma, float* w) {
  double t[2 * R + 1], tot = 0.0;
  for (int k = -R; k <= R; ++k) {
    t[k + R] = R == 0 ? 1.0 : exp(-(double)k * k / (2.0 * sigma * sigma));
    tot += t[k + R];
  }
  for (int k = 0; k <= 2 * R; ++k) w[k] = static_cast<float>(t[k] / tot);
}

// Decode a tile index (x fastest, then y, then z chunk).
__device__ __forceinline__ void tile_origin(const Tiling& t, int b, int ty, int& x0,
                                            int& y0, int& z0) {
  const int tx_i = b % t.tiles_x;
  const int ty_i = (b / t.tiles_x) % t.tiles_y;
  const int ch = b / (t.tiles_x * t.tiles_y);
  x0 = tx_i * kTX;
  y0 = ty_i * ty;
  z0 = ch * t.cz;
}

}  // namespace lmr
