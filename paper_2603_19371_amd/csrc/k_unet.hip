// Kernels of the learned initializer's 3D U-Net: dense 3x3x3 convolutions
// on the MFMA matrix cores (BF16 operands, FP32 accumulation) and the
// memory-bound pieces around them (pooling, upsampling, ReLU gradient, MSE,
// Adam, weight packing).
//
// Layouts.  Activations are channels-last BF16: element (v, c) of a tensor
// with channel stride ld sits at v*ld + c, so a channel concatenation is two
// tensors sharing one buffer at different channel offsets.  Weights are FP32
// masters [27][cin][cout] (tap t = 9 (dz+1) + 3 (dy+1) + (dx+1) reads the
// input at v + (dx, dy, dz)), packed per step into BF16
//   Wf  forward
//   Wb  transposed, tap order reversed (gradient with respect to the input =
//       convolution of dZ with the flipped, transposed kernel)
// with cin_p, cout_p the channel counts rounded up to 16, zero padded.  A pack
// is a sequence of MFMA weight operands, [output tile][input chunk][27 taps]
// of 16 x 16 channels: lane l holds input channels 4 (l / 16) .. + 3 of
// output channel l % 16 in elements 4 l .. 4 l + 3, so an operand is one
// contiguous 512-byte read.
//
// MFMA operand layout (16x16 output tile, K = 4 g or 8 g per lane group
// g = lane / 16): lane l feeds row l % 16 of A and column l % 16 of B with
// the same K slots, and receives D[4 g + j][l % 16], j = 0..3.  Which K a
// slot maps to is irrelevant as long as A and B agree.
#include <hip/hip_runtime.h>

#include <type_traits>

#include "lmr_internal.h"
#include "unet_internal.h"

namespace lmr {

namespace {

typedef short s4 __attribute__((ext_vector_type(4)));
typedef __bf16 b8 __attribute__((ext_vector_type(8)));
typedef float f4 __attribute__((ext_vector_type(4)));
typedef float f2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf2 __attribute__((ext_vector_type(2)));

// FP32 -> BF16, round to nearest even (NaN stays NaN).
__device__ __forceinline__ uint16_t f2bf(float v) {
  uint32_t b = __float_as_uint(v);
  if ((b & 0x7F800000u) == 0x7F800000u)
    return static_cast<uint16_t>((b >> 16) | ((b & 0xFFFFu) ? 0x40u : 0u));
  b += 0x7FFFu + ((b >> 16) & 1u);
  return static_cast<uint16_t>(b >> 16);
}
__device__ __forceinline__ float bf2f(uint16_t h) {
  return __uint_as_float(static_cast<uint32_t>(h) << 16);
}
// Eight BF16 operand slots from two groups of four (bit patterns).
__device__ __forceinline__ b8 cat_bf16(s4 lo, s4 hi) {
  typedef short s8 __attribute__((ext_vector_type(8)));
  const s8 v = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
  return __builtin_bit_cast(b8, v);
}

// K = 16 per instruction: 4 BF16 per lane.
struct K16 {
  static constexpr int KW = 16;
  typedef s4 vec;
  __device__ static vec zero() { return vec{0, 0, 0, 0}; }
  __device__ static vec load(const uint16_t* p) { return *reinterpret_cast<const s4*>(p); }
  __device__ static vec load_w(const uint16_t* p) { return load(p); }
  __device__ static f4 mma(vec a, vec b, f4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(a, b, c, 0, 0, 0);
  }
};
// K = 32 per instruction (gfx950): 8 BF16 per lane.
struct K32 {
  static constexpr int KW = 32;
  typedef b8 vec;
  __device__ static vec zero() {
    vec z;
#pragma unroll
    for (int j = 0; j < 8; ++j) z[j] = static_cast<__bf16>(0.0f);
    return z;
  }
  __device__ static vec load(const uint16_t* p) { return *reinterpret_cast<const b8*>(p); }
  // two consecutive quads of a packed operand (16 lanes apart)
  __device__ static vec load_w(const uint16_t* p) {
    return cat_bf16(*reinterpret_cast<const s4*>(p), *reinterpret_cast<const s4*>(p + 64));
  }
  __device__ static f4 mma(vec a, vec b, f4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
  }
};

// ----------------------------------------------------------- convolution
// A block covers 64 consecutive output voxels along x (4 waves x 16) and 16
// output channels; K runs over the 27 taps and the input channels.
// A[m][k] = X[voxel x0 + m shifted by tap][channel], B[k][n] = W[tap][n][k].
template <class MM>
__global__ void __launch_bounds__(256) k_conv(ConvArgs a) {
  constexpr int KL = MM::KW / 4;  // K slots per lane
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  const int x0 = blockIdx.x * 64 + wv * 16;
  if (x0 >= a.nx) return;
  const int nco = a.cout_p / 16;
  const int y = blockIdx.y;
  const int z = blockIdx.z / nco, co0 = (blockIdx.z % nco) * 16;
  const int m = lane & 15, kq = lane >> 4;
  const int xa = x0 + m;
  f4 acc = {0.f, 0.f, 0.f, 0.f};
  for (int t = 0; t < 27; ++t) {
    const int dz = t / 9 - 1, dy = (t / 3) % 3 - 1, dx = t % 3 - 1;
    const int zz = z + dz, yy = y + dy, xx = xa + dx;
    const bool in = (unsigned)zz < (unsigned)a.nz && (unsigned)yy < (unsigned)a.ny &&
                    (unsigned)xx < (unsigned)a.nx;
    const uint16_t* xp =
        a.X + (in ? ((long long)(zz * a.ny + yy) * a.nx + xx) * a.ldx : 0);
    const uint16_t* wt = a.W + ((long long)(co0 / 16) * (a.cin_p / 16) * 27 + t) * 256;
    for (int c0 = 0; c0 < a.cin_p; c0 += MM::KW) {
      const int ci = c0 + KL * kq;
      typename MM::vec av = MM::zero();
      if (in && ci < a.cin_valid) av = MM::load(xp + ci);
      // quad ci / 4 of the input chunk ci / 16
      const uint16_t* wq = wt + (ci / 16) * 27 * 256 + (((ci % 16) / 4) * 16 + m) * 4;
      acc = MM::mma(av, MM::load_w(wq), acc);
    }
  }
  const int co = co0 + m;
  if (co >= a.cout) return;
  const float b = a.bias ? a.bias[co] : 0.0f;
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const int xo = x0 + 4 * kq + j;
    if (xo >= a.nx) continue;
    const long long v = (long long)(z * a.ny + y) * a.nx + xo;
    float r = acc[j] + b;
    if (a.relu) r = fmaxf(r, 0.0f);
    if (a.mask && !(bf2f(a.mask[v * a.ldm + co]) > 0.0f)) r = 0.0f;
    if (a.Y) a.Y[v * a.ldy + co] = f2bf(r);
    if (a.yf) a.yf[v * a.ldf + co] = r;
  }
}

// The same convolution with the operands staged in LDS.  A block of four
// waves owns 16 x TY (x, y) output voxels of WZ z planes, RW rows of one plane
// per wave, and 16 NT output channels.  Per chunk of 16 input channels it
// stages the (WZ + 2) x (TY + 2) x 18 input halo and the chunk's weight
// operands, then each wave runs the MFMAs of its rows for all 27 taps from
// LDS.  Every load of a chunk is issued before the first is used and the next
// chunk's loads are in flight during the current chunk's MFMAs.  Input
// positions outside the volume, and channels past cin_valid, read 0 through
// the buffer resource (an offset beyond the tensor).
//
// What bounds it is staging and LDS, not the MFMA rate.  A tile of 4 planes x
// 4 rows stages 648 halo voxels for 256 outputs where one plane of 16 rows
// takes 972.  An operand read is 512 bytes per wave for one 16-cycle MFMA, so
// a wave holds the (RW + 2) x 3 input operands of a tap plane in registers: a
// halo row serves the y taps of up to three output rows, 18 reads where 36
// would be made at RW = 4.  Forward pass at 80x96x112 per layer: 16 -> 16
// channels at full resolution 39 -> 26 us, 48 -> 16 88 -> 55, 96 -> 32 at half
// 41 -> 31, 192 -> 64 at a quarter 45 -> 25, 128 -> 128 at an eighth 29 -> 17
// us.  Each output is the same sequence of products for every tile shape:
// chunks, tap planes and tap pairs in order.
//
// The MFMA computes D[co][voxel] = sum_ci W[co][ci] X[voxel][ci] (weights as
// the A operand), so that each lane receives four consecutive output channels
// of one voxel: the epilogue stores them as one 8-byte (BF16) or 16-byte
// (FP32) write, zeroing those whose ReLU was inactive (a.mask).
//
// LDS input rows (one voxel: 16 channels) are 40 bytes apart.  An operand
// read takes the same 8-byte quad of 16 consecutive rows; with a 32-byte
// pitch those fall on 4 bank groups (a 4-way conflict), with 40 bytes (10
// dwords) 10 m mod 32 covers all 16 even banks.  The pitch keeps every LDS
// address affine in the tap.  Weight operands are stored as packed, read
// lane after lane.
//
// V16: the input is staged in 16-byte items (channel stride, offset and
// count multiples of 8); otherwise in 8-byte quads, those past cin_valid
// written as zeros without a read (the 2-channel input: 36 -> 23 us).
// MFMAs keep the order in which they are written; anything else may move.  A
// 16x16x16 and a 16x16x32 product in a row on one accumulator, either way
// round, need five wait states that the compiler does not insert: the second
// reads the accumulator as it was before the first (measured with integer
// operands: half of all sums wrong with up to four wait states, none with
// five or with any other MFMA in between).
__device__ __forceinline__ void keep_product_order() {
  __builtin_amdgcn_sched_barrier(0x7F6);  // all kinds but MFMA
}

constexpr int kCT = 16;            // tile edge along x
constexpr int kCH = kCT + 2;       // halo tile edge
constexpr int kPitch = 20;         // LDS row pitch, uint16 elements (40 bytes)
template <int NT, int RW, int WZ, bool V16>
__global__ void __launch_bounds__(256) k_conv_tile(ConvArgs a) {
  static_assert(NT * RW >= 2, "another accumulator's product between dependent ones");
  constexpr int TY = RW * (4 / WZ);                        // rows of the tile
  constexpr int HY = TY + 2, P = (WZ + 2) * HY * kCH;      // halo rows, positions
  // staged items per thread: 16-byte halves of a voxel's 16 channels, or whole
  // voxels in 8-byte quads
  constexpr int XI = V16 ? 2 * P : P, XPER = (XI + 255) / 256, QPER = V16 ? 1 : 4;
  constexpr int WC = 27 * 32;  // 16-byte items of one chunk's weight operands
  constexpr int WI = NT * WC, WPER = (WI + 255) / 256;
  __shared__ __attribute__((aligned(16))) uint16_t s_x[P * kPitch];
  __shared__ __attribute__((aligned(16))) uint16_t s_w[NT * 27 * 256];
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  const int nco = a.cout_p / (16 * NT), nch = a.cin_p / 16;
  // tile id: channel tile fastest, then x, y, z; each XCD takes a contiguous
  // range of ids, so the blocks that read an input plane (those of output
  // planes z-1, z, z+1, and every channel tile) mostly share one L2
  const int tiles_x = (a.nx + kCT - 1) / kCT, tiles_y = (a.ny + TY - 1) / TY;
  int b = xcd_remap(blockIdx.x, gridDim.x);
  const int co0 = (b % nco) * 16 * NT;
  b /= nco;
  const int x0 = (b % tiles_x) * kCT;
  b /= tiles_x;
  const int y0 = (b % tiles_y) * TY, z0 = (b / tiles_y) * WZ;
  const int wz = wv % WZ, wy = (wv / WZ) * RW;  // the wave's plane and first row
  const int m = lane & 15, kq = lane >> 4;
  // ---- input staging: element offset of each item of this thread (channel
  // group 0; -1: outside the volume) and its channel within the group
  const long long nvox = (long long)a.nz * a.ny * a.nx;
  const RBuf bx = make_rbuf(
      a.X, static_cast<unsigned>(((nvox - 1) * a.ldx + ((a.cin_valid + 3) & ~3)) * 2));
  auto item = [&](int j, int& pos, int& ch) {
    const int it = tid + 256 * j;
    pos = V16 ? it >> 1 : it;
    ch = V16 ? 8 * (it & 1) : 0;
    return it < XI;
  };
  int xoff[XPER];
#pragma unroll
  for (int j = 0; j < XPER; ++j) {
    int pos, ch;
    const bool ok = item(j, pos, ch);
    const int gz = z0 + pos / (HY * kCH) - 1, gy = y0 + (pos / kCH) % HY - 1,
              gx = x0 + pos % kCH - 1;
    const bool in = ok && (unsigned)gz < (unsigned)a.nz && (unsigned)gy < (unsigned)a.ny &&
                    (unsigned)gx < (unsigned)a.nx;
    xoff[j] = in ? ((gz * a.ny + gy) * a.nx + gx) * a.ldx + ch : -1;
  }
  const RBuf bw = make_rbuf(a.W, static_cast<unsigned>(27LL * a.cout_p * a.cin_p * 2));
  using Item = std::conditional_t<V16, uint4, uint2>;
  Item rx[XPER][QPER];
  uint4 rw[WPER];
  auto fetch = [&](int chunk) {
    const int c0 = 16 * chunk;
#pragma unroll
    for (int j = 0; j < XPER; ++j) {
      if constexpr (V16) {
        int pos, ch;
        item(j, pos, ch);
        const unsigned o = xoff[j] >= 0 && c0 + ch < a.cin_valid
                               ? static_cast<unsigned>(xoff[j] + c0) * 2u
                               : kFarOffset;
        const auto v = __builtin_amdgcn_raw_buffer_load_b128(bx.r, o, 0, 0);
        rx[j][0] = uint4{static_cast<unsigned>(v[0]), static_cast<unsigned>(v[1]),
                         static_cast<unsigned>(v[2]), static_cast<unsigned>(v[3])};
      } else {
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          rx[j][q] = uint2{0, 0};
          if (c0 + 4 * q < a.cin_valid) {
            const unsigned o =
                xoff[j] >= 0 ? static_cast<unsigned>(xoff[j] + c0 + 4 * q) * 2u : kFarOffset;
            const auto v = __builtin_amdgcn_raw_buffer_load_b64(bx.r, o, 0, 0);
            rx[j][q] = uint2{static_cast<unsigned>(v[0]), static_cast<unsigned>(v[1])};
          }
        }
      }
    }
#pragma unroll
    for (int j = 0; j < WPER; ++j) {
      const int it = tid + 256 * j;
      const int n = it / WC, r = it % WC;
      const unsigned o =
          it < WI ? static_cast<unsigned>((((co0 >> 4) + n) * nch + chunk) * WC + r) * 16u
                  : kFarOffset;
      const auto v = __builtin_amdgcn_raw_buffer_load_b128(bw.r, o, 0, 0);
      rw[j] = uint4{static_cast<unsigned>(v[0]), static_cast<unsigned>(v[1]),
                    static_cast<unsigned>(v[2]), static_cast<unsigned>(v[3])};
    }
  };
  auto commit = [&]() {
#pragma unroll
    for (int j = 0; j < XPER; ++j) {
      int pos, ch;
      if (!item(j, pos, ch)) continue;
      uint16_t* d = s_x + pos * kPitch + ch;
      if constexpr (V16) {
        *reinterpret_cast<uint2*>(d) = uint2{rx[j][0].x, rx[j][0].y};
        *reinterpret_cast<uint2*>(d + 4) = uint2{rx[j][0].z, rx[j][0].w};
      } else {
#pragma unroll
        for (int q = 0; q < 4; ++q) *reinterpret_cast<uint2*>(d + 4 * q) = rx[j][q];
      }
    }
#pragma unroll
    for (int j = 0; j < WPER; ++j) {
      const int it = tid + 256 * j;
      if (it < WI) *reinterpret_cast<uint4*>(&s_w[it * 8]) = rw[j];
    }
  };
  f4 acc[NT][RW];
#pragma unroll
  for (int n = 0; n < NT; ++n)
#pragma unroll
    for (int r = 0; r < RW; ++r) acc[n][r] = f4{0.f, 0.f, 0.f, 0.f};
  fetch(0);
  for (int chunk = 0; chunk < nch; ++chunk) {
    __syncthreads();  // the previous chunk's operands are no longer read
    commit();
    __syncthreads();
    if (chunk + 1 < nch) fetch(chunk + 1);  // in flight during this chunk's MFMAs
#pragma unroll
    for (int dz = 0; dz < 3; ++dz) {
      // halo voxel m of rows wy .. wy + RW + 1 of plane wz + dz
      const uint16_t* xp = s_x + (((wz + dz) * HY + wy) * kCH + m) * kPitch + 4 * kq;
      const uint16_t* wp = s_w + dz * 9 * 256 + lane * 4;
      s4 X[RW + 2][3], w[NT][9];
#pragma unroll
      for (int n = 0; n < NT; ++n)
#pragma unroll
        for (int t = 0; t < 9; ++t)
          w[n][t] = *reinterpret_cast<const s4*>(wp + (n * 27 + t) * 256);
#pragma unroll
      for (int r = 0; r < RW + 2; ++r)
#pragma unroll
        for (int dx = 0; dx < 3; ++dx)
          X[r][dx] = *reinterpret_cast<const s4*>(xp + (r * kCH + dx) * kPitch);
      // taps 2p and 2p + 1 as one K = 32 product (each lane's eight K slots:
      // its four channels of the first tap, then the same four of the
      // second, in both operands); the ninth tap as a K = 16 product
#pragma unroll
      for (int tp = 0; tp < 4; ++tp) {
        const int ta = 2 * tp, tb = ta + 1;
        b8 wt[NT];
#pragma unroll
        for (int n = 0; n < NT; ++n) wt[n] = cat_bf16(w[n][ta], w[n][tb]);
#pragma unroll
        for (int r = 0; r < RW; ++r) {
          const b8 xv = cat_bf16(X[r + ta / 3][ta % 3], X[r + tb / 3][tb % 3]);
#pragma unroll
          for (int n = 0; n < NT; ++n) {
            acc[n][r] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wt[n], xv, acc[n][r], 0, 0, 0);
            keep_product_order();
          }
        }
      }
#pragma unroll
      for (int r = 0; r < RW; ++r)
#pragma unroll
        for (int n = 0; n < NT; ++n) {
          acc[n][r] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(w[n][8], X[r + 2][2],
                                                                acc[n][r], 0, 0, 0);
          keep_product_order();
        }
    }
  }
  // D[4 kq + j][m]: output channel co0 + 16 n + 4 kq + j of voxel x0 + m in
  // row y0 + wy + r of plane z0 + wz
  const int x = x0 + m, z = z0 + wz;
  if (x >= a.nx || z >= a.nz) return;
  const bool vec = a.cout % 4 == 0 && a.ldy % 4 == 0 && a.ldf % 4 == 0 && a.ldm % 4 == 0 &&
                   (reinterpret_cast<uintptr_t>(a.Y) % 8) == 0 &&
                   (reinterpret_cast<uintptr_t>(a.mask) % 8) == 0 &&
                   (reinterpret_cast<uintptr_t>(a.yf) % 16) == 0;
  // voxel of row r: v0 + r nx (v0: this lane's voxel in row y0 + wy)
  const long long v0 = (long long)(z * a.ny + y0 + wy) * a.nx + x;
  uint16_t* const yrow = a.Y ? a.Y + v0 * a.ldy : nullptr;
  float* const frow = a.yf ? a.yf + v0 * a.ldf : nullptr;
  const uint16_t* const mrow = a.mask ? a.mask + v0 * a.ldm : nullptr;
  const long long ystep = (long long)a.nx * a.ldy, fstep = (long long)a.nx * a.ldf,
                  mstep = (long long)a.nx * a.ldm;
#pragma unroll
  for (int n = 0; n < NT; ++n) {
    const int cb = co0 + 16 * n + 4 * kq;
    if (cb >= a.cout) continue;
    float bias[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) bias[j] = (a.bias && cb + j < a.cout) ? a.bias[cb + j] : 0.0f;
#pragma unroll
    for (int r = 0; r < RW; ++r) {
      if (y0 + wy + r >= a.ny) continue;
      float o[4];
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        o[j] = acc[n][r][j] + bias[j];
        if (a.relu) o[j] = fmaxf(o[j], 0.0f);
      }
      if (vec) {
        if (mrow) {
          const uint2 q = *reinterpret_cast<const uint2*>(mrow + r * mstep + cb);
          if (!(bf2f(static_cast<uint16_t>(q.x)) > 0.0f)) o[0] = 0.0f;
          if (!(bf2f(static_cast<uint16_t>(q.x >> 16)) > 0.0f)) o[1] = 0.0f;
          if (!(bf2f(static_cast<uint16_t>(q.y)) > 0.0f)) o[2] = 0.0f;
          if (!(bf2f(static_cast<uint16_t>(q.y >> 16)) > 0.0f)) o[3] = 0.0f;
        }
        if (yrow) {
          const bf2 lo = __builtin_convertvector(f2{o[0], o[1]}, bf2);
          const bf2 hi = __builtin_convertvector(f2{o[2], o[3]}, bf2);
          *reinterpret_cast<uint2*>(yrow + r * ystep + cb) =
              uint2{__builtin_bit_cast(unsigned, lo), __builtin_bit_cast(unsigned, hi)};
        }
        if (frow) *reinterpret_cast<f4*>(frow + r * fstep + cb) = f4{o[0], o[1], o[2], o[3]};
      } else {
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          if (cb + j >= a.cout) continue;
          if (mrow && !(bf2f(mrow[r * mstep + cb + j]) > 0.0f)) o[j] = 0.0f;
          if (yrow) yrow[r * ystep + cb + j] = f2bf(o[j]);
          if (frow) frow[r * fstep + cb + j] = o[j];
        }
      }
    }
  }
}

// Weight gradient, partial over a brick of 16 x 16 (x, y) voxels and a range
// of z planes.  A block of four waves takes one brick, one tile of 16 input
// channels and one tile of 16 output channels; it marches through its planes
// with the input planes z-1, z, z+1 (halo 18 x 18) and the output-gradient
// plane z staged in LDS as they lie in memory, 16 channels per voxel:
//   A[ci][k] = X[voxel k shifted by tap][ci],  B[k][co] = dZ[voxel k][co]
// with K running over 16 voxels of a row (lane group g takes voxels 4g..4g+3).
// An operand is four voxels of one channel per lane, a transpose of what LDS
// holds: gfx950's transposing read (ds_read_b64_tr_b16) gives it, where a
// transposed copy in LDS takes 36 two-byte writes per thread and plane.  Wave
// w owns rows 4w..4w+3 of the brick and keeps the 27 tap tiles in registers;
// the 6 x 3 operands of a tap plane serve its four rows.  The next planes'
// loads are in flight during the MFMAs of the current one, the first three
// planes are requested together, and 168 registers leave room for a third
// block per compute unit: the block's time is the latency of its planes.  At
// the end the four waves' tiles are added in LDS in wave order (a fixed
// order; lane after lane, since the tile's own layout is a 4-way bank
// conflict) and the block writes one partial; blocks of input tile 0 also sum
// dZ for the bias gradient.  With the reduction, 80x96x112: 16 -> 16 channels
// 52 -> 37 us, 48 -> 16 105 -> 80, all 15 layers 701 -> 520 us.
//
// XV, DV: X and dZ are staged in 16-byte items (channel stride, offset and
// count multiples of 8), else in 8-byte quads.
constexpr int kWgPos = kCH * kCH;     // halo voxels of a plane
constexpr int kWgSlot = kWgPos * 16;  // elements per staged input plane
struct WgradArgs {
  const uint16_t* X;
  int ldx, cin, cin_p;
  const uint16_t* dZ;
  int ldz, cout, cout_p;
  int nz, ny, nx;
  int zper, nzp;  // planes per block, z parts
  float* part;
  float* partb;
};

// Staging of NPOS voxels x 16 channels by a block of 256 threads: 16-byte
// halves of a voxel (V16) or its 8-byte quads.
template <int NPOS, bool V16>
struct WgStage {
  static constexpr int ITEMS = V16 ? 2 * NPOS : NPOS, PER = (ITEMS + 255) / 256;
  static constexpr int QN = V16 ? 1 : 4;
  using Item = std::conditional_t<V16, uint4, uint2>;
  int off[PER];  // element offset within a plane (-1: outside)
  Item v[PER][QN];
  // item j of this thread: voxel and first channel
  __device__ static bool item(int j, int& pos, int& ch) {
    const int it = threadIdx.x + 256 * j;
    pos = V16 ? it >> 1 : it;
    ch = V16 ? 8 * (it & 1) : 0;
    return it < ITEMS;
  }
  // plane_off: element offset of the plane and channel tile; nc: channels of
  // the tile that exist
  __device__ void fetch(const RBuf& b, long long plane_off, bool zok, int nc) {
#pragma unroll
    for (int j = 0; j < PER; ++j) {
      int pos, ch;
      item(j, pos, ch);
      const bool ok = zok && off[j] >= 0;
      const unsigned o = static_cast<unsigned>((plane_off + off[j]) * 2);
      if constexpr (V16) {
        const auto q =
            __builtin_amdgcn_raw_buffer_load_b128(b.r, ok && ch < nc ? o : kFarOffset, 0, 0);
        v[j][0] = uint4{static_cast<unsigned>(q[0]), static_cast<unsigned>(q[1]),
                        static_cast<unsigned>(q[2]), static_cast<unsigned>(q[3])};
      } else {
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          v[j][k] = uint2{0, 0};
          if (4 * k < nc) {
            const auto q =
                __builtin_amdgcn_raw_buffer_load_b64(b.r, ok ? o + 8 * k : kFarOffset, 0, 0);
            v[j][k] = uint2{static_cast<unsigned>(q[0]), static_cast<unsigned>(q[1])};
          }
        }
      }
    }
  }
  __device__ void commit(uint16_t* d) const {
#pragma unroll
    for (int j = 0; j < PER; ++j) {
      int pos, ch;
      if (!item(j, pos, ch)) continue;
#pragma unroll
      for (int k = 0; k < QN; ++k)
        *reinterpret_cast<Item*>(d + pos * 16 + ch + 4 * k) = v[j][k];
    }
  }
};

// Operand of 16 consecutive voxels from LDS voxel p (16 channels each): lane l
// receives voxels 4 (l / 16) .. + 3 of channel l % 16.
__device__ __forceinline__ s4 read_tr(const uint16_t* p) {
  const int l = threadIdx.x & 63;
  uint16_t* q = const_cast<uint16_t*>(p) + (4 * (l >> 4) + ((l & 15) >> 2)) * 16 + (l & 3) * 4;
  return __builtin_amdgcn_ds_read_tr16_b64_v4i16(
      (__attribute__((address_space(3))) s4*)q);
}

template <bool XV, bool DV>
__global__ void __launch_bounds__(256, XV && DV ? 3 : 2) k_wgrad(WgradArgs a) {
  __shared__ __attribute__((aligned(16))) uint16_t s_x[3 * kWgSlot];  // [slot][hy][hx][ci]
  __shared__ __attribute__((aligned(16))) uint16_t s_d[16 * 16 * 16];  // [y][x][co]
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  const int m = lane & 15, kq = lane >> 4;
  const int nci = a.cin_p / 16, nco = a.cout_p / 16;
  const int nbx = (a.nx + 15) / 16, nby = (a.ny + 15) / 16;
  int b = blockIdx.x;
  const int cb = b % nco;
  b /= nco;
  const int ib = b % nci;
  b /= nci;
  const int chunk = b;  // (z part, brick y, brick x), brick x fastest
  const int bx = b % nbx;
  b /= nbx;
  const int by = b % nby;
  const int zp = b / nby;
  const int x0 = bx * 16, y0 = by * 16;
  const int zb = zp * a.zper, ze = min(a.nz, zb + a.zper);
  const long long nvox = (long long)a.nz * a.ny * a.nx;
  const RBuf rx = make_rbuf(
      a.X, static_cast<unsigned>(((nvox - 1) * a.ldx + ((a.cin + 3) & ~3)) * 2));
  const RBuf rd = make_rbuf(
      a.dZ, static_cast<unsigned>(((nvox - 1) * a.ldz + ((a.cout + 3) & ~3)) * 2));
  WgStage<kWgPos, XV> px;
  WgStage<256, DV> pd;
#pragma unroll
  for (int j = 0; j < px.PER; ++j) {
    int pos, ch;
    const bool ok = px.item(j, pos, ch);
    const int gy = y0 - 1 + pos / kCH, gx = x0 - 1 + pos % kCH;
    px.off[j] = ok && (unsigned)gy < (unsigned)a.ny && (unsigned)gx < (unsigned)a.nx
                    ? (gy * a.nx + gx) * a.ldx + ch
                    : -1;
  }
#pragma unroll
  for (int j = 0; j < pd.PER; ++j) {
    int pos, ch;
    pd.item(j, pos, ch);
    const int gy = y0 + pos / 16, gx = x0 + pos % 16;
    pd.off[j] = gy < a.ny && gx < a.nx ? (gy * a.nx + gx) * a.ldz + ch : -1;
  }
  const long long plane_x = (long long)a.ny * a.nx * a.ldx,
                  plane_d = (long long)a.ny * a.nx * a.ldz;
  auto fetch_x = [&](WgStage<kWgPos, XV>& st, int gz) {
    const bool zok = (unsigned)gz < (unsigned)a.nz;
    st.fetch(rx, (zok ? gz : 0) * plane_x + ib * 16, zok, a.cin - ib * 16);
  };
  auto fetch_d = [&](int gz) { pd.fetch(rd, gz * plane_d + cb * 16, true, a.cout - cb * 16); };
  f4 acc[27];
#pragma unroll
  for (int t = 0; t < 27; ++t) acc[t] = f4{0.f, 0.f, 0.f, 0.f};
  float bs = 0.0f;
  // planes zb - 1 and zb (requested together with the first step's), then
  // the march
  {
    WgStage<kWgPos, XV> p0 = px, p1 = px;
    fetch_x(p0, zb - 1);
    fetch_x(p1, zb);
    fetch_x(px, zb + 1);
    fetch_d(zb);
    p0.commit(s_x + ((zb + 2) % 3) * kWgSlot);
    p1.commit(s_x + (zb % 3) * kWgSlot);
  }
  for (int z = zb; z < ze; ++z) {
    __syncthreads();  // the plane z - 2 slot and the dZ plane are no longer read
    px.commit(s_x + ((z + 1) % 3) * kWgSlot);
    pd.commit(s_d);
    __syncthreads();
    if (z + 1 < ze) {
      fetch_x(px, z + 2);
      fetch_d(z + 1);
    }
    s4 dv[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) dv[r] = read_tr(s_d + (4 * wv + r) * 256);
    if (ib == 0) {
#pragma unroll
      for (int r = 0; r < 4; ++r)
#pragma unroll
        for (int i = 0; i < 4; ++i) bs += bf2f(static_cast<uint16_t>(dv[r][i]));
    }
#pragma unroll
    for (int dz = 0; dz < 3; ++dz) {
      // halo rows 4 wv .. 4 wv + 5, x taps 0 .. 2
      const uint16_t* xs = s_x + ((z + 2 + dz) % 3) * kWgSlot + 4 * wv * kCH * 16;
      s4 X[6][3];
#pragma unroll
      for (int r = 0; r < 6; ++r)
#pragma unroll
        for (int dx = 0; dx < 3; ++dx) X[r][dx] = read_tr(xs + (r * kCH + dx) * 16);
      // rows 2p and 2p + 1 as one K = 32 product: each lane's eight K slots
      // are its four voxels of the first row, then the same four of the second
#pragma unroll
      for (int rp = 0; rp < 2; ++rp) {
        const b8 bv = cat_bf16(dv[2 * rp], dv[2 * rp + 1]);
#pragma unroll
        for (int dy = 0; dy < 3; ++dy)
#pragma unroll
          for (int dx = 0; dx < 3; ++dx) {
            const int t = dz * 9 + dy * 3 + dx;
            acc[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
                cat_bf16(X[2 * rp + dy][dx], X[2 * rp + 1 + dy][dx]), bv, acc[t], 0, 0, 0);
          }
      }
    }
  }
  // the four waves' tiles added in LDS in wave order, lane after lane:
  // element j of lane l of tap t at (4 t + j) 64 + l
  static_assert(3 * kWgSlot * 2 >= 27 * 256 * 4, "the tap tiles fit the staged planes");
  float* red = reinterpret_cast<float*>(s_x);
  __shared__ float red_b[16];
  bs += __shfl_xor(bs, 16);
  bs += __shfl_xor(bs, 32);
  for (int w = 0; w < 4; ++w) {
    __syncthreads();
    if (wv == w) {
#pragma unroll
      for (int t = 0; t < 27; ++t)
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          float* d = red + (4 * t + j) * 64 + lane;
          *d = (w == 0 ? 0.0f : *d) + acc[t][j];
        }
      if (kq == 0) red_b[m] = (w == 0 ? 0.0f : red_b[m]) + bs;
    }
  }
  __syncthreads();
  // D[4 (l / 16) + j][l % 16] is (input channel, output channel)
  float* out = a.part + (long long)chunk * 27 * a.cin_p * a.cout_p;
  for (int e = tid; e < 27 * 256; e += 256) {
    const int t = e >> 8, j = (e >> 6) & 3, l = e & 63;
    out[((long long)t * a.cin_p + ib * 16 + 4 * (l >> 4) + j) * a.cout_p + cb * 16 + (l & 15)] =
        red[e];
  }
  if (ib == 0 && tid < 16) a.partb[(long long)chunk * a.cout_p + cb * 16 + tid] = red_b[tid];
}

// dW[t][ci][co] and db[co] = sums over chunks of the padded partials.  A block
// of 256 threads reduces 16 consecutive outputs: 16 threads per output each
// sum the chunks c = q, q + 16, ... (q = the thread's share), then the 16
// shares are added in order q = 0..15 (a fixed order, so the result does not
// depend on scheduling).  Many short sums in parallel instead of one long one
// per output: the partials of a layer can hold thousands of chunks.  The
// blocks past the weights' reduce the bias (a launch of its own cost 5 to 8
// us a layer).
constexpr int kRedShare = 16;
__global__ void __launch_bounds__(256)
    k_reduce(const float* __restrict__ part, const float* __restrict__ partb, int nchunks,
             int cin, int cout, int cin_p, int cout_p, int wblocks, float* __restrict__ dW,
             float* __restrict__ db, int accumulate) {
  constexpr int NO = 256 / kRedShare;
  __shared__ float red[kRedShare][NO];
  const bool bias = (int)blockIdx.x >= wblocks;
  const long long n = bias ? cout : 27LL * cin * cout,
                  stride = bias ? cout_p : 27LL * cin_p * cout_p;
  const int lo = threadIdx.x % NO, q = threadIdx.x / NO;
  const long long i = (long long)(bias ? blockIdx.x - wblocks : blockIdx.x) * NO + lo;
  float s = 0.0f;
  if (i < n) {
    long long o = i;
    if (!bias) {
      const int t = static_cast<int>(i / ((long long)cin * cout));
      const int r = static_cast<int>(i % ((long long)cin * cout));
      o = ((long long)t * cin_p + r / cout) * cout_p + r % cout;
    }
    const float* p = (bias ? partb : part) + o;
    for (int c = q; c < nchunks; c += kRedShare) s += p[c * stride];
  }
  red[q][lo] = s;
  __syncthreads();
  if (q == 0 && i < n) {
    float tot = 0.0f;
#pragma unroll
    for (int k = 0; k < kRedShare; ++k) tot += red[k][lo];
    float* d = (bias ? db : dW) + i;
    *d = accumulate ? *d + tot : tot;
  }
}

// ------------------------------------------------------- resampling ops
// Eight channels per thread (16-byte accesses; channel counts, strides and
// offsets multiples of 8), 32-bit indices.  They move each tensor once and
// are bound by memory; with one channel per thread and 64-bit divisions per
// element they were bound by instructions (gradient of the pooling at
// 80x96x112, 16 of 48 interleaved channels: 51 us and 33 for the ReLU mask
// after it, now 35 together; of the upsampling 21 and 9, now 16).
// mask (may be null): activations at the output's positions; the gradient is
// written as 0 where they are not positive.
struct F8 {
  float v[8];
};
__device__ __forceinline__ F8 load8(const uint16_t* p) {
  const uint4 q = *reinterpret_cast<const uint4*>(p);
  const unsigned w[4] = {q.x, q.y, q.z, q.w};
  F8 r;
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    r.v[2 * k] = __uint_as_float(w[k] << 16);
    r.v[2 * k + 1] = __uint_as_float(w[k] & 0xFFFF0000u);
  }
  return r;
}
__device__ __forceinline__ void store8(uint16_t* p, const F8& r) {
  unsigned w[4];
#pragma unroll
  for (int k = 0; k < 4; ++k)
    w[k] = __builtin_bit_cast(unsigned,
                              __builtin_convertvector(f2{r.v[2 * k], r.v[2 * k + 1]}, bf2));
  *reinterpret_cast<uint4*>(p) = uint4{w[0], w[1], w[2], w[3]};
}
__device__ __forceinline__ void mask8(F8& r, const uint16_t* a) {
  const F8 m = load8(a);
#pragma unroll
  for (int k = 0; k < 8; ++k)
    if (!(m.v[k] > 0.0f)) r.v[k] = 0.0f;
}
__device__ __forceinline__ long long child(int z, int y, int x, int k, int ny, int nx) {
  return ((long long)(2 * z + (k >> 2)) * ny + 2 * y + ((k >> 1) & 1)) * nx + 2 * x + (k & 1);
}

// 2x2x2 average pooling from fine dims (nz, ny, nx).
__global__ void k_pool2(const uint16_t* __restrict__ X, int ldx, int C, int nz, int ny,
                        int nx, uint16_t* __restrict__ Y, int ldy) {
  const int cy = ny / 2, cx = nx / 2, G = C / 8, n = (nz / 2) * cy * cx * G;
  for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < n; i += gridDim.x * blockDim.x) {
    const int g = i % G, v = i / G;
    const int x = v % cx, y = (v / cx) % cy, z = v / (cx * cy);
    F8 f[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) f[k] = load8(X + child(z, y, x, k, ny, nx) * ldx + 8 * g);
    F8 s;
#pragma unroll
    for (int c = 0; c < 8; ++c) {
      s.v[c] = 0.0f;
#pragma unroll
      for (int k = 0; k < 8; ++k) s.v[c] += f[k].v[c];
      s.v[c] *= 0.125f;
    }
    store8(Y + (long long)v * ldy + 8 * g, s);
  }
}

// Gradient of the pooling, added to dX: every fine voxel receives dY / 8.
__global__ void k_pool2_back(const uint16_t* __restrict__ dY, int ldy, int C, int nz, int ny,
                             int nx, uint16_t* __restrict__ dX, int ldx,
                             const uint16_t* __restrict__ mask, int ldm) {
  const int G = C / 8, n = nz * ny * nx * G;
  for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < n; i += gridDim.x * blockDim.x) {
    const int g = i % G, v = i / G;
    const int x = v % nx, y = (v / nx) % ny, z = v / (nx * ny);
    const int cv = ((z >> 1) * (ny >> 1) + (y >> 1)) * (nx >> 1) + (x >> 1);
    uint16_t* d = dX + (long long)v * ldx + 8 * g;
    F8 r = load8(dY + (long long)cv * ldy + 8 * g);
    const F8 o = load8(d);
#pragma unroll
    for (int c = 0; c < 8; ++c) r.v[c] = r.v[c] * 0.125f + o.v[c];
    if (mask) mask8(r, mask + (long long)v * ldm + 8 * g);
    store8(d, r);
  }
}

// x2 nearest-neighbour upsampling to fine dims (nz, ny, nx).
__global__ void k_up2(const uint16_t* __restrict__ X, int ldx, int C, int nz, int ny, int nx,
                      uint16_t* __restrict__ Y, int ldy) {
  const int G = C / 8, n = nz * ny * nx * G;
  for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < n; i += gridDim.x * blockDim.x) {
    const int g = i % G, v = i / G;
    const int x = v % nx, y = (v / nx) % ny, z = v / (nx * ny);
    const int cv = ((z >> 1) * (ny >> 1) + (y >> 1)) * (nx >> 1) + (x >> 1);
    *reinterpret_cast<uint4*>(Y + (long long)v * ldy + 8 * g) =
        *reinterpret_cast<const uint4*>(X + (long long)cv * ldx + 8 * g);
  }
}

// Gradient of the upsampling: the sum over the 8 fine children.
__global__ void k_up2_back(const uint16_t* __restrict__ dY, int ldy, int C, int nz, int ny,
                           int nx, uint16_t* __restrict__ dX, int ldx,
                           const uint16_t* __restrict__ mask, int ldm) {
  const int cy = ny / 2, cx = nx / 2, G = C / 8, n = (nz / 2) * cy * cx * G;
  for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < n; i += gridDim.x * blockDim.x) {
    const int g = i % G, v = i / G;
    const int x = v % cx, y = (v / cx) % cy, z = v / (cx * cy);
    F8 f[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) f[k] = load8(dY + child(z, y, x, k, ny, nx) * ldy + 8 * g);
    F8 s;
#pragma unroll
    for (int c = 0; c < 8; ++c) {
      s.v[c] = 0.0f;
#pragma unroll
      for (int k = 0; k < 8; ++k) s.v[c] += f[k].v[c];
    }
    if (mask) mask8(s, mask + (long long)v * ldm + 8 * g);
    store8(dX + (long long)v * ldx + 8 * g, s);
  }
}

template <typename T>
__global__ void k_input(const T* __restrict__ F, const T* __restrict__ M, int nz, int ny,
                        int nx, int pool, uint16_t* __restrict__ X) {
  const long long n = (long long)nz * ny * nx;
  const int fy = pool ? 2 * ny : ny, fx = pool ? 2 * nx : nx;
  for (long long v = blockIdx.x * (long long)blockDim.x + threadIdx.x; v < n;
       v += (long long)gridDim.x * blockDim.x) {
    float f = 0.0f, m = 0.0f;
    if (pool) {
      const int x = static_cast<int>(v % nx), y = static_cast<int>((v / nx) % ny),
                z = static_cast<int>(v / ((long long)nx * ny));
#pragma unroll
      for (int k = 0; k < 8; ++k) {
        const int i = static_cast<int>(child(z, y, x, k, fy, fx));
        f += ldf(F, i);
        m += ldf(M, i);
      }
      f *= 0.125f;
      m *= 0.125f;
    } else {
      f = ldf(F, static_cast<int>(v));
      m = ldf(M, static_cast<int>(v));
    }
    X[v * 4 + 0] = f2bf(f);
    X[v * 4 + 1] = f2bf(m);
    X[v * 4 + 2] = 0;
    X[v * 4 + 3] = 0;
  }
}

__global__ void k_head_to_field(const float* __restrict__ yf, int ldf, long long N,
                                float* __restrict__ field) {
  for (long long v = blockIdx.x * (long long)blockDim.x + threadIdx.x; v < N;
       v += (long long)gridDim.x * blockDim.x)
#pragma unroll
    for (int c = 0; c < 3; ++c) field[c * N + v] = yf[v * ldf + c];
}

// Squared error per block (FP64) and the BF16 gradient 2 (out - target) / (3N).
__global__ void __launch_bounds__(256)
    k_mse(const float* __restrict__ yf, int ldf, const float* __restrict__ target,
          float tscale, long long N, uint16_t* __restrict__ dout, int ld,
          double* __restrict__ part) {
  __shared__ double red[256];
  double s = 0.0;
  const float scale = static_cast<float>(2.0 / (3.0 * static_cast<double>(N)));
  for (long long v = blockIdx.x * (long long)blockDim.x + threadIdx.x; v < N;
       v += (long long)gridDim.x * blockDim.x) {
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      const float d = yf[v * ldf + c] - tscale * target[c * N + v];
      s += static_cast<double>(d) * d;
      dout[v * ld + c] = f2bf(scale * d);
    }
  }
  red[threadIdx.x] = s;
  __syncthreads();
  for (int w = 128; w > 0; w >>= 1) {
    if (threadIdx.x < w) red[threadIdx.x] += red[threadIdx.x + w];
    __syncthreads();
  }
  if (threadIdx.x == 0) part[blockIdx.x] = red[0];
}

// One block of 256 threads: thread t sums partials t, t + 256, ... in order,
// then a fixed tree adds the 256 sums (the result does not depend on timing).
__global__ void __launch_bounds__(256)
    k_mse_final(const double* __restrict__ part, int n, double inv, double* __restrict__ loss) {
  __shared__ double sh[256];
  double s = 0.0;
  for (int i = threadIdx.x; i < n; i += 256) s += part[i];
  sh[threadIdx.x] = s;
  __syncthreads();
  for (int w = 128; w > 0; w >>= 1) {
    if (threadIdx.x < w) sh[threadIdx.x] += sh[threadIdx.x + w];
    __syncthreads();
  }
  if (threadIdx.x == 0) *loss = sh[0] * inv;
}

__global__ void k_fill_u16(uint16_t* __restrict__ p, long long n) {
  for (long long i = blockIdx.x * (long long)blockDim.x + threadIdx.x; i < n;
       i += (long long)gridDim.x * blockDim.x)
    p[i] = 0;
}

// Adam on FP32 master parameters (bias-corrected moments: c1 = 1 - b1^t,
// c2 = 1 - b2^t); the gradient is scaled by gscale first.
__global__ void k_adam(float* __restrict__ p, float* __restrict__ m, float* __restrict__ v,
                       const float* __restrict__ g, long long n, float lr, float b1,
                       float b2, float eps, float c1, float c2, float gscale) {
  for (long long i = blockIdx.x * (long long)blockDim.x + threadIdx.x; i < n;
       i += (long long)gridDim.x * blockDim.x) {
    const float gi = g[i] * gscale;
    const float mi = b1 * m[i] + (1.0f - b1) * gi;
    const float vi = b2 * v[i] + (1.0f - b2) * gi * gi;
    m[i] = mi;
    v[i] = vi;
    p[i] -= lr * (mi / c1) / (sqrtf(vi / c2) + eps);
  }
}

__global__ void k_pack(const float* __restrict__ W, int cin, int cout, int cin_p,
                       int cout_p, uint16_t* __restrict__ Wf, uint16_t* __restrict__ Wb) {
  const int nci = cin_p / 16, nco = cout_p / 16;
  const long long n = 27LL * cin_p * cout_p;
  for (long long i = blockIdx.x * (long long)blockDim.x + threadIdx.x; i < n;
       i += (long long)gridDim.x * blockDim.x) {
    const int t = static_cast<int>(i / ((long long)cin_p * cout_p));
    const int r = static_cast<int>(i % ((long long)cin_p * cout_p));
    const int ci = r / cout_p, co = r % cout_p;
    const float w = (ci < cin && co < cout) ? W[((long long)t * cin + ci) * cout + co] : 0.0f;
    const uint16_t h = f2bf(w);
    // element of the operand: quad of the reduction channel, then the output
    // channel, then the channel within the quad
    const long long f = (((long long)(co / 16) * nci + ci / 16) * 27 + t) * 256 +
                        (((ci % 16) / 4) * 16 + co % 16) * 4 + ci % 4;
    const long long bk = (((long long)(ci / 16) * nco + co / 16) * 27 + (26 - t)) * 256 +
                         (((co % 16) / 4) * 16 + ci % 16) * 4 + co % 4;
    Wf[f] = h;
    Wb[bk] = h;
  }
}

unsigned grid_n(long long n) {
  long long b = (n + 255) / 256;
  if (b > 16384) b = 16384;
  if (b < 1) b = 1;
  return static_cast<unsigned>(b);
}

// Split of the weight gradient over z: about 512 blocks in total (two per
// compute unit), each marching through zper planes of one brick.
void wgrad_split(int cin_p, int cout_p, int nz, int ny, int nx, int& zper, int& nzp) {
  const long long per = (long long)(cin_p / 16) * (cout_p / 16) * ((nx + 15) / 16) *
                        ((ny + 15) / 16);
  long long want = (512 + per - 1) / per;
  if (want > nz) want = nz;
  if (want < 1) want = 1;
  zper = static_cast<int>((nz + want - 1) / want);
  nzp = (nz + zper - 1) / zper;
}
long long wgrad_chunks(int cin_p, int cout_p, int nz, int ny, int nx) {
  int zper, nzp;
  wgrad_split(cin_p, cout_p, nz, ny, nx, zper, nzp);
  return (long long)nzp * ((ny + 15) / 16) * ((nx + 15) / 16);
}

}  // namespace

namespace {

template <int RW, int WZ>
long long conv_tiles(const ConvArgs& a) {
  constexpr int TY = RW * (4 / WZ);
  return (long long)((a.nx + kCT - 1) / kCT) * ((a.ny + TY - 1) / TY) *
         ((a.nz + WZ - 1) / WZ);
}

template <int NT, int RW, int WZ>
hipError_t conv_tile(const ConvArgs& a, hipStream_t s) {
  const dim3 grid(static_cast<unsigned>(conv_tiles<RW, WZ>(a) * (a.cout_p / (16 * NT))));
  if (a.ldx % 8 || a.cin_valid % 8 || (reinterpret_cast<uintptr_t>(a.X) % 16))
    hipLaunchKernelGGL((k_conv_tile<NT, RW, WZ, false>), grid, dim3(256), 0, s, a);
  else
    hipLaunchKernelGGL((k_conv_tile<NT, RW, WZ, true>), grid, dim3(256), 0, s, a);
  return hipGetLastError();
}

}  // namespace

hipError_t unet_conv(const ConvArgs& a, hipStream_t s) {
  const long long tile_bytes =
      ((long long)a.nz * a.ny * a.nx * a.ldx + ((a.cin_valid + 3) & ~3)) * 2;
  if (a.ldx % 4 == 0 && (reinterpret_cast<uintptr_t>(a.X) % 8) == 0 &&
      tile_bytes < static_cast<long long>(kFarOffset) - 16) {
    // 32 output channels per block where the layer has them and that still
    // gives every compute unit a block: an input operand then feeds two
    // MFMAs and the halo is staged half as often (40x48x56, 96 -> 32: 31 us,
    // 36 us with 16); the coarser levels have too few tiles for it
    // (20x24x28, 192 -> 64: 31 us, 24 us with 16).
    if (a.cout_p % 32 == 0 && conv_tiles<4, 4>(a) * (a.cout_p / 32) >= device_cus())
      return conv_tile<2, 4, 4>(a, s);
    return conv_tile<1, 4, 4>(a, s);
  }
  dim3 grid((a.nx + 63) / 64, a.ny, a.nz * (a.cout_p / 16));
  const bool k32 = a.cin_p % 32 == 0 && a.ldx % 8 == 0 && a.cin_valid % 8 == 0 &&
                   (reinterpret_cast<uintptr_t>(a.X) % 16) == 0;
  if (k32)
    hipLaunchKernelGGL(k_conv<K32>, grid, dim3(256), 0, s, a);
  else
    hipLaunchKernelGGL(k_conv<K16>, grid, dim3(256), 0, s, a);
  return hipGetLastError();
}

long long unet_wgrad_part_floats(int cin_p, int cout_p, int nz, int ny, int nx) {
  return wgrad_chunks(cin_p, cout_p, nz, ny, nx) * 27 * cin_p * cout_p;
}

long long unet_wgrad_bias_floats(int cin_p, int cout_p, int nz, int ny, int nx) {
  return wgrad_chunks(cin_p, cout_p, nz, ny, nx) * cout_p;
}

hipError_t unet_wgrad(const uint16_t* X, int ldx, int cin, int cin_p, const uint16_t* dZ,
                      int ldz, int cout, int cout_p, int nz, int ny, int nx, float* part,
                      float* partb, float* dW, float* db, int accumulate, hipStream_t s) {
  // both tensors are read through 32-bit byte offsets
  const long long nvox = (long long)nz * ny * nx;
  if ((nvox * ldx + 4) * 2 >= static_cast<long long>(kFarOffset) ||
      (nvox * ldz + 4) * 2 >= static_cast<long long>(kFarOffset) || ldx % 4 || ldz % 4 ||
      reinterpret_cast<uintptr_t>(X) % 8 || reinterpret_cast<uintptr_t>(dZ) % 8)
    return hipErrorInvalidValue;
  WgradArgs w{X, ldx, cin, cin_p, dZ, ldz, cout, cout_p, nz, ny, nx, 0, 0, part, partb};
  wgrad_split(cin_p, cout_p, nz, ny, nx, w.zper, w.nzp);
  const long long nch = wgrad_chunks(cin_p, cout_p, nz, ny, nx);
  const unsigned blocks = static_cast<unsigned>(nch * (cin_p / 16) * (cout_p / 16));
  const bool xv = ldx % 8 == 0 && cin % 8 == 0 && reinterpret_cast<uintptr_t>(X) % 16 == 0;
  const bool dv = ldz % 8 == 0 && cout % 8 == 0 && reinterpret_cast<uintptr_t>(dZ) % 16 == 0;
  auto* kernel = xv ? (dv ? k_wgrad<true, true> : k_wgrad<true, false>)
                    : (dv ? k_wgrad<false, true> : k_wgrad<false, false>);
  hipLaunchKernelGGL(kernel, dim3(blocks), dim3(256), 0, s, w);
  const long long per = 256 / kRedShare, wblocks = (27LL * cin * cout + per - 1) / per;
  hipLaunchKernelGGL(k_reduce, dim3(static_cast<unsigned>(wblocks + (cout + per - 1) / per)),
                     dim3(256), 0, s, part, partb, static_cast<int>(nch), cin, cout, cin_p,
                     cout_p, static_cast<int>(wblocks), dW, db, accumulate);
  return hipGetLastError();
}

// Eight channels per access: counts, strides and bases.
static bool by_eight(int C, int ld, const void* p) {
  return C % 8 == 0 && ld % 8 == 0 && reinterpret_cast<uintptr_t>(p) % 16 == 0;
}

hipError_t unet_pool2(const uint16_t* X, int ldx, int C, int nz, int ny, int nx,
                      uint16_t* Y, int ldy, hipStream_t s) {
  const long long n = (long long)nz * ny * nx * C / 64;
  if (!by_eight(C, ldx, X) || !by_eight(C, ldy, Y) || n >= (1LL << 30))
    return hipErrorInvalidValue;
  hipLaunchKernelGGL(k_pool2, dim3(grid_n(n)), dim3(256), 0, s, X, ldx, C, nz, ny, nx, Y, ldy);
  return hipGetLastError();
}

hipError_t unet_pool2_back(const uint16_t* dY, int ldy, int C, int nz, int ny, int nx,
                           uint16_t* dX, int ldx, const uint16_t* mask, int ldm,
                           hipStream_t s) {
  const long long n = (long long)nz * ny * nx * C / 8;
  if (!by_eight(C, ldy, dY) || !by_eight(C, ldx, dX) || !by_eight(C, ldm, mask) ||
      n >= (1LL << 30))
    return hipErrorInvalidValue;
  hipLaunchKernelGGL(k_pool2_back, dim3(grid_n(n)), dim3(256), 0, s, dY, ldy, C, nz, ny, nx,
                     dX, ldx, mask, ldm);
  return hipGetLastError();
}

hipError_t unet_up2(const uint16_t* X, int ldx, int C, int nz, int ny, int nx, uint16_t* Y,
                    int ldy, hipStream_t s) {
  const long long n = (long long)nz * ny * nx * C / 8;
  if (!by_eight(C, ldx, X) || !by_eight(C, ldy, Y) || n >= (1LL << 30))
    return hipErrorInvalidValue;
  hipLaunchKernelGGL(k_up2, dim3(grid_n(n)), dim3(256), 0, s, X, ldx, C, nz, ny, nx, Y, ldy);
  return hipGetLastError();
}

hipError_t unet_up2_back(const uint16_t* dY, int ldy, int C, int nz, int ny, int nx,
                         uint16_t* dX, int ldx, const uint16_t* mask, int ldm,
                         hipStream_t s) {
  const long long n = (long long)nz * ny * nx * C / 64;
  if (!by_eight(C, ldy, dY) || !by_eight(C, ldx, dX) || !by_eight(C, ldm, mask) ||
      n >= (1LL << 30))
    return hipErrorInvalidValue;
  hipLaunchKernelGGL(k_up2_back, dim3(grid_n(n)), dim3(256), 0, s, dY, ldy, C, nz, ny, nx, dX,
                     ldx, mask, ldm);
  return hipGetLastError();
}

hipError_t unet_input(const void* F, const void* M, lmr_dtype t, int nz, int ny, int nx,
                      int pool, uint16_t* X, hipStream_t s) {
  const long long n = (long long)nz * ny * nx;
  if (t == LMR_BF16)
    hipLaunchKernelGGL(k_input<uint16_t>, dim3(grid_n(n)), dim3(256), 0, s,
                       static_cast<const uint16_t*>(F), static_cast<const uint16_t*>(M), nz,
                       ny, nx, pool, X);
  else
    hipLaunchKernelGGL(k_input<float>, dim3(grid_n(n)), dim3(256), 0, s,
                       static_cast<const float*>(F), static_cast<const float*>(M), nz, ny,
                       nx, pool, X);
  return hipGetLastError();
}

hipError_t unet_head_to_field(const float* yf, int ldf, long long N, float* field,
                              hipStream_t s) {
  hipLaunchKernelGGL(k_head_to_field, dim3(grid_n(N)), dim3(256), 0, s, yf, ldf, N, field);
  return hipGetLastError();
}

int unet_mse_blocks(long long N) {
  const unsigned g = grid_n(N);
  return static_cast<int>(g > 1024 ? 1024 : g);
}

hipError_t unet_mse(const float* yf, int ldf, const float* target, float tscale,
                    long long N, uint16_t* dout, int ld, double* part, double* loss,
                    hipStream_t s) {
  const int nb = unet_mse_blocks(N);
  hipLaunchKernelGGL(k_mse, dim3(nb), dim3(256), 0, s, yf, ldf, target, tscale, N, dout, ld,
                     part);
  hipLaunchKernelGGL(k_mse_final, dim3(1), dim3(256), 0, s, part, nb,
                     1.0 / (3.0 * static_cast<double>(N)), loss);
  return hipGetLastError();
}

hipError_t unet_zero(uint16_t* p, long long n, hipStream_t s) {
  hipLaunchKernelGGL(k_fill_u16, dim3(grid_n(n)), dim3(256), 0, s, p, n);
  return hipGetLastError();
}

hipError_t unet_adam(float* p, float* m, float* v, const float* g, long long n, float lr,
                     float b1, float b2, float eps, float c1, float c2, float gscale,
                     hipStream_t s) {
  hipLaunchKernelGGL(k_adam, dim3(grid_n(n)), dim3(256), 0, s, p, m, v, g, n, lr, b1, b2,
                     eps, c1, c2, gscale);
  return hipGetLastError();
}

hipError_t unet_pack(const float* W, int cin, int cout, int cin_p, int cout_p,
                     uint16_t* Wf, uint16_t* Wb, hipStream_t s) {
  hipLaunchKernelGGL(k_pack, dim3(grid_n(27LL * cin_p * cout_p)), dim3(256), 0, s, W, cin,
                     cout, cin_p, cout_p, Wf, Wb);
  return hipGetLastError();
}

}  // namespace lmr
