// Coarse-to-fine pyramid (Sec. 2.1: each level inherits the warp of the
// previous one): average pooling of the images and x2 upsampling of the field.
//
//   k_avgpool        out = mean of each f^3 block, in FP32 whatever the input
//                    type (the pooled levels hold 1/8 or less of the voxels)
//   k_upsample_field fine index i samples the coarse field at (i - 0.5)/2,
//                    clamped to the coarse grid (voxel-centre alignment), by
//                    trilinear interpolation; the values are doubled because
//                    displacements are in voxels of the finer grid.
#include "pyramid.h"

#include <algorithm>

namespace lmr {

namespace {

// FC > 0: the factor is FC, known at compile time, and the f^3 loads of an
// output are all requested before the first add (same order of additions);
// FC = 0: any factor f
template <typename T, int FC>
__global__ void __launch_bounds__(256)
    k_avgpool(const T* __restrict__ in, int nz, int ny, int nx, int f_rt,
              float* __restrict__ out) {
  const int f = FC > 0 ? FC : f_rt;
  const int cz = nz / f, cy = ny / f, cx = nx / f;
  const long long n = (long long)cz * cy * cx;
  const float inv = 1.0f / static_cast<float>(f * f * f);
  for (long long o = blockIdx.x * (long long)blockDim.x + threadIdx.x; o < n;
       o += (long long)gridDim.x * blockDim.x) {
    const int x = static_cast<int>(o % cx);
    const int y = static_cast<int>((o / cx) % cy);
    const int z = static_cast<int>(o / ((long long)cx * cy));
    float s = 0.0f;
    if constexpr (FC > 0) {
      float v[FC * FC * FC];
#pragma unroll
      for (int k = 0; k < FC; ++k)
#pragma unroll
        for (int j = 0; j < FC; ++j)
#pragma unroll
          for (int i = 0; i < FC; ++i)
            v[(k * FC + j) * FC + i] =
                ldf(in, ((long long)(z * FC + k) * ny + (y * FC + j)) * nx + (x * FC + i));
#pragma unroll
      for (int q = 0; q < FC * FC * FC; ++q) s += v[q];
    } else {
      for (int k = 0; k < f; ++k)
        for (int j = 0; j < f; ++j)
          for (int i = 0; i < f; ++i)
            s += ldf(in, ((long long)(z * f + k) * ny + (y * f + j)) * nx + (x * f + i));
    }
    out[o] = s * inv;
  }
}

__device__ __forceinline__ void src_coord(int i, int nc, int& i0, int& i1, float& t) {
  float s = (static_cast<float>(i) - 0.5f) * 0.5f;
  s = fminf(fmaxf(s, 0.0f), static_cast<float>(nc - 1));
  const float b = floorf(s);
  i0 = static_cast<int>(b);
  i1 = i0 + 1 < nc ? i0 + 1 : i0;
  t = s - b;
}

// One thread per fine x and pair of fine rows and planes: the fine indices
// 2 m + 1 and 2 m + 2 lie between the coarse ones m and m + 1, so the four
// outputs share their eight corners (m = -1 and the last one hold a single
// fine index each).  Bound by the stores; with a thread per output the
// corners were read, and the index taken apart in 64-bit divisions, four times
// as often (to 160x192x224: 47 us, now 24; to 80x96x112: 11, 6.6).
constexpr int kUpX = 64, kUpY = 4;

__global__ void __launch_bounds__(kUpX* kUpY)
    k_upsample_field(const DevState* __restrict__ st, const float* uc0,
                     const float* uc1, int nzc, int nyc, int nxc, float* __restrict__ uf) {
  // the coarse field: uc0, or with a pair state the buffer its ping-pong
  // index names (the level's current field, read where it lies)
  const float* __restrict__ uc = (st && st->cur) ? uc1 : uc0;
  const int nz = 2 * nzc, ny = 2 * nyc, nx = 2 * nxc;
  const long long N = (long long)nz * ny * nx, Nc = (long long)nzc * nyc * nxc;
  const int x = blockIdx.x * kUpX + threadIdx.x;
  if (x >= nx) return;
  int x0, x1, y0, y1, z0, z1;
  float tx, ty[2], tz[2];
  src_coord(x, nxc, x0, x1, tx);
  const int my0 = static_cast<int>(blockIdx.y * kUpY + threadIdx.y) - 1;
  for (int my = my0; my < nyc; my += gridDim.y * kUpY) {
    const int ya = max(2 * my + 1, 0), yb = min(2 * my + 2, ny - 1);
    src_coord(ya, nyc, y0, y1, ty[0]);
    src_coord(yb, nyc, y0, y1, ty[1]);
    for (int mz = static_cast<int>(blockIdx.z) - 1; mz < nzc; mz += gridDim.z) {
      const int za = max(2 * mz + 1, 0), zb = min(2 * mz + 2, nz - 1);
      src_coord(za, nzc, z0, z1, tz[0]);
      src_coord(zb, nzc, z0, z1, tz[1]);
#pragma unroll
      for (int c = 0; c < 3; ++c) {
        const float* a = uc + c * Nc;
        auto row = [&](int zz, int yy) {
          const float* r = a + ((long long)zz * nyc + yy) * nxc;
          return (1 - tx) * r[x0] + tx * r[x1];
        };
        const float r00 = row(z0, y0), r01 = row(z0, y1), r10 = row(z1, y0), r11 = row(z1, y1);
        float* o = uf + c * N + x;
#pragma unroll
        for (int j = 0; j < 2; ++j) {
          const float v0 = (1 - ty[j]) * r00 + ty[j] * r01;
          const float v1 = (1 - ty[j]) * r10 + ty[j] * r11;
          const int y = j ? yb : ya;
#pragma unroll
          for (int k = 0; k < 2; ++k) {
            const int z = k ? zb : za;
            o[((long long)z * ny + y) * nx] = 2.0f * ((1 - tz[k]) * v0 + tz[k] * v1);
          }
        }
      }
    }
  }
}

unsigned grid_for(long long n) {
  long long b = (n + 255) / 256;
  if (b > 16384) b = 16384;
  if (b < 1) b = 1;
  return static_cast<unsigned>(b);
}

}  // namespace

hipError_t launch_avgpool(const void* in, lmr_dtype t, int nz, int ny, int nx, int f,
                          float* out, hipStream_t s) {
  const long long n = (long long)(nz / f) * (ny / f) * (nx / f);
  const dim3 grid(grid_for(n)), blk(256);
  if (t == LMR_BF16) {
    const auto* p = static_cast<const uint16_t*>(in);
    if (f == 2)
      hipLaunchKernelGGL((k_avgpool<uint16_t, 2>), grid, blk, 0, s, p, nz, ny, nx, f, out);
    else if (f == 4)
      hipLaunchKernelGGL((k_avgpool<uint16_t, 4>), grid, blk, 0, s, p, nz, ny, nx, f, out);
    else
      hipLaunchKernelGGL((k_avgpool<uint16_t, 0>), grid, blk, 0, s, p, nz, ny, nx, f, out);
  } else {
    const auto* p = static_cast<const float*>(in);
    if (f == 2)
      hipLaunchKernelGGL((k_avgpool<float, 2>), grid, blk, 0, s, p, nz, ny, nx, f, out);
    else if (f == 4)
      hipLaunchKernelGGL((k_avgpool<float, 4>), grid, blk, 0, s, p, nz, ny, nx, f, out);
    else
      hipLaunchKernelGGL((k_avgpool<float, 0>), grid, blk, 0, s, p, nz, ny, nx, f, out);
  }
  return hipGetLastError();
}

hipError_t launch_upsample_field(const float* uc, int nzc, int nyc, int nxc, float* uf,
                                 hipStream_t s) {
  return launch_upsample_cur(nullptr, uc, uc, nzc, nyc, nxc, uf, s);
}

hipError_t launch_upsample_cur(const DevState* st, const float* U0, const float* U1,
                               int nzc, int nyc, int nxc, float* uf, hipStream_t s) {
  const dim3 grid((2u * nxc + kUpX - 1) / kUpX, std::min((nyc + 1u + kUpY - 1) / kUpY, 65535u),
                  std::min(nzc + 1, 65535));
  hipLaunchKernelGGL(k_upsample_field, grid, dim3(kUpX, kUpY), 0, s, st, U0, U1, nzc, nyc, nxc,
                     uf);
  return hipGetLastError();
}

}  // namespace lmr
