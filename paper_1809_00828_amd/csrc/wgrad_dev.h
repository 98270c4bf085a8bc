// Where the weight gradient's threads load (k_conv3d_wgrad, k_learned.hip).
#pragma once
#include <hip/hip_runtime.h>

#include <cstdint>

namespace fc {

constexpr int kWgradThreads = 256;
constexpr int kWgradXIter = 8;   // 2 channels of 108 pairs of halo values at a time
constexpr int kWgradGIter = 2;   // 8 channels of 32 pairs of voxels at a time

// A thread's pair of halo values of x, the same in every brick and pair of channels:
// channel of the pair, offsets from the brick's corner, that of the brick's first voxel,
// and the bits of their coordinates (z 0-5, y 6-11, x 12-17) among those inside the grid.
struct WgradX {
  bool act;   // the other threads load what thread 0 loads
  int c, row, col;
  int off0, off1, own;
  uint32_t need0, need1;
};

// Ns: the grid of x; up: half the gradient's, nearest upsampling.
__host__ __device__ __forceinline__ WgradX wgrad_x(int tid, int Ns, int up) {
  WgradX t;
  t.act = tid < 216;
  const int xt = t.act ? tid : 0;
  t.c = xt / 108;
  const int q = xt - 108 * t.c;
  t.row = q / 3;
  t.col = q - 3 * t.row;
  const int hz = t.row / 6, hy = t.row - 6 * hz, hx = 2 * t.col;
  auto below = [&](int h) { return up ? (h + 1) >> 1 : h; };   // ((h - 1) >> up) + 1
  t.off0 = (below(hz) * Ns + below(hy)) * Ns + below(hx);
  t.off1 = t.off0 - below(hx) + below(hx + 1);
  t.own = (below(1) * Ns + below(1)) * Ns + below(1);
  t.need0 = (1u << hz) | (64u << hy) | (4096u << hx);
  t.need1 = (1u << hz) | (64u << hy) | (8192u << hx);
  return t;
}

// The same for its pair of voxels of the gradient on the grid N, from the brick's first.
struct WgradG {
  int c, pair, off;
  uint32_t need0, need1;
};

__host__ __device__ __forceinline__ WgradG wgrad_g(int tid, int N) {
  WgradG t;
  t.c = tid >> 5;
  t.pair = tid & 31;
  const int pz = t.pair >> 3, py = (t.pair >> 1) & 3, px = 2 * (t.pair & 1);
  t.off = (pz * N + py) * N + px;
  t.need0 = (2u << pz) | (128u << py) | (8192u << px);
  t.need1 = (2u << pz) | (128u << py) | (16384u << px);
  return t;
}

// Coordinates of brick (bx, by, bz) with its halo that lie inside the grid N, as bits.
__host__ __device__ __forceinline__ uint32_t wgrad_inside(int bx, int by, int bz, int N) {
  auto inside = [&](int c) {   // bit h: coordinate 4 c - 1 + h is in the grid
    const int last = N + 1 - 4 * c;
    return (c == 0 ? 62u : 63u) & ((1u << (last < 6 ? last : 6)) - 1);
  };
  return inside(bz) | (inside(by) << 6) | (inside(bx) << 12);
}

// The halo's corner in x (outside the array for the first bricks: only offsets inside
// the grid, or `own`, are added to it).
__host__ __device__ __forceinline__ int64_t wgrad_corner(int bx, int by, int bz, int Ns, int up) {
  const int step = 4 >> up;
  return ((int64_t)(bz * step - 1) * Ns + by * step - 1) * Ns + bx * step - 1;
}

}  // namespace fc
