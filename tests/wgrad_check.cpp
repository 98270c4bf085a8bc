// Host check of every load of the weight gradient's kernel: the library's own offsets
// (wgrad_dev.h), put together as the kernel does, stay inside x and g for ragged grids
// and channels, and a lane whose coordinate is inside the grid reads that voxel.
// Prints the number of failures.
#include <cstdio>

#include "wgrad_dev.h"

using namespace fc;

static long bad = 0, seen = 0;

static void load(int64_t at, int64_t end, bool in, int64_t voxel) {
  ++seen;
  if (at < 0 || at >= end || (in && at != voxel)) ++bad;
}

static void layer(int Ci, int Co, int N, int up, int B) {
  const int nb = (N + 3) / 4, Ns = up ? (N + 1) / 2 : N;
  const int64_t V = (int64_t)N * N * N, Vs = (int64_t)Ns * Ns * Ns;
  for (int tid = 0; tid < kWgradThreads; ++tid) {
    const WgradX X = wgrad_x(tid, Ns, up);
    const WgradG G = wgrad_g(tid, N);
    for (int b = 0; b < B; b += B > 1 ? B - 1 : 1)
      for (int k = 0; k < nb * nb * nb; ++k) {
        const int bx = k % nb, by = k / nb % nb, bz = k / (nb * nb);
        const uint32_t in = wgrad_inside(bx, by, bz, N);
        const int64_t corner = wgrad_corner(bx, by, bz, Ns, up);
        for (int h = 0; h < 2; ++h) {
          const uint32_t need = h ? X.need1 : X.need0, gneed = h ? G.need1 : G.need0;
          const bool xin = (in & need) == need, gin = (in & gneed) == gneed;
          // the voxels that the pair stands for
          const int vx = 4 * bx - 1 + 2 * X.col + h, vy = 4 * by - 1 + X.row % 6,
                    vz = 4 * bz - 1 + X.row / 6;
          const bool grid = vx >= 0 && vx < N && vy >= 0 && vy < N && vz >= 0 && vz < N;
          if (xin != grid) ++bad;
          const int64_t vox = grid ? ((int64_t)(vz >> up) * Ns + (vy >> up)) * Ns + (vx >> up) : 0;
          const int gz = 4 * bz + (G.pair >> 3), gy = 4 * by + (G.pair >> 1 & 3),
                    gx = 4 * bx + 2 * (G.pair & 1) + h;
          if (gin != (gx < N && gy < N && gz < N)) ++bad;
          for (int i0 = 0; i0 < Ci; i0 += 16) {
            const int nx = Ci - i0 < 16 ? Ci - i0 : 16;
            for (int it = 0; it < kWgradXIter && 2 * it < nx; ++it) {
              const int64_t ci = 2 * it + 1 < nx ? X.c * Vs : 0;
              const int64_t base = ((int64_t)b * Ci + i0 + 2 * it) * Vs + ci;
              load(base + corner + (xin ? h ? X.off1 : X.off0 : X.own), B * Ci * Vs, xin,
                   base + vox);
            }
          }
          for (int o0 = 0; o0 < Co; o0 += 16) {
            const int ng = Co - o0 < 16 ? Co - o0 : 16;
            for (int it = 0; it < kWgradGIter && 8 * it < ng; ++it) {
              const int c = o0 + 8 * it + (8 * it + G.c < ng ? G.c : 0);
              const int64_t base = ((int64_t)b * Co + c) * V;
              load(base + ((int64_t)4 * bz * N + 4 * by) * N + 4 * bx +
                       (gin ? G.off + h : 0),
                   B * Co * V, gin, base + ((int64_t)gz * N + gy) * N + gx);
            }
          }
        }
      }
  }
}

int main() {
  const int cases[][5] = {{2, 8, 9, 0, 6},   {8, 8, 9, 0, 6},   {16, 8, 9, 1, 6},  {8, 16, 5, 0, 6},
                          {32, 16, 5, 1, 3}, {32, 32, 3, 1, 2}, {32, 32, 2, 0, 6}, {1, 3, 9, 0, 2},
                          {3, 3, 8, 0, 2},   {5, 17, 5, 0, 2},  {33, 33, 2, 0, 2}, {17, 33, 3, 0, 1},
                          {33, 17, 3, 1, 1}, {8, 1, 25, 0, 2},  {2, 8, 33, 0, 1},  {20, 48, 2, 1, 1},
                          {7, 9, 7, 1, 2},   {1, 1, 4, 0, 1},   {9, 2, 6, 1, 3}};
  for (auto& c : cases) layer(c[0], c[1], c[2], c[3], c[4]);
  std::printf("loads %ld failures %ld\n", seen, bad);
  return bad ? 1 : 0;
}
