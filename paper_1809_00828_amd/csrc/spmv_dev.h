// Sliced copy of a scalar lattice matrix (degree P <= 4, two or three
// dimensions) and its product kernel body, for one problem and for batches.
//
// Along each direction an index is either an interior vertex of the cell grid
// (box of 2P + 1 columns) or any other index (P + 1).  Rows of the same kind in
// every direction have boxes of equal shape: each of these 8 (in 2-D 4) classes
// is enumerated x fastest and cut into slices of 64 rows, one row per lane, so
// every lane of a slice takes the same steps and only the last slice of a class
// has idle lanes.  Slices are ordered by the plane and line of their first row,
// whatever their class, so neighbouring slices share their x entries.
//
// Bound by HBM (the values are read once): 1.08 GB in 213 us at 64^3 cells, p =
// 2, 5.1 TB/s.  Slices that end with their lattice line idle 3 lanes in 4 on
// small grids and leave the rows x = 0 and x = n1 - 1 to the row layout; against
// those: 35 -> 15 us at 24^3, p = 2; 135 -> 74 us at 24^3, p = 3; 299 -> 165 us
// at 20^3, p = 4; 115 -> 89 us at 48^3 and 217 -> 213 us at 64^3, p = 2.
#pragma once
#include "dev_common.h"

namespace fc {

// i-th index of a class along one direction and the start of its box
template <int P>
__device__ __forceinline__ int sell_index(bool vertex, int i, int n1, int* lo) {
  if (vertex) {
    *lo = P * i;
    return P * (i + 1);
  }
  // 0, the indices inside the cells, n1 - 1
  int g = 0;
  if constexpr (P > 1) g = i == 0 ? 0 : ((i - 1) / (P - 1)) * P + 1 + (i - 1) % (P - 1);
  g = (P == 1 ? i > 0 : g >= n1) ? n1 - 1 : g;
  *lo = min((g / P) * P, n1 - 1 - P);
  return g;
}

struct SellRow {
  int row;     // row (= lattice node) of this lane
  int base;    // first column of its box
  bool valid;
};

template <int P>
__device__ __forceinline__ SellRow sell_row(const SellSlice sl, int l, const SellView& A) {
  const bool vx = sl.cls & 1, vy = sl.cls & 2, vz = sl.cls & 4;
  const uint32_t cx = vx ? A.nv : A.nn, cy = vy ? A.nv : A.nn;
  const uint32_t count = cx * cy * (A.dim == 3 ? (vz ? A.nv : A.nn) : 1);
  const uint32_t t0 = (uint32_t)sl.chunk * 64 + l;
  const uint32_t t = min(t0, count - 1);   // idle lanes repeat the last row
  const uint32_t line = fdiv(t, vx ? A.dv : A.dn);
  const int ix = (int)(t - line * cx);
  int iy = (int)line, iz = 0;
  if (A.dim == 3) {
    iz = (int)fdiv(line, vy ? A.dv : A.dn);
    iy = (int)(line - (uint32_t)iz * cy);
  }
  int lx, ly, lz = 0, gz = 0;
  const int gx = sell_index<P>(vx, ix, A.n1, &lx);
  const int gy = sell_index<P>(vy, iy, A.n1, &ly);
  if (A.dim == 3) gz = sell_index<P>(vz, iz, A.n1, &lz);
  SellRow r;
  r.row = gx + A.n1 * (gy + A.n1 * gz);
  r.base = lx + A.n1 * (ly + A.n1 * lz);
  r.valid = t0 < count;
  return r;
}

typedef double d2 __attribute__((ext_vector_type(2)));
typedef double d2a8 __attribute__((ext_vector_type(2), aligned(8)));

// The vector a product gathers from: x itself, or p = z + beta p_old, formed as it
// is read.
struct GatherX {
  const double* x;
  __device__ __forceinline__ double one(int i) const { return x[i]; }
  __device__ __forceinline__ d2 two(int i) const {
    return *reinterpret_cast<const d2a8*>(x + i);
  }
};
struct GatherP {
  const double *z, *p;
  double beta;
  __device__ __forceinline__ double one(int i) const { return fma(beta, p[i], z[i]); }
  __device__ __forceinline__ d2 two(int i) const {
    const d2 pv = *reinterpret_cast<const d2a8*>(p + i), zv = *reinterpret_cast<const d2a8*>(z + i);
    return d2{fma(beta, pv.x, zv.x), fma(beta, pv.y, zv.y)};
  }
};

// Box entries x-pencil by x-pencil (kx fastest).  Pencils go two per round, all
// their loads issued before the first FMA: a round's 2K entries are K paired
// values per lane (one 16-byte load each, 1 KB contiguous per wave; 8 % faster
// than one 8-byte load per entry at 64^3 cells, p = 2), and each pencil's x run
// is read two entries per load.  A last round with one pencil reads its odd
// last entry alone.  kNT: the values (read once) are streamed non-temporally.
// The pencil's (y, z) offsets are stepped, not divided out of its index.
// Two pencils per round: 1 % faster than four and 3 % faster than eight at 64^3
// cells, p = 2.
template <int K, bool kNT, class X>
__device__ __forceinline__ double sell_pencils(const double* __restrict__ vs, int l, const X& x,
                                               int base, int len1, int npen, int n1) {
  double acc = 0.0;
  int qy = 0, qz = 0;   // offsets of pencil q
  for (int q = 0; q < npen; q += 2) {
    const double* vr = vs + (int64_t)128 * K * (q / 2) + 2 * l;
    const int xp0 = base + n1 * (qy + n1 * qz);
    if (++qy == len1) {
      qy = 0;
      ++qz;
    }
    if (q + 1 < npen) {
      const int xp1 = base + n1 * (qy + n1 * qz);
      if (++qy == len1) {
        qy = 0;
        ++qz;
      }
      double a[2 * K], b[2 * K];
#pragma unroll
      for (int j = 0; j < K; ++j) {
        const d2* p = reinterpret_cast<const d2*>(vr + 128 * j);
        const d2 t = kNT ? __builtin_nontemporal_load(p) : *p;
        a[2 * j] = t.x;
        a[2 * j + 1] = t.y;
      }
#pragma unroll
      for (int kx = 0; kx + 1 < K; kx += 2) {
        const d2 t0 = x.two(xp0 + kx), t1 = x.two(xp1 + kx);
        b[kx] = t0.x;
        b[kx + 1] = t0.y;
        b[K + kx] = t1.x;
        b[K + kx + 1] = t1.y;
      }
      if (K & 1) {
        b[K - 1] = x.one(xp0 + K - 1);
        b[2 * K - 1] = x.one(xp1 + K - 1);
      }
#pragma unroll
      for (int e = 0; e < 2 * K; ++e) acc = fma(a[e], b[e], acc);
    } else {
      double a[K], b[K];
#pragma unroll
      for (int j = 0; j < K / 2; ++j) {
        const d2* p = reinterpret_cast<const d2*>(vr + 128 * j);
        const d2 t = kNT ? __builtin_nontemporal_load(p) : *p;
        a[2 * j] = t.x;
        a[2 * j + 1] = t.y;
      }
      if (K & 1) {
        const double* p = vr - l + 128 * (K / 2);   // the odd last entry, alone
        a[K - 1] = kNT ? __builtin_nontemporal_load(p) : *p;
      }
#pragma unroll
      for (int kx = 0; kx + 1 < K; kx += 2) {
        const d2 t0 = x.two(xp0 + kx);
        b[kx] = t0.x;
        b[kx + 1] = t0.y;
      }
      if (K & 1) b[K - 1] = x.one(xp0 + K - 1);
#pragma unroll
      for (int e = 0; e < K; ++e) acc = fma(a[e], b[e], acc);
    }
  }
  return acc;
}

// y = A x on one slice, by one wave.  Returns (x, y) of this lane's row.  p_new (may
// be null): x of the row is stored there.
template <int P, bool kNT, class X>
__device__ __forceinline__ double sell_slice_product(const SellView& A, const SellSlice sl, int l,
                                                     const X& x, double* __restrict__ y,
                                                     double* __restrict__ p_new = nullptr) {
  const SellRow r = sell_row<P>(sl, l, A);
  const int len1 = sl.cls & 2 ? 2 * P + 1 : P + 1;
  const int npen = len1 * (A.dim == 3 ? (sl.cls & 4 ? 2 * P + 1 : P + 1) : 1);
  const double* vs = A.val + sl.off;
  const double acc = sl.cls & 1
                         ? sell_pencils<2 * P + 1, kNT>(vs, l, x, r.base, len1, npen, A.n1)
                         : sell_pencils<P + 1, kNT>(vs, l, x, r.base, len1, npen, A.n1);
  if (!r.valid) return 0.0;
  y[r.row] = acc;
  const double xr = x.one(r.row);
  if (p_new) p_new[r.row] = xr;
  return xr * acc;
}

}  // namespace fc
