// Device helpers of the Schwarz block products shared by the single-problem
// and batched kernels.
#pragma once
#include "dev_common.h"

namespace fc {

// Elements per block of the wrapped-diagonal symmetric layout.
__host__ __device__ __forceinline__ int64_t sym_block_stride_dev(int m) {
  return (int64_t)(m / 2 + 1) * m;
}

// Offset of stored entry (k, i) = P_B[i][(i + k) mod m] of a block in the
// wrapped-diagonal layout.  m > 64 (one block per workgroup): stored row by
// stored row.  m <= 64 (one lane per column i): stored rows 2j and 2j + 1
// interleaved column by column, so a lane's two entries are adjacent and
// one two-wide load; an odd last stored row follows alone.
__host__ __device__ __forceinline__ int64_t sym_offset(int k, int i, int m) {
  if (m > 64) return (int64_t)k * m + i;
  const int npair = (m / 2 + 1) & ~1;   // stored rows that come in pairs
  return k < npair ? (int64_t)(k & ~1) * m + 2 * i + (k & 1) : (int64_t)k * m + i;
}

// Offset of the stored entry that stands for P_B[i][j].
__host__ __device__ __forceinline__ int64_t sym_entry(int i, int j, int m) {
  const int k = j >= i ? j - i : j - i + m;
  return k <= m / 2 ? sym_offset(k, i, m) : sym_offset(m - k, j, m);
}

template <typename T>
__device__ __forceinline__ double to_f64(T v);
template <>
__device__ __forceinline__ double to_f64<double>(double v) { return v; }
template <>
__device__ __forceinline__ double to_f64<float>(float v) { return (double)v; }
template <>
__device__ __forceinline__ double to_f64<uint16_t>(uint16_t v) { return (double)bf16_to_f32(v); }

template <typename T>
__device__ __forceinline__ float to_f32(T v);
template <>
__device__ __forceinline__ float to_f32<float>(float v) { return v; }
template <>
__device__ __forceinline__ float to_f32<uint16_t>(uint16_t v) { return bf16_to_f32(v); }
template <>
__device__ __forceinline__ float to_f32<double>(double v) { return (float)v; }

// Accumulator: FP64 for FP64 storage, FP32 for the low-precision copies.
template <typename T>
struct Acc {
  using type = float;
};
template <>
struct Acc<double> {
  using type = double;
};

template <typename A, typename T>
__device__ __forceinline__ A madd(T a, double r, A acc) {
  if constexpr (sizeof(A) == 8)
    return fma(to_f64<T>(a), r, acc);
  else
    return fmaf(to_f32<T>(a), (float)r, acc);
}

__device__ __forceinline__ double gather_r(const double* r, const double* q, double alpha,
                                           int64_t dof) {
  double v = r[dof];
  if (q) v = fma(-alpha, q[dof], v);
  return v;
}

// Symmetric product of one block (m > 64) by a whole workgroup of
// 64 ceil(m/64) threads, one output row i per thread (threads with i >= m
// take part in the loads and barriers only).  A chunk of stored rows is one
// contiguous run of the block; every thread loads 16-byte pieces of it
// (half the load instructions of one entry per thread, and no idle lanes),
// non-temporally, into LDS, and each thread then reads its own entry and
// the rotated one back from LDS, so HBM and L2 see each stored entry exactly
// once.  The next chunk's loads are issued before the current chunk is
// summed.  gather() writes the block's right-hand side to rB (m entries, in
// LDS) once the first chunk's loads are in flight.  Chunks of few rows: the less
// LDS a workgroup holds, the more of them stream at once.  tile (16-byte aligned) holds kStageRows * m entries,
// as tile[kk * m + j] for stored row k0 + kk.
template <typename T, int kStageRows, typename RB, typename F>
__device__ __forceinline__ double sym_block_staged(const T* __restrict__ Qb, const RB* rB,
                                                        int m, int i, T* tile, F&& gather) {
  using A = typename Acc<T>::type;
  constexpr int V = 16 / sizeof(T);                // entries per 16-byte piece
  static_assert(kStageRows % V == 0, "whole pieces per thread");
  constexpr int kPer = kStageRows / V;             // pieces per thread per chunk (m <= threads)
  typedef T tv __attribute__((ext_vector_type(V), aligned(sizeof(T))));
  typedef T tva __attribute__((ext_vector_type(V), aligned(16)));
  const int nt = blockDim.x, t = threadIdx.x;
  const bool act = i < m;
  const int h = m / 2;
  const bool even = (m & 1) == 0;
  A acc0 = 0, acc1 = 0;
  int ip = i, im = i;
  // chunk k0's pieces are loaded while chunk k0 - kStageRows is summed
  auto load_chunk = [&](int k0, tv* v) {
    const int cnt = min(kStageRows, h + 1 - k0) * m;
    const T* src = Qb + (int64_t)k0 * m;
#pragma unroll
    for (int u = 0; u < kPer; ++u) {
      const int e = (t + nt * u) * V;
      if (e + V <= cnt) {
        v[u] = __builtin_nontemporal_load(reinterpret_cast<const tv*>(src + e));
      } else {
#pragma unroll
        for (int c = 0; c < V; ++c) v[u][c] = e + c < cnt ? __builtin_nontemporal_load(src + e + c) : T(0);
      }
    }
  };
  tv v[kPer];
  load_chunk(0, v);
  gather();
  for (int k0 = 0; k0 <= h; k0 += kStageRows) {
    const int cnt = min(kStageRows, h + 1 - k0) * m;   // entries of this chunk
    __syncthreads();   // previous chunk's reads are done
#pragma unroll
    for (int u = 0; u < kPer; ++u) {
      const int e = (t + nt * u) * V;
      if (e < cnt) *reinterpret_cast<tva*>(tile + e) = v[u];   // the pad past cnt is never read
    }
    __syncthreads();
    if (k0 + kStageRows <= h) load_chunk(k0 + kStageRows, v);
    if (act) {
#pragma unroll
      for (int kk = 0; kk < kStageRows; ++kk) {
        const int k = k0 + kk;
        if (k > h) break;
        const T* row = tile + kk * m;
        if (k == 0) {
          acc0 = madd<A>(row[i], rB[i], acc0);
          continue;
        }
        ip = (ip + 1 == m) ? 0 : ip + 1;
        im = (im == 0) ? m - 1 : im - 1;
        acc0 = madd<A>(row[i], rB[ip], acc0);
        if (!(even && k == h)) acc1 = madd<A>(row[im], rB[im], acc1);
      }
    }
  }
  return (double)acc0 + (double)acc1;
}

// Wrapped-diagonal symmetric product for one block row i (0 <= i < m), in
// either layout of sym_offset.
template <typename T>
__device__ __forceinline__ double sym_row(const T* __restrict__ Qb, const double* rb, int m,
                                          int i) {
  using A = typename Acc<T>::type;
  const int h = m / 2;
  const bool even = (m & 1) == 0;
  A acc0 = 0, acc1 = 0;
  acc0 = madd<A>(Qb[sym_offset(0, i, m)], rb[i], acc0);
  int ip = i, im = i;
#pragma unroll 4
  for (int k = 1; k <= h; ++k) {
    ip = (ip + 1 == m) ? 0 : ip + 1;   // (i + k) mod m
    im = (im == 0) ? m - 1 : im - 1;   // (i - k) mod m
    acc0 = madd<A>(Qb[sym_offset(k, i, m)], rb[ip], acc0);
    if (!(even && k == h)) acc1 = madd<A>(Qb[sym_offset(k, im, m)], rb[im], acc1);
  }
  return (double)acc0 + (double)acc1;
}

// One block (m > 64) by a workgroup of 64 ceil(m / 64) threads, its stored rows
// staged through LDS.  The right-hand side is
// gathered, and the step length taken, behind the first loads of the inverse.
// dof_of(i): unknown of row i (< 0: none).  yb null: nothing is stored.
template <typename T, int kRows, class Dof>
__device__ __forceinline__ void schwarz_staged_block(
    const T* __restrict__ Qb, double* __restrict__ yb, int m, const double* __restrict__ r,
    const double* __restrict__ q, const double* __restrict__ isd, CgScalars* sc,
    const AlphaIn ai, bool first, typename Acc<T>::type* rB, T* tile, double* red, Dof&& dof_of) {
  using A = typename Acc<T>::type;
  const int i = threadIdx.x;
  const bool act = i < m;
  int64_t dof = -1;
  bool stop = false;
  auto gather = [&] {
    double alpha = (sc && q && !ai.np) ? sc->alpha : 0.0;
    double gr = 0.0, gq = 0.0, gs = 1.0;
    if (act) {
      dof = dof_of(i);
      if (dof >= 0) {
        gr = r[dof];
        if (q) gq = q[dof];
        if (isd) gs = isd[dof];
      }
    }
    if (ai.np) stop = !cg_alpha(sc, ai, red, &alpha, first);
    if (act) rB[i] = dof >= 0 ? (A)((q ? fma(-alpha, gq, gr) : gr) * gs) : A(0);
  };
  const double v = sym_block_staged<T, kRows>(Qb, rB, m, i, tile, gather);
  if (act && !stop && yb) yb[i] = dof < 0 ? 0.0 : isd ? v * isd[dof] : v;
}

// Column i of the stored rows of a block of kM <= 64, in pairs (sym_offset): one
// two-wide load each.
template <typename T, int kM>
__device__ __forceinline__ void small_rows(const T* __restrict__ Pb, int i, T (&v)[kM / 2 + 1]) {
  constexpr int kH = kM / 2, kNP = (kH + 1) & ~1;
  typedef T t2 __attribute__((ext_vector_type(2), aligned(sizeof(T))));
#pragma unroll
  for (int k = 0; k < kNP; k += 2) {
    const t2 t = *reinterpret_cast<const t2*>(Pb + k * kM + 2 * i);
    v[k] = t.x;
    v[k + 1] = t.y;
  }
  if constexpr (kNP < kH + 1) v[kH] = Pb[kH * kM + i];
}

// Row i of the product from its lane's column v and the right-hand side rb of the
// block whose columns lie in lanes g0 .. g0 + kM - 1.
template <typename T, int kM>
__device__ __forceinline__ double small_product(const T (&v)[kM / 2 + 1], const double* rb, int i,
                                                int g0) {
  using A = typename Acc<T>::type;
  constexpr int kH = kM / 2;
  A acc0 = madd<A>(v[0], rb[i], A(0)), acc1 = 0;
#pragma unroll
  for (int k = 1; k <= kH; ++k) {
    const int ip = i + k < kM ? i + k : i + k - kM;   // (i + k) mod m
    const int im = i >= k ? i - k : i - k + kM;       // (i - k) mod m
    const T vr = __shfl(v[k], g0 + im, 64);
    acc0 = madd<A>(v[k], rb[ip], acc0);
    if (!((kM & 1) == 0 && k == kH)) acc1 = madd<A>(vr, rb[im], acc1);
  }
  return (double)acc0 + (double)acc1;
}

// m <= 64: each wave handles floor(64/m) blocks, one lane per output row.
// kM > 0 (m = kM known at compile time): lane i loads its
// column of the stored rows (Q_B[k][i] = P_B[i][(i + k) mod m], k = 0 ..
// m/2; two rows per load, as sym_offset pairs them) into registers before
// it gathers r_B, so the block's stream is in
// flight during the gather; the entries P_B[i][(i - k) mod m] =
// Q_B[k][(i - k) mod m] are then read from the lane that loaded them (a
// cross-lane read within the wave).  kM = 0: any m, the stored rows read
// after the gather (sym_row).  kLat: the blocks are the cells of
// a lattice in order, so a row's unknown follows from the block and row
// indices and the gather of r_B is issued together with the stored rows.  tile: index of the
// workgroup's 4 floor(64/m) blocks; dof_of(blk, i): unknown of row i (< 0:
// none).
template <typename T, int kM, bool kLat, class Dof>
__device__ __forceinline__ void schwarz_small_tile(
    const T* __restrict__ P, int64_t block_stride, int m_arg, const double* __restrict__ r,
    const double* __restrict__ q, const double* __restrict__ isd, CgScalars* sc,
    const AlphaIn ai, bool first, double* __restrict__ y, int64_t n_blocks,
    const PullLattice& lat, int64_t tile, double (*rB)[64], double* red, Dof&& dof_of) {
  const int m = kM > 0 ? kM : m_arg;
  double alpha = (sc && q && !ai.np) ? sc->alpha : 0.0;
  const int bpw = 64 / m;
  const int w = threadIdx.x / 64, l = threadIdx.x % 64;
  const int lb = l / m, i = l % m;
  const int64_t blk = (tile * 4 + w) * bpw + lb;
  const bool active = lb < bpw && blk < n_blocks;
  // lanes without a block read block 0 (always present) and store nothing
  const T* Pb = P + (active ? blk : 0) * block_stride;
  constexpr int kH = kM / 2;
  T v[kH + 1];
  int64_t dof = -1;
  double g_r = 0.0, g_q = 0.0, g_s = 1.0;
  if constexpr (kLat) {
    // the gathered entries are loaded first and the stored rows next, all
    // without branches (a lane without a block reads unknown 0), and only
    // then combined: the wait for the gather does not wait for the rows
    // (the lattice is set for scalar problems only: one unknown per node)
    dof = active ? lattice_cell_node(lat, (int)blk, i) : 0;
    g_r = r[dof];
    g_q = (q ? q : r)[dof];
    g_s = (isd ? isd : r)[dof];
  }
  if constexpr (kM > 0) small_rows<T, kM>(Pb, i, v);
  if constexpr (!kLat) {
    if (active) {
      dof = dof_of(blk, i);
      if (dof >= 0) {
        g_r = r[dof];
        if (q) g_q = q[dof];
        if (isd) g_s = isd[dof];
      }
    }
  }
  if (ai.np && !cg_alpha(sc, ai, red, &alpha, first)) return;
  const double rv = (q ? fma(-alpha, g_q, g_r) : g_r) * (isd ? g_s : 1.0);
  if (active) rB[w][l] = rv;
  __syncthreads();
  double out;
  if constexpr (kM > 0) {
    // every lane takes part in the cross-lane reads; a lane without a block
    // reads its own group's entries and discards the result
    const int g0 = (active ? lb : 0) * kM;
    out = small_product<T, kM>(v, &rB[w][g0], i, g0);
  } else {
    if (!active) return;
    const double* rb = &rB[w][lb * m];
    out = sym_row<T>(Pb, rb, m, i);
  }
  if (!active) return;
  y[blk * m + i] = dof < 0 ? 0.0 : isd ? out * isd[dof] : out;
}

// List of the block sizes m <= 64 with kernels of their own: scalar and vector
// problems at p = 1 .. 3 (2-D and 3-D) and p up to 6 (2-D).
#define FC_SMALL_SIZES(X) \
  X(8) X(9) X(16) X(18) X(24) X(25) X(27) X(32) X(36) X(49) X(50) X(64)

}  // namespace fc
