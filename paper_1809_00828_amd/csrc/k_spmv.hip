// Block-sparse (BSR) matrix-vector product y = A x for the assembled finite
// cell stiffness matrix (Sec. 3.1, Eq. 2); the product with A is half of
// every PCG iteration (Sec. 5.4 names the matrix-vector products as the
// dominant work of the solver).
//
// Layout (row-SoA BSR): the values of block row i are stored entry-major,
// val[rowptr[i]*B*B + e*L + k] for entry e of the k-th block of the row,
// so G lanes sweeping the blocks of one row read G consecutive values per
// entry (two adjacent blocks per lane for 2x2 and 3x3 blocks, so each entry
// of a lane is one 16-byte load).  A group of G lanes owns one block row;
// its partial sums are combined with a butterfly reduction.  Every block row reads its own
// stored values once per product; FP64 3x3 values and column indices are
// streamed with non-temporal loads, which leaves the cache to the gathered x
// entries (neighbouring rows of the lattice share most of their columns).
// The group width G is fixed at set-up from the mean row length, so the
// summation order of a row, and with it every result, is the same in every
// process.
//
// Tiles of 256/G rows are dealt out so that the workgroups resident on one
// XCD (hardware ids congruent mod 8) walk one contiguous range of rows and
// share that XCD's L2 for x.  The PCG variant leaves one partial (x, y) per
// workgroup, up to 1,024 of them; the workgroups of the block products sum them
// in a fixed order (no atomics).
//
// Matrices assembled from a problem description have lattice rows: the
// columns and the start of each row follow from the row's lattice indices
// and are computed, not read.  Scalar ones (degree p <= 4) also keep a
// sliced copy, 64 rows with boxes of equal shape per slice (spmv_dev.h), for
// the whole-matrix product (k_spmv_sell below) unless the rows are few and
// long (routes.h).
#include <algorithm>
#include <cstdlib>
#include <vector>

#include "dev_common.h"
#include "k_spmv.h"
#include "routes.h"
#include "spmv_dev.h"

namespace fc {

// Matrix data is read once per product.  FP64 3x3 blocks read it
// non-temporally; scalar rows and the FP32 copy read it through the caches,
// which is 13 % faster at 64^3 p = 2 and 3.5 % for the FP32 rows of the
// mixed product (measured; there the non-temporal stream costs more than
// it saves).
template <bool kNT, typename T>
__device__ __forceinline__ T stream_load(const T* p) {
  if constexpr (kNT) return __builtin_nontemporal_load(p);
  else return *p;
}

// rows (may be null): the launch covers only these n_rows block rows
// (ascending), the others of y are left alone.
// kLat: columns computed from the lattice box (col is not read).
// XT: type of x (FP32 for the FP32 rows of the mixed product, which round
// x to FP32 before every product anyway).
// U: blocks per lane per pass (all loads of a pass are in flight together);
// U = 2 takes two adjacent blocks, so each entry is one two-wide load (half
// the load instructions of two separate blocks: 5.5 % faster for the 3x3
// rows of 32^3-cell p = 3 elasticity).
// kNT: stream the matrix values non-temporally.
// At most 96 VGPRs, five waves per SIMD: the paired loads otherwise take 105
// VGPRs and four waves, which is 3 % slower.
template <int B, int G, typename T, bool kLat, typename XT, int U, bool kNT>
__global__ __launch_bounds__(256, 5) void k_spmv_bsr(
    const int32_t* __restrict__ rowptr, const int32_t* __restrict__ col,
    const T* __restrict__ val, const XT* __restrict__ x,
    double* __restrict__ y, int64_t n_rows, const CgScalars* __restrict__ sc,
    double* __restrict__ partial, const int32_t* __restrict__ rows, const LatticeInfo lat) {
  constexpr int BB = B * B;
  constexpr int RPW = 256 / G;   // rows per tile
  __shared__ double lds[16];
  if (sc && sc->done) return;
  const int64_t ntiles = (n_rows + RPW - 1) / RPW;
  // XCD-contiguous tile ranges
  const XcdRange xr_ = xcd_range(blockIdx.x, gridDim.x, ntiles);
  const uint32_t j = xr_.j, per = xr_.per;
  const int64_t t0 = xr_.t0, t1 = xr_.t1;
  const int lane = threadIdx.x % G;
  double dot = 0.0;
  for (int64_t tile = t0 + j; tile < t1; tile += per) {
    // one row per wave (G = 64): the row and everything derived from it are
    // wave-uniform, so they are computed once per wave in scalar registers
    const int wrow = G == 64 ? (int)__builtin_amdgcn_readfirstlane(threadIdx.x / G)
                             : (int)(threadIdx.x / G);
    const int64_t idx = tile * RPW + wrow;
    if (idx >= n_rows) continue;
    const int64_t row = rows ? (int64_t)rows[idx] : idx;
    // on the lattice the row's start and length follow from its indices,
    // so the value stream does not wait for a row-pointer load
    RowBox box;
    int64_t base;
    int L;
    if constexpr (kLat) {
      int c[3];
      lattice_coords(row, lat, c);
      box = row_box_at(c, lat);
      base = lattice_row_start_at(c, box, lat);
      L = box.len[0] * box.len[1] * box.len[2];
    } else {
      base = rowptr[row];
      L = rowptr[row + 1] - (int32_t)base;
    }
    const T* v = val + base * BB;
    double acc[B];
    float accf[B];
#pragma unroll
    for (int i = 0; i < B; ++i) {
      acc[i] = 0.0;
      accf[i] = 0.0f;
    }
    // U == 2: a lane takes two adjacent blocks, so each entry of the pair
    // is one 2-wide load (16 bytes for FP64; 8-byte aligned, which the
    // hardware loads as one access)
    constexpr bool kPair = U == 2;
    const int k0 = kPair ? 2 * lane : lane;
    for (int k = k0; k < L; k += U * G) {
      int c[U];
      T a[U][BB];
      if constexpr (kPair) {
        typedef T t2 __attribute__((ext_vector_type(2), aligned(sizeof(T))));
#pragma unroll
        for (int u = 0; u < 2; ++u) {
          const bool on = k + u < L;
          if constexpr (kLat)
            c[u] = on ? lattice_col(box, k + u, lat.n1) : -1;
          else
            c[u] = on ? stream_load<kNT>(col + base + k + u) : -1;
        }
        if (k + 1 < L) {
#pragma unroll
          for (int e = 0; e < BB; ++e) {
            const t2* p = reinterpret_cast<const t2*>(v + (int64_t)e * L + k);
            const t2 t = kNT ? __builtin_nontemporal_load(p) : *p;
            a[0][e] = t.x;
            a[1][e] = t.y;
          }
        } else {
#pragma unroll
          for (int e = 0; e < BB; ++e) {
            a[0][e] = stream_load<kNT>(v + (int64_t)e * L + k);
            a[1][e] = T(0);
          }
        }
      } else {
#pragma unroll
        for (int u = 0; u < U; ++u) {
          const int ku = k + u * G;
          const bool on = ku < L;
          if constexpr (kLat)
            c[u] = on ? lattice_col(box, ku, lat.n1) : -1;
          else
            c[u] = on ? stream_load<kNT>(col + base + ku) : -1;
#pragma unroll
          for (int e = 0; e < BB; ++e)
            a[u][e] = on ? stream_load<kNT>(v + (int64_t)e * L + ku) : T(0);
        }
      }
      XT xv[U][B];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        if constexpr (B == 3) {
          typedef XT x2 __attribute__((ext_vector_type(2), aligned(sizeof(XT))));
          const int64_t cc = c[u] >= 0 ? (int64_t)c[u] * B : 0;
          const x2 t = *reinterpret_cast<const x2*>(x + cc);
          const XT t2 = x[cc + 2];
          xv[u][0] = c[u] >= 0 ? t.x : XT(0);
          xv[u][1] = c[u] >= 0 ? t.y : XT(0);
          xv[u][2] = c[u] >= 0 ? t2 : XT(0);
        } else {
#pragma unroll
          for (int jj = 0; jj < B; ++jj) xv[u][jj] = c[u] >= 0 ? x[(int64_t)c[u] * B + jj] : XT(0);
        }
      }
#pragma unroll
      for (int u = 0; u < U; ++u)
#pragma unroll
        for (int i = 0; i < B; ++i)
#pragma unroll
          for (int jj = 0; jj < B; ++jj) {
            if constexpr (sizeof(T) == 8)
              acc[i] = fma((double)a[u][i * B + jj], (double)xv[u][jj], acc[i]);
            else
              accf[i] = fmaf((float)a[u][i * B + jj], (float)xv[u][jj], accf[i]);
          }
    }
    constexpr int kOut = G == 64 ? 63 : 0;   // the lane that holds the row's sums
#pragma unroll
    for (int i = 0; i < B; ++i) {
      if constexpr (G == 64)
        acc[i] = wave_sum_last(sizeof(T) == 8 ? acc[i] : (double)accf[i]);
      else if constexpr (sizeof(T) == 8)
        acc[i] = group_sum<G>(acc[i]);
      else
        acc[i] = (double)group_sum<G>(accf[i]);
    }
    if (lane == kOut) {
#pragma unroll
      for (int i = 0; i < B; ++i) {
        y[row * B + i] = acc[i];
        if (partial) dot = fma((double)x[row * B + i], acc[i], dot);
      }
    }
  }
  if (!partial) return;
  dot = block_sum(dot, lds);
  if (threadIdx.x == 0) partial[blockIdx.x] = dot;
}

// ---------------------------------------------------------------- sliced
// sell_val from the row layout, one workgroup per slice
template <int P>
__global__ __launch_bounds__(256) void k_sell_build(const double* __restrict__ val,
                                                    const SellView A, const LatticeInfo lat,
                                                    double* __restrict__ sv) {
  for (int64_t s = blockIdx.x; s < A.n_slices; s += gridDim.x) {
    const SellSlice sl = A.slices[s];
    const int l = threadIdx.x % 64;
    const SellRow r = sell_row<P>(sl, l, A);
    int c[3];
    lattice_coords(r.row, lat, c);
    const RowBox box = row_box_at(c, lat);
    const int len = box.len[0] * box.len[1] * box.len[2];
    const double* v = val + lattice_row_start_at(c, box, lat);
    for (int k = threadIdx.x / 64; k < len; k += 4) {
      // entries in pairs: lane l holds entries 2j, 2j + 1 at 128 j + 2 l + 0/1;
      // an odd last entry alone at 128 j + l
      const int dst = (k == len - 1 && (len & 1)) ? (k / 2) * 128 + l
                                                  : (k / 2) * 128 + 2 * l + (k & 1);
      sv[sl.off + dst] = r.valid ? v[k] : 0.0;
    }
  }
}

// y = A x, one wave per slice.  partial (may be null): (x, y) per workgroup.
template <int P, bool kNT>
__global__ __launch_bounds__(256) void k_spmv_sell(const SellView A, const double* __restrict__ x,
                                                   double* __restrict__ y,
                                                   double* __restrict__ partial,
                                                   const CgScalars* __restrict__ sc) {
  __shared__ double lds[4];
  if (sc && sc->done) return;
  // the slice is wave-uniform, and what depends on it alone stays in scalar
  // registers
  const int l = threadIdx.x % 64, w = __builtin_amdgcn_readfirstlane(threadIdx.x / 64);
  const int64_t s = xcd_remap(blockIdx.x, gridDim.x) * 4 + w;
  double dot = 0.0;
  if (s < A.n_slices) dot = sell_slice_product<P, kNT>(A, A.slices[s], l, GatherX{x}, y);
  if (!partial) return;
  dot = wave_sum_last(dot);
  if (l == 63) lds[w] = dot;
  __syncthreads();
  if (threadIdx.x == 0) partial[blockIdx.x] = ((lds[0] + lds[1]) + lds[2]) + lds[3];
}

// The same on p = z + beta p_old, with beta from the np <= kBetaSets partial sets of
// the pull (cg_beta_sum): the p update of a step, its stop test and scalars (by the
// first workgroup) and the product of the next, in one launch.  p goes to p_new,
// since neighbours still read p_old.
template <int P>
__global__ __launch_bounds__(256) void k_spmv_sell_beta(
    const SellView A, const double* __restrict__ z, const double* __restrict__ p_old,
    double* __restrict__ p_new, double* __restrict__ y, double* __restrict__ partial,
    const double* __restrict__ sets, int np, CgScalars* sc) {
  __shared__ double red[3][4];
  if (beta_stopped(sc, blockIdx.x == 0)) return;
  const int l = threadIdx.x % 64, w = __builtin_amdgcn_readfirstlane(threadIdx.x / 64);
  const int64_t s = xcd_remap(blockIdx.x, gridDim.x) * 4 + w;
  const double rz_old = sc->rz;
  const double rz = cg_beta_sum(sets, np, np, red, blockIdx.x == 0);
  if (blockIdx.x == 0 && threadIdx.x == 0) cg_beta_finish(sc, rz, red);
  double dot = 0.0;
  if (s < A.n_slices)
    dot = sell_slice_product<P, true>(A, A.slices[s], l, GatherP{z, p_old, rz / rz_old}, y, p_new);
  dot = wave_sum_last(dot);
  __syncthreads();   // red is read
  if (l == 63) red[0][w] = dot;
  __syncthreads();
  if (threadIdx.x == 0)
    partial[blockIdx.x] = ((red[0][0] + red[0][1]) + red[0][2]) + red[0][3];
}

hipError_t launch_spmv_beta(const DeviceBsr& A, const double* z, const double* p_old,
                            double* p_new, double* q, CgScalars* sc, double* partial,
                            const double* sets, int np, hipStream_t s) {
  const SellView v = sell_view(A);
  const dim3 g((unsigned)((A.n_slices + 3) / 4)), b(256);
#define FC_SELL(PP)                                                                       \
  hipLaunchKernelGGL(k_spmv_sell_beta<PP>, g, b, 0, s, v, z, p_old, p_new, q, partial, sets, \
                     np, sc)
  switch (A.lat.p) {
    case 1: FC_SELL(1); break;
    case 2: FC_SELL(2); break;
    case 3: FC_SELL(3); break;
    default: FC_SELL(4); break;
  }
#undef FC_SELL
  return hipGetLastError();
}

// Launch shape.  G lanes per block row: enough lanes that one pass of U
// blocks per lane (eight scalar blocks, two 3x3 blocks) covers the mean row,
// rounded up to 8, 16, 32 or 64 (FC_SPMV_GROUP overrides it).  Measured on
// MI355X this picks the fastest width for both FP64 workloads: 64 for the
// 3x3 rows of 32^3-cell p = 3 elasticity (about 122 blocks), 8 for the
// scalar rows of 64^3-cell p = 2 Poisson (about 63).
static int env_int(const char* name, int dflt) {
  const char* e = std::getenv(name);
  return e ? std::atoi(e) : dflt;
}

int spmv_group_for(const DeviceBsr& A) {
  const double mean = A.n_rows ? double(A.nnzb) / double(A.n_rows) : 1.0;
  const int U = A.bdim == 1 ? 8 : 2;
  const double lanes = mean / U;
  if (lanes <= 8) return 8;
  if (lanes <= 16) return 16;
  if (lanes <= 32) return 32;
  return 64;
}

static int group_width(const DeviceBsr& A) {
  static const int forced = env_int("FC_SPMV_GROUP", 0);
  if (forced == 8 || forced == 16 || forced == 32 || forced == 64) return forced;
  return A.group ? A.group : spmv_group_for(A);
}

static int64_t num_tiles(const DeviceBsr& A) {
  const int rpw = 256 / group_width(A);
  return (A.n_rows + rpw - 1) / rpw;
}

static bool lattice_allowed() {
  static const bool v = env_int("FC_SPMV_LATTICE", 1) != 0;
  return v;
}

bool spmv_has_sell(const DeviceBsr& A) {
  return lattice_allowed() && A.lat.dim > 0 && A.bdim == 1 && A.sell_val;
}

bool spmv_uses_sell(const DeviceBsr& A) {
  return spmv_has_sell(A) && !few_long_rows(A.nnzb, A.n_rows, A.n_slices);
}

bool spmv_step_joins(const DeviceBsr& A) {
  return spmv_has_sell(A) && step_joins(A.nnzb, A.max_row);
}

bool spmv_step_uses_sell(const DeviceBsr& A) {
  return spmv_step_joins(A) ? !rows_beat_join(A.nnzb, A.n_rows, A.n_slices) : spmv_uses_sell(A);
}

// Workgroups of the whole-matrix product (one (x, y) partial each when asked).
static int64_t spmv_blocks(const DeviceBsr& A, bool sell) {
  return sell ? (A.n_slices + 3) / 4 : num_tiles(A);
}

template <int B, typename T, typename XT>
static hipError_t spmv_dispatch(const DeviceBsr& A, const T* val, const XT* x,
                                double* y, hipStream_t s, const CgScalars* sc,
                                double* partial, const int32_t* rows, int64_t n_list,
                                bool sell) {
  const int G = group_width(A);
  const int64_t n_rows = rows ? n_list : A.n_rows;
  const int64_t nt = (n_rows + 256 / G - 1) / (256 / G);
  if (nt == 0) return hipSuccess;
  const bool lat = lattice_allowed() && A.lat.dim > 0;
  // the whole scalar matrix with its sliced copy
  if constexpr (B == 1 && sizeof(T) == 8 && sizeof(XT) == 8) {
    if (sell && !rows) {
      const SellView v = sell_view(A);
      dim3 g((unsigned)spmv_blocks(A, true)), b(256);
      // values streamed non-temporally (3 % faster at 64^3 cells, p = 2;
      // FC_SPMV_SELL_NT=0 reads them through the caches)
      static const bool sell_nt = env_int("FC_SPMV_SELL_NT", 1) != 0;
#define FC_SELL(PP)                                                                          \
  do {                                                                                       \
    if (sell_nt)                                                                             \
      hipLaunchKernelGGL((k_spmv_sell<PP, true>), g, b, 0, s, v, (const double*)x, y, partial, \
                         sc);                                                                \
    else                                                                                     \
      hipLaunchKernelGGL((k_spmv_sell<PP, false>), g, b, 0, s, v, (const double*)x, y,       \
                         partial, sc);                                                       \
  } while (0)
      switch (A.lat.p) {
        case 1: FC_SELL(1); break;
        case 2: FC_SELL(2); break;
        case 3: FC_SELL(3); break;
        default: FC_SELL(4); break;
      }
#undef FC_SELL
      return hipGetLastError();
    }
  }
  dim3 grid((unsigned)nt), block(256);
  // 3x3 blocks: two per lane per pass (nine values each), FP64 values
  // non-temporal; scalar rows: eight per lane per pass through the caches
  constexpr bool kNT = B != 1 && sizeof(T) == 8;
  constexpr int kU = B == 1 ? 8 : 2;
#define FC_SPMV_CASE(GG)                                                                     \
  case GG:                                                                                   \
    if (lat)                                                                                 \
      hipLaunchKernelGGL((k_spmv_bsr<B, GG, T, true, XT, kU, kNT>), grid, block, 0, s,       \
                         A.rowptr, A.col, val, x, y, n_rows, sc, partial, rows, A.lat);      \
    else                                                                                     \
      hipLaunchKernelGGL((k_spmv_bsr<B, GG, T, false, XT, kU, kNT>), grid, block, 0, s,      \
                         A.rowptr, A.col, val, x, y, n_rows, sc, partial, rows, A.lat);      \
    break;
  switch (G) {
    FC_SPMV_CASE(8)
    FC_SPMV_CASE(16)
    FC_SPMV_CASE(32)
    FC_SPMV_CASE(64)
  }
#undef FC_SPMV_CASE
  return hipGetLastError();
}

template <typename T, typename XT = double>
static hipError_t spmv_any(const DeviceBsr& A, const T* val, const XT* x, double* y,
                           hipStream_t s, const CgScalars* sc, double* partial,
                           const int32_t* rows = nullptr, int64_t n_list = 0,
                           bool sell = false) {
  switch (A.bdim) {
    case 1: return spmv_dispatch<1, T, XT>(A, val, x, y, s, sc, partial, rows, n_list, sell);
    case 2: return spmv_dispatch<2, T, XT>(A, val, x, y, s, sc, partial, rows, n_list, sell);
    case 3: return spmv_dispatch<3, T, XT>(A, val, x, y, s, sc, partial, rows, n_list, sell);
  }
  return hipErrorInvalidValue;
}

hipError_t launch_spmv(const DeviceBsr& A, const double* x, double* y, hipStream_t s) {
  return spmv_any<double>(A, A.val, x, y, s, nullptr, nullptr, nullptr, 0, spmv_uses_sell(A));
}

// Up to 1,024 workgroups the product leaves one (x, y) partial per workgroup
// (every workgroup of the next kernel sums them, four loads a thread at most);
// more, and the reduction at the end of a workgroup costs more than a pass
// over both vectors: it holds the workgroup's waves until the slowest row is
// done (11 % of the product at 32^3 cells, p = 3 elasticity).
int spmv_dot_blocks(const DeviceBsr& A, bool sell) {
  const int64_t nb = spmv_blocks(A, sell);
  return nb <= 1024 ? (int)nb : 0;
}

// Host side of the sliced copy: the slices of every class in the order of their
// first rows, then the copy on the device.
static hipError_t spmv_build_sell(DeviceBsr& A, hipStream_t s) {
  const LatticeInfo lat = A.lat;
  const int64_t n1 = lat.n1;
  const int p = lat.p, n = (lat.n1 - 1) / p;
  const int64_t nv = n - 1, nn = n1 - nv;
  struct Entry {
    int64_t first;   // line of the slice's first row
    SellSlice sl;
  };
  std::vector<Entry> list;
  auto index = [&](bool vertex, int64_t i) -> int64_t {
    if (vertex) return p * (i + 1);
    if (i == 0 || p == 1) return i == 0 ? 0 : n1 - 1;
    return std::min<int64_t>(n1 - 1, ((i - 1) / (p - 1)) * p + 1 + (i - 1) % (p - 1));
  };
  for (int cls = 0; cls < (lat.dim == 3 ? 8 : 4); ++cls) {
    const bool vy = cls & 2, vz = cls & 4;
    const int64_t cx = cls & 1 ? nv : nn, cy = vy ? nv : nn, cz = lat.dim < 3 ? 1 : vz ? nv : nn;
    for (int64_t t = 0; t < cx * cy * cz; t += 64) {
      const int64_t line = t / cx;
      const int64_t y = index(vy, line % cy), z = lat.dim == 3 ? index(vz, line / cy) : 0;
      list.push_back({z * n1 + y, {0, cls, (int32_t)(t / 64)}});
    }
  }
  std::stable_sort(list.begin(), list.end(),
                   [](const Entry& a, const Entry& b) { return a.first < b.first; });
  std::vector<SellSlice> slices;
  slices.reserve(list.size());
  int64_t off = 0;
  for (Entry& e : list) {
    e.sl.off = off;
    slices.push_back(e.sl);
    int64_t len = 64;
    for (int d = 0; d < lat.dim; ++d) len *= e.sl.cls >> d & 1 ? 2 * p + 1 : p + 1;
    off += len;
  }
  hipError_t e = dev_malloc(&A.sell_val, (size_t)off * sizeof(double));
  if (e == hipSuccess) e = dev_malloc(&A.sell_slices, slices.size() * sizeof(SellSlice));
  if (e == hipSuccess)
    e = hipMemcpyAsync(A.sell_slices, slices.data(), slices.size() * sizeof(SellSlice),
                       hipMemcpyHostToDevice, s);
  if (e == hipSuccess) {
    A.n_slices = (int64_t)slices.size();
    A.sell_nv = (int32_t)nv;
    const SellView v = sell_view(A);
    const dim3 g((unsigned)std::min<int64_t>(A.n_slices, 65536)), b(256);
    switch (p) {
      case 1: hipLaunchKernelGGL(k_sell_build<1>, g, b, 0, s, A.val, v, lat, A.sell_val); break;
      case 2: hipLaunchKernelGGL(k_sell_build<2>, g, b, 0, s, A.val, v, lat, A.sell_val); break;
      case 3: hipLaunchKernelGGL(k_sell_build<3>, g, b, 0, s, A.val, v, lat, A.sell_val); break;
      default: hipLaunchKernelGGL(k_sell_build<4>, g, b, 0, s, A.val, v, lat, A.sell_val); break;
    }
    e = hipGetLastError();
  }
  if (e == hipSuccess) e = hipStreamSynchronize(s);   // the host vector dies here
  if (e != hipSuccess) {
    for (void* q : {(void*)A.sell_val, (void*)A.sell_slices})
      if (q) (void)hipFree(q);
    A.sell_val = nullptr;
    A.sell_slices = nullptr;
    // without room for the copy the row layout serves every product
    if (e == hipErrorOutOfMemory) {
      (void)hipGetLastError();
      return hipSuccess;
    }
  }
  return e;
}

// mismatches between stored rows and lattice boxes: length, start and
// columns (counted with an atomic only where one occurs)
__global__ void k_check_lattice(const int32_t* __restrict__ rowptr, const int32_t* __restrict__ col,
                                int64_t n_rows, const LatticeInfo lat,
                                unsigned long long* __restrict__ bad) {
  for (int64_t row = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; row < n_rows;
       row += (int64_t)gridDim.x * blockDim.x) {
    const RowBox b = row_box(row, lat);
    const int64_t base = rowptr[row];
    const int L = rowptr[row + 1] - (int32_t)base;
    int miss = L != b.len[0] * b.len[1] * b.len[2] || base != lattice_row_start(row, lat);
    for (int k = 0; k < L && !miss; ++k) miss = col[base + k] != lattice_col(b, k, lat.n1);
    if (miss) atomicAdd(bad, 1ull);
  }
}

hipError_t spmv_enable_lattice(DeviceBsr& A, int dim, int n1, int p, hipStream_t s) {
  A.lat = LatticeInfo{};
  if (dim < 1 || dim > 3 || p < 1 || A.n_rows == 0) return hipSuccess;
  int64_t nodes = 1;
  for (int k = 0; k < dim; ++k) nodes *= n1;
  if (nodes != A.n_rows) return hipSuccess;
  unsigned long long* bad = nullptr;
  hipError_t e = dev_malloc(&bad, sizeof(*bad));
  if (e != hipSuccess) return e;
  unsigned long long hbad = 1;
  const LatticeInfo lat = make_lattice_info(dim, n1, p);
  e = hipMemsetAsync(bad, 0, sizeof(*bad), s);
  if (e == hipSuccess) {
    hipLaunchKernelGGL(k_check_lattice, dim3(2048), dim3(256), 0, s, A.rowptr, A.col, A.n_rows,
                       lat, bad);
    e = hipGetLastError();
  }
  if (e == hipSuccess) e = hipMemcpyAsync(&hbad, bad, sizeof(hbad), hipMemcpyDeviceToHost, s);
  if (e == hipSuccess) e = hipStreamSynchronize(s);
  (void)hipFree(bad);
  if (e == hipSuccess && hbad == 0) A.lat = lat;
  if (e == hipSuccess && A.lat.dim >= 2 && A.bdim == 1 && p <= 4 && env_int("FC_SPMV_SELL", 1))
    e = spmv_build_sell(A, s);
  return e;
}

hipError_t launch_spmv_pq(const DeviceBsr& A, const double* p, double* q, CgScalars* sc,
                          double* partial, bool sell, hipStream_t s) {
  return spmv_any<double>(A, A.val, p, q, s, sc, partial, nullptr, 0, sell);
}

hipError_t launch_spmv_mixed(const DeviceBsr& A, const double* p, const float* p32, double* q,
                             const CgScalars* sc, hipStream_t s) {
  hipError_t e = hipSuccess;
  if (A.n_hi > 0 &&
      (e = spmv_any<double>(A, A.val, p, q, s, sc, nullptr, A.rows_hi, A.n_hi)) != hipSuccess)
    return e;
  if (A.n_lo > 0)
    e = spmv_any<float, float>(A, A.val32, p32, q, s, sc, nullptr, A.rows_lo, A.n_lo);
  return e;
}

}  // namespace fc
