// Device helpers shared by the libfc kernels (gfx950, wave64).
#pragma once
#include <hip/hip_runtime.h>

#include <cstdint>

#include "fc_internal.h"

namespace fc {

constexpr int kWave = 64;
constexpr int kNumXcd = 8;   // MI355X: 8 XCDs, workgroups dispatched round-robin

// v, opaque to the compiler: what is derived from it is computed where it is
// used and not kept in registers across a loop.
__device__ __forceinline__ int opaque(int v) {
  asm volatile("" : "+v"(v));
  return v;
}

// A pointer into device memory that was itself loaded from memory.  The compiler knows
// that of kernel arguments only and takes flat loads otherwise, whose waits are those of
// LDS as well.
template <typename T>
__device__ __forceinline__ T* as_global(T* p) {
  return (T*)(__attribute__((address_space(1))) T*)(uintptr_t)p;
}

// Map the hardware workgroup id to a logical tile id so that the
// workgroups that land on one XCD (ids congruent mod 8) process one
// contiguous range of tiles and share that XCD's L2.  A bijection on
// [0, nwg) for any nwg.
__device__ __forceinline__ uint32_t xcd_remap(uint32_t bid, uint32_t nwg) {
  const uint32_t x = bid % kNumXcd, j = bid / kNumXcd;
  const uint32_t q = nwg / kNumXcd, r = nwg % kNumXcd;
  return (x < r) ? x * (q + 1) + j : r * (q + 1) + (x - r) * q + j;
}

// Contiguous tile range [t0, t1) of the XCD of workgroup bid, walked by
// that XCD's workgroups from j with stride per.  Workgroups are dealt out
// round-robin over min(nwg, kNumXcd) XCDs, so a grid with fewer workgroups
// than XCDs still covers every tile.
struct XcdRange {
  int64_t t0, t1;
  uint32_t j, per;
};

__device__ __forceinline__ XcdRange xcd_range(uint32_t bid, uint32_t nwg, int64_t ntiles) {
  const uint32_t nx = nwg < (uint32_t)kNumXcd ? nwg : (uint32_t)kNumXcd;
  const uint32_t x = bid % nx;
  XcdRange r;
  r.j = bid / nx;
  r.per = nwg / nx + (x < nwg % nx ? 1u : 0u);
  // eight XCDs (every grid of eight workgroups or more): a shift instead of
  // a 64-bit division, which costs hundreds of scalar instructions per wave
  if (nx == (uint32_t)kNumXcd) {
    r.t0 = (ntiles * x) >> 3;
    r.t1 = (ntiles * (x + 1)) >> 3;
  } else {
    r.t0 = ntiles * x / nx;
    r.t1 = ntiles * (x + 1) / nx;
  }
  return r;
}

template <int W, typename T>
__device__ __forceinline__ T group_sum(T v) {
#pragma unroll
  for (int o = W / 2; o > 0; o >>= 1) v += __shfl_xor(v, o, W);
  return v;
}

// Sum over a wave with DPP moves (row shifts within rows of 16 lanes, then
// row broadcasts): the total lands in lane 63, in a fixed order.
template <int C, int RM>
__device__ __forceinline__ double dpp64(double v) {
  const long long b = __double_as_longlong(v);
  const int lo = __builtin_amdgcn_update_dpp(0, (int)b, C, RM, 0xf, false);
  const int hi = __builtin_amdgcn_update_dpp(0, (int)(b >> 32), C, RM, 0xf, false);
  return __longlong_as_double(((long long)hi << 32) | (long long)(unsigned)lo);
}
// (over every 16 lanes: in the last of them)
__device__ __forceinline__ double row16_sum_last(double v) {
  v += dpp64<0x111, 0xf>(v);   // row_shr:1
  v += dpp64<0x112, 0xf>(v);   // row_shr:2
  v += dpp64<0x114, 0xf>(v);   // row_shr:4
  v += dpp64<0x118, 0xf>(v);   // row_shr:8
  return v;
}
__device__ __forceinline__ double wave_sum_last(double v) {
  v = row16_sum_last(v);
  v += dpp64<0x142, 0xa>(v);   // row_bcast:15 into rows 1 and 3
  v += dpp64<0x143, 0xc>(v);   // row_bcast:31 into rows 2 and 3
  return v;
}

// Deterministic sum over the workgroup (blockDim.x a multiple of 64, at
// most 1024).  Every thread receives the result.
template <typename T>
__device__ __forceinline__ T block_sum(T v, T* lds /* >= 16 */) {
  v = group_sum<kWave>(v);
  const int w = threadIdx.x / kWave, l = threadIdx.x % kWave;
  const int nw = blockDim.x / kWave;
  __syncthreads();
  if (l == 0) lds[w] = v;
  __syncthreads();
  T t = 0;
  for (int i = 0; i < nw; ++i) t += lds[i];
  __syncthreads();
  return t;
}

// Whether the run has stopped, for kernels of either place in a step (sc may be null),
// that may take alpha (first: the workgroup that stores the scalars), and that
// take beta.
__device__ __forceinline__ bool cg_stopped(const CgScalars* sc) {
  return sc && (sc->done | sc->halt);
}
__device__ __forceinline__ bool alpha_stopped(CgScalars* sc, bool takes, bool first) {
  if (!takes) return cg_stopped(sc);
  const int32_t done = sc->done;
  if (done && first && threadIdx.x == 0) sc->halt = done;
  return done;
}
__device__ __forceinline__ bool beta_stopped(CgScalars* sc, bool first) {
  const int32_t halt = sc->halt;
  if (halt && first && threadIdx.x == 0) sc->done = halt;
  return halt;
}

// Step length alpha = (r, z) / (p, q) from the (p, q) partials, by every
// workgroup on its own (a fixed order, so all agree); the first one also
// counts the step and stores the scalars.  False: breakdown, the step is not
// taken.  red: LDS of at least 16 doubles.
__device__ __forceinline__ bool cg_alpha(CgScalars* sc, const AlphaIn ai, double* red,
                                         double* alpha, bool first) {
  const double rz = sc->rzn;
  double t = 0.0;
  for (int i = threadIdx.x; i < ai.np; i += blockDim.x) t += ai.partial[i];
  t = wave_sum_last(t);
  const int w = threadIdx.x / kWave;
  if (threadIdx.x % kWave == kWave - 1) red[w] = t;
  __syncthreads();
  double pq = red[0];
  for (int i = 1; i < (int)(blockDim.x / kWave); ++i) pq += red[i];
  const bool ok = pq > 0.0 && rz > 0.0;
  *alpha = rz / pq;
  if (first && threadIdx.x == 0) {
    sc->pq = pq;
    sc->rz = rz;
    sc->iter += 1;
    if (ok) sc->alpha = *alpha;
    else sc->halt = (pq != pq || rz != rz) ? 4 : 3;
  }
  return ok;
}

// Stop test (Eq. 12 or the plain residual) and the scalars of the next step,
// by one thread.  sc->rz stays: the workgroups that update p divide by it.
__device__ __forceinline__ void cg_beta_store(CgScalars* sc, double rz, double zz, double rr) {
  const bool precond = sc->stop == FC_STOP_PRECOND;
  const double crit = sqrt(precond ? zz : rr) / (precond ? sc->zn0 : sc->rn0);
  sc->zz = zz;
  sc->rr = rr;
  sc->crit = crit;
  if (sc->history) sc->history[sc->iter] = crit;
  sc->beta = rz / sc->rz;
  sc->rzn = rz;
  if (!(crit == crit) || !(rz == rz) || isinf(rz)) {
    sc->done = 4;
  } else if (crit <= sc->tol) {
    sc->done = 1;
  } else if (sc->iter >= sc->maxit) {
    sc->done = 2;
  }
}

// (r, z) from the pull's np <= kBetaSets partial sets (value k of set j at k stride + j),
// by every workgroup of 256 in the same order.  The first one also leaves the sums of
// (z, z) and (r, r) in red: one thread of it then tests for the stop and stores the
// scalars (cg_beta_finish).
constexpr int kBetaSets = 1024;
__device__ __forceinline__ double cg_beta_sum(const double* __restrict__ sets, int64_t stride,
                                              int np, double (*red)[4], bool first) {
  const int nk = first ? 3 : 1, w = threadIdx.x / kWave;
  for (int k = 0; k < nk; ++k) {
    double v[kBetaSets / 256];
#pragma unroll
    for (int u = 0; u < kBetaSets / 256; ++u) {
      const int j = threadIdx.x + 256 * u;
      v[u] = j < np ? sets[k * stride + j] : 0.0;
    }
    const double t = wave_sum_last((v[0] + v[1]) + (v[2] + v[3]));
    if (threadIdx.x % kWave == kWave - 1) red[k][w] = t;
  }
  __syncthreads();
  return ((red[0][0] + red[0][1]) + red[0][2]) + red[0][3];
}
__device__ __forceinline__ void cg_beta_finish(CgScalars* sc, double rz, double (*red)[4]) {
  cg_beta_store(sc, rz, ((red[1][0] + red[1][1]) + red[1][2]) + red[1][3],
                ((red[2][0] + red[2][1]) + red[2][2]) + red[2][3]);
}

__device__ __forceinline__ double load_relaxed(const double* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Last-workgroup election: every workgroup calls this once after writing
// its partial results; returns true in exactly one workgroup, the last to
// arrive, which may then read every partial.  The ticket is reset for the
// next use by the winner.
__device__ __forceinline__ bool last_block(uint32_t* ticket, uint32_t nblocks,
                                           int* lds_flag) {
  __syncthreads();
  if (threadIdx.x == 0) {
    __threadfence();
    uint32_t old = __hip_atomic_fetch_add(ticket, 1u, __ATOMIC_ACQ_REL,
                                          __HIP_MEMORY_SCOPE_AGENT);
    int win = (old == nblocks - 1) ? 1 : 0;
    if (win) __hip_atomic_store(ticket, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    *lds_flag = win;
  }
  __syncthreads();
  bool win = *lds_flag != 0;
  if (win) __threadfence();
  return win;
}

// Fixed-order sum of n partials by the whole workgroup.
__device__ __forceinline__ double sum_partials(const double* part, int n,
                                               double* lds) {
  double t = 0.0;
  for (int i = threadIdx.x; i < n; i += blockDim.x) t += load_relaxed(part + i);
  return block_sum(t, lds);
}

// n / d with the multiplier of make_fastdiv
__host__ __device__ __forceinline__ uint32_t fdiv(uint32_t n, const FastDiv f) {
  const uint32_t t = (uint32_t)(((uint64_t)n * f.m) >> 32);   // v_mul_hi_u32 on the device
  return (t + ((n - t) >> f.s1)) >> f.s2;
}

// Lattice indices of row node `row` (fewer than 2^31 rows: the row
// pointers are 32-bit), first direction fastest.
__device__ __forceinline__ void lattice_coords(int64_t row, const LatticeInfo& lat, int c[3]) {
  uint32_t r = (uint32_t)row;
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    c[k] = 0;
    if (k < lat.dim) {
      const uint32_t q = fdiv(r, lat.dn1);
      c[k] = (int)(r - q * (uint32_t)lat.n1);
      r = q;
    }
  }
}

struct RowBox {
  int lo[3], len[3];
  float inv[2];   // 1 / len[0], 1 / len[1] (approximate, see lattice_col)
};

__device__ __forceinline__ RowBox row_box_at(const int c[3], const LatticeInfo& lat) {
  RowBox b;
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    b.lo[k] = 0;
    b.len[k] = 1;
    if (k < lat.dim) {
      const int g = c[k];
      const int q = (int)fdiv((uint32_t)g, lat.dp);
      if (g == q * lat.p) {
        const int lo = max(0, g - lat.p), hi = min(lat.n1 - 1, g + lat.p);
        b.lo[k] = lo;
        b.len[k] = hi - lo + 1;
      } else {
        b.lo[k] = q * lat.p;
        b.len[k] = lat.p + 1;
      }
    }
  }
  b.inv[0] = __builtin_amdgcn_rcpf((float)b.len[0]);
  b.inv[1] = __builtin_amdgcn_rcpf((float)b.len[1]);
  return b;
}

// Lattice box of row node `row`: for every direction the range of lattice
// indices of the functions whose support meets the row's support (a vertex
// index reaches one cell to each side, an interior index only its cell).
__device__ __forceinline__ RowBox row_box(int64_t row, const LatticeInfo& lat) {
  int c[3];
  lattice_coords(row, lat, c);
  return row_box_at(c, lat);
}

// Row start of a node in a matrix whose rows are the lattice nodes in order
// and hold exactly their lattice boxes (the layout the SpMV checks before it
// computes columns).  Along one direction, node g reaches len(g) nodes:
// 2p + 1 for an inner vertex index, p + 1 for a boundary vertex or any
// other index.  The box of node (x, y, z) holds len(x) len(y) len(z)
// entries, so with S(g) = sum_{j<g} len(j) and T = S(n1) the entries before
// it number S(z) T^2 + len(z) S(y) T + len(z) len(y) S(x).
__device__ __forceinline__ int64_t lattice_len(int g, const LatticeInfo& lat) {
  if (g != (int)fdiv((uint32_t)g, lat.dp) * lat.p) return lat.p + 1;
  return (g == 0 || g == lat.n1 - 1) ? lat.p + 1 : 2 * lat.p + 1;
}

__device__ __forceinline__ int64_t lattice_prefix(int g, const LatticeInfo& lat) {
  // every period of p indices holds one vertex and p - 1 other indices; the
  // boundary vertices 0 and n1 - 1 reach p fewer nodes (the last one lies
  // in a whole period only when p = 1)
  const int p = lat.p;
  const int q = (int)fdiv((uint32_t)g, lat.dp), rm = g - q * p;
  int64_t s = (int64_t)q * (2 * p + 1 + (int64_t)(p - 1) * (p + 1));
  if (q > 0) s -= p;
  if ((int64_t)q * p > lat.n1 - 1) s -= p;
  if (rm > 0) s += lattice_len(q * p, lat) + (int64_t)(rm - 1) * (p + 1);
  return s;
}

__device__ __forceinline__ int64_t lattice_row_start_at(const int c[3], const RowBox& b,
                                                        const LatticeInfo& lat) {
  const int64_t T = lattice_prefix(lat.n1, lat);
  // from the last direction down: S(c_k) T^k times the box lengths above k
  int64_t base = 0, outer = 1;
  if (lat.dim == 3) {
    base += lattice_prefix(c[2], lat) * T * T;
    outer = b.len[2];
  }
  if (lat.dim >= 2) {
    base += lattice_prefix(c[1], lat) * T * outer;
    outer *= b.len[1];
  }
  base += lattice_prefix(c[0], lat) * outer;
  return base;
}

__device__ __forceinline__ int64_t lattice_row_start(int64_t row, const LatticeInfo& lat) {
  int c[3];
  lattice_coords(row, lat, c);
  return lattice_row_start_at(c, row_box_at(c, lat), lat);
}

// column of the k-th block of the row (first direction fastest).  k < 2^12
// and the lengths are small, so floor((k + 1/2) / len) from the approximate
// reciprocal is exact: the quotient lies at least 1/(2 len) from an integer,
// far beyond the reciprocal's relative error of about 2^-22.
__device__ __forceinline__ int lattice_col(const RowBox& b, int k, int n1) {
  const int r = (int)(((float)k + 0.5f) * b.inv[0]);
  const int kx = k - r * b.len[0];
  const int kz = (int)(((float)r + 0.5f) * b.inv[1]);
  const int ky = r - kz * b.len[1];
  return (b.lo[0] + kx) + n1 * ((b.lo[1] + ky) + n1 * (b.lo[2] + kz));
}

// Where the outputs of the cells holding lattice index g along one direction
// lie in the block outputs (cells are the blocks, in order; cs and ls are the
// distances of a cell step and of a local-index step along this direction).
// A vertex index (g a multiple of p) is local 1 (right end) of the cell to its
// left, slot 0, and local 0 of the cell to its right, slot 1; any other index
// is local g % p + 1 of its cell, slot 1.  An absent slot repeats the present
// one's offset, so both can be loaded without a branch.
struct PullDir {
  int off0, off1;
  bool on0, on1;
};

__device__ __forceinline__ PullDir pull_dir(uint32_t g, const PullLattice& L, int cs, int ls) {
  const uint32_t e = fdiv(g, L.dp), rem = g - e * (uint32_t)L.p;
  PullDir d;
  d.on0 = rem == 0 && e > 0;
  d.on1 = rem != 0 || e < (uint32_t)L.n;
  const int left = ((int)e - 1) * cs + ls;
  const int own = (int)e * cs + (rem == 0 ? 0 : (int)rem + 1) * ls;
  d.off0 = d.on0 ? left : own;
  d.off1 = d.on1 ? own : left;
  return d;
}

// Block outputs holding component c of node `node`, in ascending block
// (= cell) order, zero where a cell is absent: at most eight loads, all
// independent.  Consecutive lanes take consecutive unknowns, so whether a
// second cell exists along the second and third directions is mostly the same
// for a whole wave: a wave without one skips its loads.
__device__ __forceinline__ void pull_lattice_load(const double* __restrict__ y,
                                                  const PullLattice& L, int m, int bd,
                                                  uint32_t node, int c, double v[8]) {
  const uint32_t n1 = (uint32_t)L.n1;
  const uint32_t row = fdiv(node, L.dn1), gx = node - row * n1;
  const int p1 = L.p + 1;
  const PullDir dx = pull_dir(gx, L, m, bd);
  PullDir dy{0, 0, false, true}, dz{0, 0, false, true};
  if (L.dim == 3) {
    const uint32_t gz = fdiv(row, L.dn1), gy = row - gz * n1;
    dy = pull_dir(gy, L, m * L.n, bd * p1);
    dz = pull_dir(gz, L, m * L.n * L.n, bd * p1 * p1);
  } else {
    dy = pull_dir(row, L, m * L.n, bd * p1);
  }
  const double* yc = y + c;
#pragma unroll
  for (int k = 0; k < 8; ++k) v[k] = 0.0;
  auto pair = [&](int o, bool on, double& v0, double& v1) {
    const double t0 = yc[dx.off0 + o], t1 = yc[dx.off1 + o];
    v0 = on && dx.on0 ? t0 : 0.0;
    v1 = on && dx.on1 ? t1 : 0.0;
  };
  const bool two_y = __any(dy.on0 && dy.on1), two_z = __any(dz.on0 && dz.on1);
  // a single slot: whichever of the two is present
  pair(dy.off0 + dz.off0, (!two_y || dy.on0) && (!two_z || dz.on0), v[0], v[1]);
  if (two_y) pair(dy.off1 + dz.off0, dy.on1 && (!two_z || dz.on0), v[2], v[3]);
  if (two_z) {
    pair(dy.off0 + dz.off1, (!two_y || dy.on0) && dz.on1, v[4], v[5]);
    if (two_y) pair(dy.off1 + dz.off1, dy.on1 && dz.on1, v[6], v[7]);
  }
}

// The ordered sum of pull_lattice_load's terms (adding an absent term's zero
// changes no bit: the sum starts from +0 and never becomes -0).
__device__ __forceinline__ double pull_sum8(const double v[8]) {
  double s = 0.0;
#pragma unroll
  for (int k = 0; k < 8; ++k) s += v[k];
  return s;
}

// Sum of the block outputs listed for a node in the node-to-block map (block
// order): four entries per round, their loads in flight together.
__device__ __forceinline__ double pull_mapped_sum(const double* __restrict__ y,
                                                  const int32_t* __restrict__ inv_ptr,
                                                  const int32_t* __restrict__ inv_idx,
                                                  uint32_t node, int c) {
  const int32_t lo = inv_ptr[node], hi = inv_ptr[node + 1];
  double s = 0.0;
  for (int32_t e = lo; e < hi; e += 4) {
    int32_t idx[4];
    double v[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) idx[u] = inv_idx[min(e + u, hi - 1)];
#pragma unroll
    for (int u = 0; u < 4; ++u) v[u] = y[(int64_t)idx[u] + c];
#pragma unroll
    for (int u = 0; u < 4; ++u)
      if (e + u < hi) s += v[u];
  }
  return s;
}

// Node of local function loc of cell e on a lattice whose cells are the
// blocks, in order (the inverse of pull_dir: local index 0 is a cell's
// left vertex, 1 its right vertex, 2 .. p its interior indices, tensor
// order with the first direction fastest).
__device__ __forceinline__ int64_t lattice_cell_node(const PullLattice L, int e, int loc) {
  int64_t node = 0, stride = 1;
  uint32_t ee = (uint32_t)e, ll = (uint32_t)loc;
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    if (k < L.dim) {
      const uint32_t eq = fdiv(ee, L.dn), lq = fdiv(ll, L.dp1);
      const int c = (int)(ee - eq * (uint32_t)L.n), l = (int)(ll - lq * (uint32_t)(L.p + 1));
      ee = eq;
      ll = lq;
      const int g = c * L.p + (l == 0 ? 0 : l == 1 ? L.p : l - 1);
      node += g * stride;
      stride *= L.n1;
    }
  }
  return node;
}

// Unknown of row i of a block whose node list starts at nodes[e * nn]
// (element blocks, or vertex patches whose lists are padded with -1 at the
// boundary): -1 for a padding row.
__device__ __forceinline__ int64_t block_dof(const int32_t* __restrict__ nodes, int64_t e, int nn,
                                             int bd, int i) {
  const int32_t nd = nodes[e * nn + i / bd];
  return nd < 0 ? int64_t(-1) : (int64_t)nd * bd + (i % bd);
}

__device__ __forceinline__ float bf16_to_f32(uint16_t v) {
  return __uint_as_float(((uint32_t)v) << 16);
}

}  // namespace fc
