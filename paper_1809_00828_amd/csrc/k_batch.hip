// Batched Schwarz-PCG: many independent finite cell problems of uneven size
// iterate together.  Every PCG step of the whole batch is a fixed sequence
// of launches over segmented work lists (problem, tile), one launch per
// shape class, so the launch count does not grow with the number of
// problems; each problem keeps its own CG scalars and stop flag, and the
// work items of a converged problem return at once.  A chunk of steps is
// captured into one hipGraph and replayed until every problem has stopped.
//
// The kernels are the single problem's, over tiles of many problems: sliced
// products for scalar lattice members (a class per degree), block products with
// the block size compiled in (a class per size), the pull from the lattice
// indices, and the step length and beta summed where they are used.  Members
// without a sliced copy take the row layout; for each such class (block
// dimension, mean row length) an autotuner at batch creation times the group
// widths 8/16/32/64 on the class's own work items and keeps the fastest.
// Lists of equal tiles are dealt so that one XCD walks a contiguous run.
#include <hip/hip_runtime.h>

#include <cstdio>
#include <cstdlib>

#include <algorithm>
#include <cmath>
#include <cstring>
#include <map>
#include <memory>
#include <new>
#include <numeric>
#include <sstream>
#include <string>
#include <type_traits>
#include <vector>

#include "dev_common.h"
#include "k_schwarz.h"
#include "k_spmv.h"
#include "routes.h"
#include "schwarz_dev.h"
#include "spmv_dev.h"

namespace fc {

struct BProb {
  const int32_t* rowptr;
  const int32_t* col;
  const double* val;       // row-SoA BSR
  int64_t n_rows;
  const int32_t* elem_nodes;
  const int32_t* block_elem;
  const double* Q;         // wrapped-diagonal symmetric local inverses
  const int32_t* inv_ptr;
  const int32_t* inv_idx;
  const double* fallback;
  double* y;
  const double* b;
  double* x;
  int64_t n_blocks, n_dofs, voff;
  int32_t nn, m, bdim;
  FastDiv dbd;
  SellView sell;           // n_slices = 0: row layout
  PullLattice lat;         // dim = 0: node-to-block map
  // tiles of pull_rounds x 512 and of wide_rounds x 2048 unknowns, at most
  // kPullTiles and kWideTiles of them: every workgroup of a later kernel sums
  // their partials
  int32_t pull_item0, pull_items, pull_rounds;
  int32_t wide_item0, wide_items, wide_rounds;
};

constexpr int kPullTiles = kBetaSets, kWideTiles = 256;

__device__ __forceinline__ AlphaIn batch_alpha(const BProb& P, const double* partial,
                                               int n_items) {
  return AlphaIn{partial + 3 * (int64_t)n_items + P.wide_item0, P.wide_items};
}

// One tile of one problem.  slot is the item's fixed position in the
// partial-sum array, so a compacted list of the still-running problems'
// items writes where the per-problem reductions read.
struct WorkItem {
  int32_t prob, tile, slot;
};

// One slice of one sliced problem of degree p.
struct SellItem {
  SellSlice sl;
  int32_t prob, p;
};

// ------------------------------------------------------------ kernels
template <int B, int G>
__global__ __launch_bounds__(256) void kb_spmv(const BProb* __restrict__ probs,
                                               const WorkItem* __restrict__ items,
                                               const CgScalars* __restrict__ sc,
                                               const double* __restrict__ pvec,
                                               double* __restrict__ qvec) {
  constexpr int BB = B * B;
  constexpr int RPW = 256 / G;
  constexpr int U = B == 1 ? 8 : 2;   // blocks per lane per pass
  const WorkItem it = items[blockIdx.x];
  const BProb& P = probs[it.prob];
  if (sc[it.prob].done) return;
  const int64_t row = (int64_t)it.tile * RPW + threadIdx.x / G;
  const int lane = threadIdx.x % G;
  const double* x = pvec + P.voff;
  if (row >= P.n_rows) return;
  const int64_t base = P.rowptr[row];
  const int L = P.rowptr[row + 1] - (int32_t)base;
  const double* v = P.val + base * BB;
  double acc[B];
#pragma unroll
  for (int i = 0; i < B; ++i) acc[i] = 0.0;
  for (int k = lane; k < L; k += U * G) {
    int c[U];
    double a[U][BB];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int ku = k + u * G;
      const bool on = ku < L;
      // scalar rows read through the caches (5 % faster on a 64-member
      // batch), 3x3 blocks non-temporally
      if constexpr (B == 1)
        c[u] = on ? P.col[base + ku] : -1;
      else
        c[u] = on ? __builtin_nontemporal_load(P.col + base + ku) : -1;
#pragma unroll
      for (int e = 0; e < BB; ++e)
        if constexpr (B == 1)
          a[u][e] = on ? v[(int64_t)e * L + ku] : 0.0;
        else
          a[u][e] = on ? __builtin_nontemporal_load(v + (int64_t)e * L + ku) : 0.0;
    }
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
      for (int i = 0; i < B; ++i)
#pragma unroll
        for (int j = 0; j < B; ++j)
          acc[i] = fma(a[u][i * B + j], c[u] >= 0 ? x[(int64_t)c[u] * B + j] : 0.0, acc[i]);
  }
#pragma unroll
  for (int i = 0; i < B; ++i) acc[i] = group_sum<G>(acc[i]);
  if (lane == 0) {
#pragma unroll
    for (int i = 0; i < B; ++i) qvec[P.voff + row * B + i] = acc[i];
  }
}

// The sliced product, one slice per wave, all degrees in one launch, the slice's
// place in its item rather than behind it, and no contiguous run per XCD (the
// members' rows differ in length, and an XCD with the long ones works alone).
// 16 members of 50k - 200k unknowns (0.58 GB): 112 us, 5.2 TB/s; a launch per
// degree, slices found through their problem 203 us; with runs per XCD 225 us;
// the row layout 290 us.
__global__ __launch_bounds__(256) void kb_spmv_sell(const BProb* __restrict__ probs,
                                                    const SellItem* __restrict__ items,
                                                    int n_items, const CgScalars* __restrict__ sc,
                                                    const double* __restrict__ pvec,
                                                    double* __restrict__ qvec) {
  const int l = threadIdx.x % 64, w = __builtin_amdgcn_readfirstlane(threadIdx.x / 64);
  const int64_t s = (int64_t)blockIdx.x * 4 + w;
  if (s >= n_items) return;
  const SellItem it = items[s];
  const BProb& B = probs[it.prob];
  if (sc[it.prob].done) return;
  const GatherX x{pvec + B.voff};
  double* y = qvec + B.voff;
  switch (it.p) {
    case 1: (void)sell_slice_product<1, true>(B.sell, it.sl, l, x, y); break;
    case 2: (void)sell_slice_product<2, true>(B.sell, it.sl, l, x, y); break;
    case 3: (void)sell_slice_product<3, true>(B.sell, it.sl, l, x, y); break;
    default: (void)sell_slice_product<4, true>(B.sell, it.sl, l, x, y); break;
  }
}

// (p, q) per wide tile into partial[3 n_items + slot].  In the SpMV it would
// hold a workgroup's waves until the slowest row finishes.
__global__ __launch_bounds__(256) void kb_pq(const BProb* __restrict__ probs,
                                             const WorkItem* __restrict__ items, int n_items,
                                             const CgScalars* __restrict__ sc,
                                             const double* __restrict__ pvec,
                                             const double* __restrict__ qvec,
                                             double* __restrict__ partial) {
  __shared__ double lds[16];
  const WorkItem it = items[xcd_remap(blockIdx.x, gridDim.x)];
  if (sc[it.prob].done) return;
  const BProb& P = probs[it.prob];
  const double *p = pvec + P.voff, *q = qvec + P.voff;
  double a[4] = {0.0, 0.0, 0.0, 0.0};
  for (int t = 0; t < P.wide_rounds; ++t) {
    const int64_t i0 = ((int64_t)it.tile * P.wide_rounds + t) * 2048 + threadIdx.x;
    double pv[8], qv[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const int64_t i = i0 + 256 * u;
      pv[u] = i < P.n_dofs ? p[i] : 0.0;
      qv[u] = i < P.n_dofs ? q[i] : 0.0;
    }
#pragma unroll
    for (int u = 0; u < 8; ++u) a[u & 3] = fma(pv[u], qv[u], a[u & 3]);
  }
  const double t = block_sum((a[0] + a[1]) + (a[2] + a[3]), lds);
  if (threadIdx.x == 0) partial[3 * (int64_t)n_items + it.slot] = t;
}

// Schwarz phase 1 on r - alpha q (q null for the start), blocks of up to 64
// rows: the workgroup of a member's first tile stores the step length.  kM: one
// block size per launch, compiled in (0: any); kMixed: every size up to 27 that
// has a kernel of its own in one launch, since each of them fills the chip for
// a few microseconds only (56 us for the 0.23 GB of 16 members' blocks of 9 to
// 27 rows, 71 us with a launch per size; the larger ones would cost it the
// waves in flight: 80 registers at m = 27, 180 at m = 64).
constexpr int kMixed = -1;
#define FC_MIXED_SIZES(X) X(8) X(9) X(16) X(18) X(24) X(25) X(27)

template <int kM, bool kLat>
__device__ __forceinline__ void batch_small(const BProb& P, const WorkItem it, int n_items,
                                            CgScalars* S, const double* rvec, const double* qvec,
                                            const double* partial, double (*rB)[64],
                                            double* red) {
  schwarz_small_tile<double, kM, kLat>(
      as_global(P.Q), sym_block_stride_dev(P.m), P.m, rvec + P.voff,
      qvec ? qvec + P.voff : nullptr, nullptr, S,
      qvec ? batch_alpha(P, partial, n_items) : AlphaIn{}, it.tile == 0, as_global(P.y),
      P.n_blocks, P.lat, it.tile, rB, red, [&](int64_t blk, int i) {
        return block_dof(as_global(P.elem_nodes), as_global(P.block_elem)[blk], P.nn, P.bdim, i);
      });
}

template <int kM, bool kLat>
__global__ __launch_bounds__(256) void kb_schwarz_small(
    const BProb* __restrict__ probs, const WorkItem* __restrict__ items, int n_items,
    CgScalars* __restrict__ sc, const double* __restrict__ rvec, const double* __restrict__ qvec,
    const double* __restrict__ partial) {
  __shared__ double rB[4][64], red[16];
  const WorkItem it = items[kM == kMixed ? blockIdx.x
                                         : xcd_remap(blockIdx.x, gridDim.x)];
  CgScalars* S = sc + it.prob;
  if (alpha_stopped(S, qvec != nullptr, it.tile == 0)) return;
  const BProb& P = probs[it.prob];
  if constexpr (kM != kMixed) {
    batch_small<kM, kLat>(P, it, n_items, S, rvec, qvec, partial, rB, red);
  } else {
#define FC_MIXED(KM) \
  case KM: batch_small<KM, kLat>(P, it, n_items, S, rvec, qvec, partial, rB, red); break;
    switch (P.m) { FC_MIXED_SIZES(FC_MIXED) }
#undef FC_MIXED
  }
}

// Blocks of more than 64 rows, one per workgroup.
template <int kRows, int kMaxM>
__global__ __launch_bounds__(256) void kb_schwarz_staged(
    const BProb* __restrict__ probs, const WorkItem* __restrict__ items, int n_items,
    CgScalars* __restrict__ sc, const double* __restrict__ rvec, const double* __restrict__ qvec,
    const double* __restrict__ partial) {
  __shared__ double rB[kMaxM], red[16];
  __shared__ __align__(16) double tile[kRows * kMaxM];
  const WorkItem it = items[xcd_remap(blockIdx.x, gridDim.x)];
  CgScalars* S = sc + it.prob;
  if (alpha_stopped(S, qvec != nullptr, it.tile == 0)) return;
  const BProb& P = probs[it.prob];
  const AlphaIn ai = qvec ? batch_alpha(P, partial, n_items) : AlphaIn{};
  const int64_t blk = it.tile;
  schwarz_staged_block<double, kRows>(
      as_global(P.Q) + blk * sym_block_stride_dev(P.m), as_global(P.y) + blk * P.m, P.m,
      rvec + P.voff,
      qvec ? qvec + P.voff : nullptr, nullptr, S, ai, it.tile == 0, rB, tile, red,
      [&](int i) {
        return block_dof(as_global(P.elem_nodes), as_global(P.block_elem)[blk], P.nn, P.bdim, i);
      });
}

// Pull + x, r updates + partial dots (mode 1), or the start (mode 0: z = S r,
// p = z and the dots of r and z).  Two unknowns per thread and round, whose
// loads are all issued before the first is used.
template <int kMode>
__global__ __launch_bounds__(256) void kb_pull(const BProb* __restrict__ probs,
                                               const WorkItem* __restrict__ items, int n_items,
                                               const CgScalars* __restrict__ sc,
                                               double* __restrict__ rvec,
                                               double* __restrict__ pvec,
                                               const double* __restrict__ qvec,
                                               double* __restrict__ zvec,
                                               double* __restrict__ partial) {
  __shared__ double lds[4][3];
  const WorkItem it = items[xcd_remap(blockIdx.x, gridDim.x)];
  const CgScalars& S = sc[it.prob];
  if (S.halt) return;
  const BProb& P = probs[it.prob];
  const double alpha = kMode == 1 ? S.alpha : 0.0;
  const uint32_t n = (uint32_t)P.n_dofs;
  double* r = rvec + P.voff;
  double* p = pvec + P.voff;
  double* z = zvec + P.voff;
  const double* q = qvec + P.voff;
  double acc[3] = {0.0, 0.0, 0.0};
  for (int t = 0; t < P.pull_rounds; ++t) {
    const uint32_t i0 = ((uint32_t)it.tile * P.pull_rounds + t) * 512 + threadIdx.x;
    if (i0 >= n) break;
    uint32_t i[2];
    double qi[2], ri[2], pi[2], xi[2], fi[2], v[2][8], s[2];
#pragma unroll
    for (int e = 0; e < 2; ++e) {
      i[e] = min(i0 + 256u * e, n - 1);
      ri[e] = r[i[e]];
      if constexpr (kMode == 1) {
        qi[e] = q[i[e]];
        pi[e] = p[i[e]];
        xi[e] = P.x[i[e]];
      }
      fi[e] = P.fallback ? P.fallback[i[e]] : 0.0;
    }
    uint32_t node[2];
    int c[2];
#pragma unroll
    for (int e = 0; e < 2; ++e) {
      node[e] = fdiv(i[e], P.dbd);
      c[e] = (int)(i[e] - node[e] * (uint32_t)P.bdim);
    }
    if (P.lat.dim > 0) {
#pragma unroll
      for (int e = 0; e < 2; ++e) pull_lattice_load(P.y, P.lat, P.m, P.bdim, node[e], c[e], v[e]);
#pragma unroll
      for (int e = 0; e < 2; ++e) s[e] = pull_sum8(v[e]);
    } else {
#pragma unroll
      for (int e = 0; e < 2; ++e) s[e] = pull_mapped_sum(P.y, P.inv_ptr, P.inv_idx, node[e], c[e]);
    }
#pragma unroll
    for (int e = 0; e < 2; ++e) {
      if (i0 + 256u * e >= n) break;
      double rn = ri[e];
      if constexpr (kMode == 1) {
        rn = fma(-alpha, qi[e], rn);
        P.x[i[e]] = fma(alpha, pi[e], xi[e]);
        r[i[e]] = rn;
      }
      const double zn = P.fallback ? fma(fi[e], rn, s[e]) : s[e];
      z[i[e]] = zn;
      if constexpr (kMode == 0) p[i[e]] = zn;
      acc[0] = fma(rn, zn, acc[0]);
      acc[1] = fma(zn, zn, acc[1]);
      acc[2] = fma(rn, rn, acc[2]);
    }
  }
  const int w = threadIdx.x / kWave;
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    acc[k] = wave_sum_last(acc[k]);
    if (threadIdx.x % kWave == kWave - 1) lds[w][k] = acc[k];
  }
  __syncthreads();
  if (threadIdx.x < 3) {
    const int k = threadIdx.x;
    partial[k * (int64_t)n_items + it.slot] = ((lds[0][k] + lds[1][k]) + lds[2][k]) + lds[3][k];
  }
}

// Scalars of the start, one workgroup per problem.
__global__ __launch_bounds__(256) void kb_start(const BProb* __restrict__ probs, CgScalars* sc,
                                                const double* __restrict__ partial, int n_items) {
  __shared__ double lds[16];
  CgScalars& S = sc[blockIdx.x];
  const BProb& P = probs[blockIdx.x];
  double t[3] = {0.0, 0.0, 0.0};
  for (int i = threadIdx.x; i < P.pull_items; i += blockDim.x)
#pragma unroll
    for (int k = 0; k < 3; ++k) t[k] += partial[k * (int64_t)n_items + P.pull_item0 + i];
  const double rz = block_sum(t[0], lds);
  const double zz = block_sum(t[1], lds);
  const double rr = block_sum(t[2], lds);
  if (threadIdx.x != 0) return;
  S.rz = rz;
  S.rzn = rz;
  S.zz = zz;
  S.rr = rr;
  S.iter = 0;
  S.zn0 = sqrt(zz);
  S.rn0 = sqrt(rr);
  const double c0 = S.stop == FC_STOP_PRECOND ? S.zn0 : S.rn0;
  S.crit = c0 > 0 ? 1.0 : 0.0;
  S.done = !(c0 == c0) ? 4 : (c0 == 0.0 ? 1 : 0);
}

// p = z + beta p with beta from the pull's partials, summed by every workgroup
// of a problem in the same order; its first one also tests for the stop and
// stores the scalars (one that still updates p after that changes nothing: p is
// not read again).
__global__ __launch_bounds__(256) void kb_beta_p(const BProb* __restrict__ probs,
                                                 const WorkItem* __restrict__ items, int n_items,
                                                 CgScalars* sc, const double* __restrict__ partial,
                                                 const double* __restrict__ zvec,
                                                 double* __restrict__ pvec) {
  __shared__ double red[3][4];
  const WorkItem it = items[xcd_remap(blockIdx.x, gridDim.x)];
  CgScalars* S = sc + it.prob;
  if (beta_stopped(S, it.tile == 0)) return;
  const BProb& P = probs[it.prob];
  const double rz_old = S->rz;
  const double* z = zvec + P.voff;
  double* p = pvec + P.voff;
  const int64_t i0 = (int64_t)it.tile * P.wide_rounds * 2048 + threadIdx.x;
  double zv[8], pv[8];
  auto load = [&](int64_t j0) {
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const int64_t i = j0 + 256 * u;
      zv[u] = i < P.n_dofs ? z[i] : 0.0;
      pv[u] = i < P.n_dofs ? p[i] : 0.0;
    }
  };
  load(i0);   // the first round's unknowns, before the sums
  const double rz = cg_beta_sum(partial + P.pull_item0, n_items, P.pull_items, red, it.tile == 0);
  const double beta = rz / rz_old;
  for (int t = 0; t < P.wide_rounds; ++t) {
    const int64_t j0 = i0 + 2048 * (int64_t)t;
    if (t > 0) load(j0);
#pragma unroll
    for (int u = 0; u < 8; ++u)
      if (j0 + 256 * u < P.n_dofs) p[j0 + 256 * u] = fma(beta, pv[u], zv[u]);
  }
  if (it.tile == 0 && threadIdx.x == 0) cg_beta_finish(S, rz, red);
}

// r = b, x = 0
__global__ __launch_bounds__(256) void kb_init(const BProb* __restrict__ probs,
                                               const WorkItem* __restrict__ items,
                                               double* __restrict__ rvec) {
  const WorkItem it = items[blockIdx.x];
  const BProb& P = probs[it.prob];
  const int64_t per = (int64_t)P.wide_rounds * 2048;
  const int64_t end = min(P.n_dofs, ((int64_t)it.tile + 1) * per);
  for (int64_t i = (int64_t)it.tile * per + threadIdx.x; i < end; i += 256) {
    rvec[P.voff + i] = P.b[i];
    P.x[i] = 0.0;
  }
}

// ---------------------------------------------------------- host side
// items: every tile of every problem of the class; act / d_act: the tiles
// of the problems still running, which the captured iteration launches.
struct SpmvClass {
  int B, G;
  std::vector<WorkItem> items;
  WorkItem* d_items = nullptr;
  int n_act = 0;
  WorkItem* d_act = nullptr;
};

struct SchwarzClass {
  int m;       // kMixed: several
  bool lat;    // gather from the lattice indices
  std::vector<WorkItem> items;
  WorkItem* d_items = nullptr;
  int n_act = 0;
  WorkItem* d_act = nullptr;
};

}  // namespace fc

struct fc_batch_s {
  int32_t nprob = 0;
  int64_t total_dofs = 0;
  std::vector<fc_precond> pcs;
  std::vector<fc::BProb> host;
  fc::BProb* d_probs = nullptr;
  std::vector<fc::SpmvClass> spmv;
  std::vector<fc::SellItem> sell;     // slices of the sliced members
  int n_act_sell = 0;
  fc::SellItem* d_act_sell = nullptr;
  std::vector<fc::SchwarzClass> schw;
  std::vector<fc::WorkItem> pull_items;
  fc::WorkItem* d_pull = nullptr;
  int n_act_pull = 0;                 // compacted pull items (see SpmvClass)
  fc::WorkItem* d_act_pull = nullptr;
  std::vector<fc::WorkItem> wide_items;
  fc::WorkItem* d_wide = nullptr;
  int n_act_wide = 0;
  fc::WorkItem* d_act_wide = nullptr;
  int64_t act_dofs = 0;               // unknowns of the problems in the lists
  double *r = nullptr, *z = nullptr, *p = nullptr, *q = nullptr, *partial = nullptr;
  fc::CgScalars* sc = nullptr;
  fc::CgScalars* host_sc = nullptr;
  hipStream_t stream = nullptr;
  hipEvent_t ev[4] = {nullptr, nullptr, nullptr, nullptr};
  hipGraphExec_t exec = nullptr;
  hipGraph_t graph = nullptr;
  std::vector<const double*> key_b;
  std::vector<double*> key_x;
  int key_chunk = 0;
  std::string report;
};

namespace fc {

static void destroy_batch(fc_batch_s* b) {
  if (!b) return;
  if (b->exec) (void)hipGraphExecDestroy(b->exec);
  if (b->graph) (void)hipGraphDestroy(b->graph);
  for (auto& c : b->spmv)
    for (void* p : {(void*)c.d_items, (void*)c.d_act}) if (p) (void)hipFree(p);
  for (auto& c : b->schw)
    for (void* p : {(void*)c.d_items, (void*)c.d_act}) if (p) (void)hipFree(p);
  for (void* p : {(void*)b->d_probs, (void*)b->d_pull, (void*)b->d_act_pull,
                  (void*)b->d_wide, (void*)b->d_act_wide, (void*)b->d_act_sell, (void*)b->r, (void*)b->z, (void*)b->p, (void*)b->q,
                  (void*)b->partial, (void*)b->sc})
    if (p) (void)hipFree(p);
  if (b->host_sc) (void)hipHostFree(b->host_sc);
  for (auto& e : b->ev) if (e) (void)hipEventDestroy(e);
  if (b->stream) (void)hipStreamDestroy(b->stream);
  delete b;
}

template <int B>
static void launch_bspmv_G(int G, dim3 g, hipStream_t s, const BProb* probs, const WorkItem* it,
                           const CgScalars* sc, const double* p, double* q) {
  switch (G) {
    case 8: hipLaunchKernelGGL((kb_spmv<B, 8>), g, dim3(256), 0, s, probs, it, sc, p, q); break;
    case 16: hipLaunchKernelGGL((kb_spmv<B, 16>), g, dim3(256), 0, s, probs, it, sc, p, q); break;
    case 32: hipLaunchKernelGGL((kb_spmv<B, 32>), g, dim3(256), 0, s, probs, it, sc, p, q); break;
    default: hipLaunchKernelGGL((kb_spmv<B, 64>), g, dim3(256), 0, s, probs, it, sc, p, q); break;
  }
}

static hipError_t launch_spmv_class(fc_batch_s& bt, const SpmvClass& c, const WorkItem* items,
                                    int n, hipStream_t s) {
  if (n == 0) return hipSuccess;
  dim3 g((unsigned)n);
  switch (c.B) {
    case 1: launch_bspmv_G<1>(c.G, g, s, bt.d_probs, items, bt.sc, bt.p, bt.q); break;
    case 2: launch_bspmv_G<2>(c.G, g, s, bt.d_probs, items, bt.sc, bt.p, bt.q); break;
    case 3: launch_bspmv_G<3>(c.G, g, s, bt.d_probs, items, bt.sc, bt.p, bt.q); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

// q null: the start
static hipError_t launch_schwarz_class(fc_batch_s& bt, const SchwarzClass& c, const WorkItem* items,
                                       int n, const double* q, hipStream_t s) {
  if (n == 0) return hipSuccess;
  const int np = (int)bt.pull_items.size();
  dim3 g((unsigned)n), b(c.m > 64 ? 64 * ((c.m + 63) / 64) : 256);
  if (c.m > 64) {
    if (c.m <= 128 && staged_rows(true, 128, n) == 16)
      hipLaunchKernelGGL((kb_schwarz_staged<16, 128>), g, b, 0, s, bt.d_probs, items, np, bt.sc,
                         bt.r, q, bt.partial);
    else if (c.m <= 128)
      hipLaunchKernelGGL((kb_schwarz_staged<4, 128>), g, b, 0, s, bt.d_probs, items, np, bt.sc,
                         bt.r, q, bt.partial);
    else
      hipLaunchKernelGGL((kb_schwarz_staged<8, 192>), g, b, 0, s, bt.d_probs, items, np, bt.sc,
                         bt.r, q, bt.partial);
    return hipGetLastError();
  }
#define FC_BSMALL(KM)                                                                         \
  case KM:                                                                                    \
    if (c.lat)                                                                                \
      hipLaunchKernelGGL((kb_schwarz_small<KM, true>), g, b, 0, s, bt.d_probs, items, np,     \
                         bt.sc, bt.r, q, bt.partial);                                         \
    else                                                                                      \
      hipLaunchKernelGGL((kb_schwarz_small<KM, false>), g, b, 0, s, bt.d_probs, items, np,    \
                         bt.sc, bt.r, q, bt.partial);                                         \
    break;
  switch (c.m) {
    FC_BSMALL(kMixed) FC_BSMALL(32) FC_BSMALL(36) FC_BSMALL(49) FC_BSMALL(50) FC_BSMALL(64)
    default:
      hipLaunchKernelGGL((kb_schwarz_small<0, false>), g, b, 0, s, bt.d_probs, items, np, bt.sc,
                         bt.r, q, bt.partial);
  }
#undef FC_BSMALL
  return hipGetLastError();
}

// The steps launch the compacted lists: tiles of the problems still running.
static hipError_t enqueue_batch_steps(fc_batch_s& bt, int chunk, hipStream_t s) {
  const int np = (int)bt.pull_items.size();
  if (bt.n_act_pull == 0) return hipSuccess;
  for (int it = 0; it < chunk; ++it) {
    if (bt.n_act_sell > 0)
      hipLaunchKernelGGL(kb_spmv_sell, dim3((bt.n_act_sell + 3) / 4), dim3(256), 0, s, bt.d_probs,
                         bt.d_act_sell, bt.n_act_sell, bt.sc, bt.p, bt.q);
    for (auto& c : bt.spmv) {
      hipError_t e = launch_spmv_class(bt, c, c.d_act, c.n_act, s);
      if (e != hipSuccess) return e;
    }
    hipLaunchKernelGGL(kb_pq, dim3(bt.n_act_wide), dim3(256), 0, s, bt.d_probs, bt.d_act_wide, np,
                       bt.sc, bt.p, bt.q, bt.partial);
    for (auto& c : bt.schw) {
      hipError_t e = launch_schwarz_class(bt, c, c.d_act, c.n_act, bt.q, s);
      if (e != hipSuccess) return e;
    }
    hipLaunchKernelGGL(kb_pull<1>, dim3(bt.n_act_pull), dim3(256), 0, s, bt.d_probs, bt.d_act_pull,
                       np, bt.sc, bt.r, bt.p, bt.q, bt.z, bt.partial);
    hipLaunchKernelGGL(kb_beta_p, dim3(bt.n_act_wide), dim3(256), 0, s, bt.d_probs, bt.d_act_wide,
                       np, bt.sc, bt.partial, bt.z, bt.p);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

// Time `reps` launches of fn on stream s (ms per launch).
template <class F>
static float time_launches(hipStream_t s, hipEvent_t e0, hipEvent_t e1, int reps, F&& fn) {
  fn();
  (void)hipEventRecord(e0, s);
  for (int i = 0; i < reps; ++i) fn();
  (void)hipEventRecord(e1, s);
  (void)hipEventSynchronize(e1);
  float ms = 0.f;
  (void)hipEventElapsedTime(&ms, e0, e1);
  return ms / reps;
}

}  // namespace fc

using namespace fc;

#define FC_TRY_B(x)                 \
  do {                              \
    fc_status s_ = (x);             \
    if (s_ != FC_OK) return s_;     \
  } while (0)

static fc_status batch_create_body(int32_t nprob, const fc_problem* problems,
                                   const fc_precond* preconds, int32_t autotune, void* stream,
                                   fc_batch* out) {
  if (nprob <= 0 || !problems || !preconds || !out) {
    set_error("fc_batch_create: invalid arguments");
    return FC_E_ARG;
  }
  *out = nullptr;
  std::unique_ptr<fc_batch_s, void (*)(fc_batch_s*)> bt(new fc_batch_s(), destroy_batch);
  fc_batch_s& B = *bt;
  B.nprob = nprob;
  hipStream_t user = (hipStream_t)stream;
  FC_HIP(hipStreamCreateWithFlags(&B.stream, hipStreamNonBlocking));
  for (auto& e : B.ev) FC_HIP(hipEventCreate(&e));
  hipStream_t s = B.stream;
  B.host.resize(nprob);
  B.pcs.assign(preconds, preconds + nprob);
  int64_t voff = 0;
  // shape classes
  std::map<std::pair<int, int>, int> spmv_key;   // (B, row-length bucket) -> class
  std::map<std::pair<int, bool>, int> schw_key;  // (m, lattice gather) -> class
  std::vector<int> spmv_cls(nprob, -1), schw_cls(nprob);
  for (int k = 0; k < nprob; ++k) {
    fc_problem pb = problems[k];
    fc_precond pc = preconds[k];
    if (!pb || !pc || pc->pb != pb) {
      set_error("fc_batch_create: problem/preconditioner mismatch");
      return FC_E_ARG;
    }
    if (!pc->Q) {
      set_error("fc_batch_create: preconditioner without symmetric copy");
      return FC_E_ARG;
    }
    if (pc->bnodes) {
      set_error("fc_batch_create: vertex-patch preconditioners are not batched");
      return FC_E_UNSUPPORTED;
    }
    BProb& P = B.host[k];
    P = BProb{};
    P.rowptr = pb->A.rowptr;
    P.col = pb->A.col;
    P.val = pb->A.val;
    P.n_rows = pb->A.n_rows;
    P.elem_nodes = pb->elem_nodes;
    P.block_elem = pc->block_elem;
    P.Q = pc->Q;
    P.inv_ptr = pc->inv_ptr;
    P.inv_idx = pc->inv_idx;
    P.fallback = pc->n_fallback ? pc->fallback : nullptr;
    P.y = pc->y;
    P.n_blocks = pc->n_blocks;
    P.n_dofs = pb->n_dofs;
    P.voff = voff;
    P.nn = pc->nn;
    P.m = pc->m;
    P.bdim = pb->bdim;
    P.dbd = make_fastdiv((uint32_t)pb->bdim);
    if (spmv_has_sell(pb->A)) P.sell = sell_view(pb->A);
    P.lat = pc->lat;
    voff += pb->n_dofs;
    if (P.sell.n_slices == 0) {
      const double mean = pb->A.n_rows ? double(pb->A.nnzb) / double(pb->A.n_rows) : 1.0;
      const int bucket = mean < 12 ? 0 : mean < 24 ? 1 : mean < 48 ? 2 : mean < 96 ? 3 : 4;
      const auto sk = std::make_pair((int)pb->bdim, bucket);
      if (!spmv_key.count(sk)) {
        spmv_key[sk] = (int)B.spmv.size();
        SpmvClass c;
        c.B = pb->bdim;
        c.G = bucket == 0 ? 8 : bucket == 1 ? 16 : bucket == 2 ? 32 : 64;
        B.spmv.push_back(c);
      }
      spmv_cls[k] = spmv_key[sk];
    }
    int size = P.m;
#define FC_MIXED(KM) \
  case KM: size = kMixed; break;
    switch (P.m) { FC_MIXED_SIZES(FC_MIXED) }
#undef FC_MIXED
    const auto hk = std::make_pair(size, P.m <= 64 && pc->lat.dim > 0 && pb->bdim == 1);
    if (!schw_key.count(hk)) {
      schw_key[hk] = (int)B.schw.size();
      SchwarzClass c;
      c.m = hk.first;
      c.lat = hk.second;
      B.schw.push_back(c);
    }
    schw_cls[k] = schw_key[hk];
  }
  B.total_dofs = voff;
  // items (SpMV tiles depend on G, rebuilt after tuning)
  auto build_spmv_items = [&](SpmvClass& c, int cls) {
    c.items.clear();
    const int rpw = 256 / c.G;
    for (int k = 0; k < nprob; ++k) {
      if (spmv_cls[k] != cls) continue;
      const int64_t nt = (B.host[k].n_rows + rpw - 1) / rpw;
      for (int64_t t = 0; t < nt; ++t) c.items.push_back({k, (int32_t)t, 0});
    }
  };
  // the members with the longest rows and the largest blocks first: the short
  // ones fill the end of a launch
  std::vector<int> order(nprob);
  std::iota(order.begin(), order.end(), 0);
  auto row_length = [&](int k) {
    return double(problems[k]->A.nnzb) / double(std::max<int64_t>(1, problems[k]->A.n_rows));
  };
  std::stable_sort(order.begin(), order.end(),
                   [&](int a, int b) { return row_length(a) > row_length(b); });
  for (int k : order) {
    const SellView& v = B.host[k].sell;
    if (v.n_slices == 0) continue;
    std::vector<SellSlice> sl(v.n_slices);
    FC_HIP(hipMemcpyAsync(sl.data(), v.slices, sl.size() * sizeof(SellSlice),
                          hipMemcpyDeviceToHost, s));
    FC_HIP(hipStreamSynchronize(s));
    for (const SellSlice& x : sl) B.sell.push_back({x, k, problems[k]->A.lat.p});
  }
  for (size_t c = 0; c < B.spmv.size(); ++c) build_spmv_items(B.spmv[c], (int)c);
  for (size_t ci = 0; ci < B.schw.size(); ++ci) {
    SchwarzClass& c = B.schw[ci];
    for (int k : order) {
      if (schw_cls[k] != (int)ci) continue;
      const int m = B.host[k].m;
      const int64_t per = m <= 64 ? 4 * (64 / m) : 1;
      const int64_t nt = (B.host[k].n_blocks + per - 1) / per;   // at least one: Q is there
      for (int64_t t = 0; t < nt; ++t) c.items.push_back({k, (int32_t)t, 0});
    }
  }
  for (int k = 0; k < nprob; ++k) {
    BProb& P = B.host[k];
    auto tiles = [&](int64_t unit, int most, int32_t* rounds, int32_t* first, int32_t* count,
                     std::vector<WorkItem>& v) {
      const int64_t units = (P.n_dofs + unit - 1) / unit;
      *rounds = (int32_t)std::max<int64_t>(1, (units + most - 1) / most);
      *count = (int32_t)((units + *rounds - 1) / *rounds);
      *first = (int32_t)v.size();
      for (int32_t t = 0; t < *count; ++t) v.push_back({k, t, (int32_t)v.size()});
    };
    tiles(512, kPullTiles, &P.pull_rounds, &P.pull_item0, &P.pull_items, B.pull_items);
    tiles(2048, kWideTiles, &P.wide_rounds, &P.wide_item0, &P.wide_items, B.wide_items);
  }
  auto upload_items = [&](std::vector<WorkItem>& v, WorkItem** d) -> fc_status {
    if (*d) {
      FC_HIP(hipFree(*d));
      *d = nullptr;
    }
    if (v.empty()) return FC_OK;
    FC_HIP(dev_malloc(d, v.size() * sizeof(WorkItem)));
    FC_HIP(hipMemcpyAsync(*d, v.data(), v.size() * sizeof(WorkItem), hipMemcpyHostToDevice, s));
    FC_HIP(hipStreamSynchronize(s));
    return FC_OK;
  };
  for (auto& c : B.spmv) FC_TRY_B(upload_items(c.items, &c.d_items));
  for (auto& c : B.schw) FC_TRY_B(upload_items(c.items, &c.d_items));
  FC_TRY_B(upload_items(B.pull_items, &B.d_pull));
  FC_TRY_B(upload_items(B.wide_items, &B.d_wide));
  const int64_t n = B.total_dofs;
  FC_HIP(dev_malloc(&B.r, n * sizeof(double)));
  FC_HIP(dev_malloc(&B.z, n * sizeof(double)));
  FC_HIP(dev_malloc(&B.p, n * sizeof(double)));
  FC_HIP(dev_malloc(&B.q, n * sizeof(double)));
  // three per pull tile, then (p, q) per wide tile
  const int64_t plen = 3 * (int64_t)B.pull_items.size() + (int64_t)B.wide_items.size();
  FC_HIP(dev_malloc(&B.partial, std::max<int64_t>(plen, 1) * sizeof(double)));
  FC_HIP(dev_malloc(&B.sc, nprob * sizeof(CgScalars)));
  FC_HIP(hipMemsetAsync(B.sc, 0, nprob * sizeof(CgScalars), s));
  FC_HIP(hipHostMalloc(&B.host_sc, nprob * sizeof(CgScalars), hipHostMallocDefault));
  FC_HIP(dev_malloc(&B.d_probs, nprob * sizeof(BProb)));
  FC_HIP(hipMemcpyAsync(B.d_probs, B.host.data(), nprob * sizeof(BProb), hipMemcpyHostToDevice, s));
  FC_HIP(hipStreamSynchronize(s));
  FC_HIP(hipEventRecord(B.ev[0], user));
  FC_HIP(hipStreamWaitEvent(s, B.ev[0], 0));

  std::ostringstream rep;
  if (autotune) {
    // all problems active (done = 0) on random-free data: p = q = r = 0 is
    // enough to time memory traffic of the real matrices and blocks
    FC_HIP(hipMemsetAsync(B.p, 0, n * sizeof(double), s));
    FC_HIP(hipMemsetAsync(B.r, 0, n * sizeof(double), s));
    for (size_t ci = 0; ci < B.spmv.size(); ++ci) {
      SpmvClass& c = B.spmv[ci];
      float best = 1e30f;
      int bestG = c.G;
      for (int G : {8, 16, 32, 64}) {
        SpmvClass trial = c;
        trial.G = G;
        build_spmv_items(trial, (int)ci);
        WorkItem* d = nullptr;
        FC_TRY_B(upload_items(trial.items, &d));
        float ms = time_launches(s, B.ev[1], B.ev[2], 3, [&]() {
          (void)launch_spmv_class(B, trial, d, (int)trial.items.size(), s);
        });
        (void)hipFree(d);
        rep << "spmv B=" << c.B << " class " << ci << " G=" << G << ": " << ms << " ms\n";
        if (ms < best) {
          best = ms;
          bestG = G;
        }
      }
      c.G = bestG;
      build_spmv_items(c, (int)ci);
    }
    FC_HIP(hipGetLastError());
    for (auto& c : B.spmv) FC_TRY_B(upload_items(c.items, &c.d_items));
  }
  if (!B.sell.empty()) rep << "sliced spmv items=" << B.sell.size() << "\n";
  for (auto& c : B.spmv)
    rep << "chosen spmv B=" << c.B << " G=" << c.G << " items=" << c.items.size() << "\n";
  for (auto& c : B.schw) {
    rep << "schwarz m=" << (c.m == kMixed ? "8..27" : std::to_string(c.m));
    rep << " items=" << c.items.size() << "\n";
  }
  B.report = rep.str();
  for (auto& c : B.spmv)
    if (!c.items.empty()) FC_HIP(dev_malloc(&c.d_act, c.items.size() * sizeof(WorkItem)));
  for (auto& c : B.schw)
    if (!c.items.empty()) FC_HIP(dev_malloc(&c.d_act, c.items.size() * sizeof(WorkItem)));
  if (!B.sell.empty()) FC_HIP(dev_malloc(&B.d_act_sell, B.sell.size() * sizeof(SellItem)));
  FC_HIP(dev_malloc(&B.d_act_pull, B.pull_items.size() * sizeof(WorkItem)));
  FC_HIP(dev_malloc(&B.d_act_wide, B.wide_items.size() * sizeof(WorkItem)));
  B.act_dofs = -1;   // lists not built yet
  FC_HIP(hipStreamSynchronize(s));
  *out = bt.release();
  return FC_OK;
}

// Running out of host memory is reported instead of crossing the C boundary.
template <class F>
static fc_status no_throw(const char* what, F&& f) {
  try {
    return f();
  } catch (const std::bad_alloc&) {
    set_error(std::string(what) + ": out of host memory");
    return FC_E_NOMEM;
  }
}

extern "C" fc_status fc_batch_create(int32_t nprob, const fc_problem* problems,
                                     const fc_precond* preconds, int32_t autotune, void* stream,
                                     fc_batch* out) {
  return no_throw("fc_batch_create", [&] {
    return batch_create_body(nprob, problems, preconds, autotune, stream, out);
  });
}

extern "C" fc_status fc_batch_info(fc_batch bt, int64_t* total_dofs, int32_t* n_spmv_classes,
                                   int32_t* n_schwarz_classes, char* report, int64_t report_len) {
  if (!bt) return FC_E_ARG;
  if (total_dofs) *total_dofs = bt->total_dofs;
  if (n_spmv_classes) *n_spmv_classes = (int32_t)bt->spmv.size() + (bt->sell.empty() ? 0 : 1);
  if (n_schwarz_classes) *n_schwarz_classes = (int32_t)bt->schw.size();
  if (report && report_len > 0) {
    const size_t k = std::min<size_t>(bt->report.size(), (size_t)report_len - 1);
    std::memcpy(report, bt->report.data(), k);
    report[k] = '\0';
  }
  return FC_OK;
}

// Launched lists = the tiles of the problems marked running (synchronous
// upload into the full-size arrays allocated at creation).
static fc_status compact_lists(fc_batch_s& B, const std::vector<char>& running) {
  auto filter = [&](const auto& all, auto* d, int* n) -> fc_status {
    std::vector<std::remove_reference_t<decltype(*d)>> v;
    v.reserve(all.size());
    for (const auto& w : all)
      if (running[w.prob]) v.push_back(w);
    *n = (int)v.size();
    if (v.empty()) return FC_OK;
    FC_HIP(hipMemcpyAsync(d, v.data(), v.size() * sizeof(*d), hipMemcpyHostToDevice, B.stream));
    FC_HIP(hipStreamSynchronize(B.stream));   // the host list dies here
    return FC_OK;
  };
  FC_TRY_B(filter(B.sell, B.d_act_sell, &B.n_act_sell));
  for (auto& c : B.spmv) FC_TRY_B(filter(c.items, c.d_act, &c.n_act));
  for (auto& c : B.schw) FC_TRY_B(filter(c.items, c.d_act, &c.n_act));
  FC_TRY_B(filter(B.pull_items, B.d_act_pull, &B.n_act_pull));
  FC_TRY_B(filter(B.wide_items, B.d_act_wide, &B.n_act_wide));
  B.act_dofs = 0;
  for (int k = 0; k < B.nprob; ++k)
    if (running[k]) B.act_dofs += B.host[k].n_dofs;
  return FC_OK;
}

// Capture `chunk` steps over the current lists into the batch's graph.
static fc_status capture_steps(fc_batch_s& B, int chunk, hipStream_t s) {
  if (B.exec) {
    FC_HIP(hipGraphExecDestroy(B.exec));
    B.exec = nullptr;
  }
  if (B.graph) {
    FC_HIP(hipGraphDestroy(B.graph));
    B.graph = nullptr;
  }
  FC_HIP(hipStreamBeginCapture(s, hipStreamCaptureModeThreadLocal));
  hipError_t e = enqueue_batch_steps(B, chunk, s);
  hipGraph_t g = nullptr;
  hipError_t e2 = hipStreamEndCapture(s, &g);
  if (e != hipSuccess) FC_HIP(e);
  FC_HIP(e2);
  B.graph = g;
  FC_HIP(hipGraphInstantiate(&B.exec, g, nullptr, nullptr, 0));
  B.key_chunk = chunk;
  return FC_OK;
}

static fc_status solve_batch_body(fc_batch bt, const double* const* b_dev, double* const* x_dev,
                                  const fc_solve_opts* opts, fc_solve_info* infos, void* stream) {
  if (!bt || !b_dev || !x_dev) {
    set_error("fc_pcg_solve_batch: invalid arguments");
    return FC_E_ARG;
  }
  fc_solve_opts o{1e-8, 300000, FC_STOP_PRECOND, FC_MODE_F64, 16, 1e-4, nullptr, 0};
  if (opts) o = *opts;
  if (o.mode != FC_MODE_F64 || !(o.tol >= 0.0) || o.maxit < 0) {
    set_error("fc_pcg_solve_batch: only FP64 mode with valid tol/maxit is supported");
    return FC_E_UNSUPPORTED;
  }
  fc_batch_s& B = *bt;
  hipStream_t s = B.stream;
  hipStream_t user = (hipStream_t)stream;
  bool changed = false;
  if ((int)B.key_b.size() != B.nprob) {
    B.key_b.assign(B.nprob, nullptr);
    B.key_x.assign(B.nprob, nullptr);
  }
  for (int k = 0; k < B.nprob; ++k) {
    if (!b_dev[k] || !x_dev[k]) {
      set_error("fc_pcg_solve_batch: NULL vector");
      return FC_E_ARG;
    }
    if (B.host[k].b != b_dev[k] || B.host[k].x != x_dev[k]) changed = true;
    B.host[k].b = b_dev[k];
    B.host[k].x = x_dev[k];
  }
  FC_HIP(hipEventRecord(B.ev[0], user));
  FC_HIP(hipStreamWaitEvent(s, B.ev[0], 0));
  if (changed)
    FC_HIP(hipMemcpyAsync(B.d_probs, B.host.data(), B.nprob * sizeof(BProb),
                          hipMemcpyHostToDevice, s));
  std::vector<CgScalars> init(B.nprob);
  for (auto& c : init) {
    std::memset(&c, 0, sizeof(c));
    c.tol = o.tol;
    c.maxit = o.maxit;
    c.stop = o.stop;
  }
  FC_HIP(hipMemcpyAsync(B.sc, init.data(), B.nprob * sizeof(CgScalars), hipMemcpyHostToDevice, s));
  FC_HIP(hipEventRecord(B.ev[1], s));
  const int np = (int)B.pull_items.size();
  // start: r = b, x = 0, z = S r, p = z, scalars
  hipLaunchKernelGGL(kb_init, dim3((unsigned)B.wide_items.size()), dim3(256), 0, s, B.d_probs,
                     B.d_wide, B.r);
  for (auto& c : B.schw)
    FC_HIP(launch_schwarz_class(B, c, c.d_items, (int)c.items.size(), nullptr, s));
  hipLaunchKernelGGL(kb_pull<0>, dim3(np), dim3(256), 0, s, B.d_probs, B.d_pull, np, B.sc, B.r,
                     B.p, B.q, B.z, B.partial);
  hipLaunchKernelGGL(kb_start, dim3(B.nprob), dim3(256), 0, s, B.d_probs, B.sc, B.partial, np);
  FC_HIP(hipGetLastError());
  const int chunk = o.check_every > 0 ? o.check_every : 16;
  // every problem runs at the start; the lists shrink as problems stop
  std::vector<char> running(B.nprob, 1);
  if (B.act_dofs != B.total_dofs || !B.exec || B.key_chunk != chunk) {
    FC_TRY_B(compact_lists(B, running));
    FC_TRY_B(capture_steps(B, chunk, s));
  }
  const int64_t max_chunks = (o.maxit + chunk - 1) / chunk + 1;
  // FC_BATCH_PROGRESS=k: report the number of converged members on stderr
  // every k chunks (long uneven batches otherwise run silently for minutes)
  const char* prog_env = std::getenv("FC_BATCH_PROGRESS");
  const int64_t prog = prog_env ? std::max<int64_t>(0, std::atoll(prog_env)) : 0;
  int64_t launched = 0;
  for (;;) {
    // no more steps than maxit leaves (a stopped step still dispatches its
    // grids: 66 us for 16 members)
    const int64_t left = o.maxit - launched * chunk;
    if (left > 0 && left < chunk)
      FC_HIP(enqueue_batch_steps(B, (int)left, s));
    else
      FC_HIP(hipGraphLaunch(B.exec, s));
    ++launched;
    FC_HIP(hipMemcpyAsync(B.host_sc, B.sc, B.nprob * sizeof(CgScalars), hipMemcpyDeviceToHost, s));
    FC_HIP(hipStreamSynchronize(s));
    int ndone = 0;
    int64_t run_dofs = 0;
    for (int k = 0; k < B.nprob; ++k) {
      running[k] = B.host_sc[k].done == 0;
      ndone += !running[k];
      if (running[k]) run_dofs += B.host[k].n_dofs;
    }
    if (prog && launched % prog == 0) {
      std::fprintf(stderr, "[batch] %lld iterations: %d of %d members stopped\n",
                   (long long)(launched * chunk), ndone, B.nprob);
      std::fflush(stderr);
    }
    if (ndone == B.nprob || launched > max_chunks) break;
    // drop stopped problems from the launched lists once they hold 30 % of
    // the unknowns (their tiles would only return at once, but each still
    // costs a workgroup dispatch)
    if (run_dofs < 0.7 * (double)B.act_dofs) {
      FC_TRY_B(compact_lists(B, running));
      FC_TRY_B(capture_steps(B, chunk, s));
    }
  }
  FC_HIP(hipEventRecord(B.ev[2], s));
  FC_HIP(hipStreamSynchronize(s));
  FC_HIP(hipStreamWaitEvent(user, B.ev[2], 0));
  float ms = 0.f;
  FC_HIP(hipEventElapsedTime(&ms, B.ev[1], B.ev[2]));
  fc_status worst = FC_OK;
  for (int k = 0; k < B.nprob; ++k) {
    const CgScalars& h = B.host_sc[k];
    fc_status st = h.done == 1 ? FC_OK : h.done == 3 ? FC_E_BREAKDOWN : h.done == 4 ? FC_E_NAN
                                                                                  : FC_E_NOTCONV;
    if (st != FC_OK && worst == FC_OK) worst = st;
    if (infos) {
      fc_solve_info& I = infos[k];
      std::memset(&I, 0, sizeof(I));
      I.iters = h.iter;
      I.outer_iters = 1;
      I.rel_res_prec = h.zn0 > 0 ? std::sqrt(h.zz) / h.zn0 : 0.0;
      I.rel_res_true = h.rn0 > 0 ? std::sqrt(h.rr) / h.rn0 : 0.0;   // recurrence residual
      I.status = st;
      I.ms_solve = ms;
    }
  }
  return worst;
}

extern "C" fc_status fc_pcg_solve_batch(fc_batch bt, const double* const* b_dev,
                                        double* const* x_dev, const fc_solve_opts* opts,
                                        fc_solve_info* infos, void* stream) {
  return no_throw("fc_pcg_solve_batch",
                  [&] { return solve_batch_body(bt, b_dev, x_dev, opts, infos, stream); });
}

extern "C" void fc_batch_destroy(fc_batch bt) { destroy_batch(bt); }
