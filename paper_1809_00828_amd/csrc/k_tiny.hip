// CG steps of a tiny problem in one workgroup.
//
// A step of a small problem is four launches of 2 - 4 us whose work is a fraction
// of that, with a gap of 1 - 4 us after each.  Where the sliced matrix and the
// local inverses together are small enough for one compute unit to read in less
// time, one workgroup of 16 waves does all steps of a chunk: p, q, r, z and the block
// outputs stay in LDS, x in registers, and a barrier stands where a launch
// did.  Bound by the chain of L2 latencies within a step.  2-D, 16^2 cells, p = 2
// (1,089 unknowns, 0.22 MB): 7.2 us a step, 15.2 in four launches.
#include "dev_common.h"
#include "k_spmv.h"
#include "k_tiny.h"
#include "routes.h"
#include "schwarz_dev.h"
#include "spmv_dev.h"

namespace fc {

constexpr int kTinyWaves = kTinyThreads / 64;

struct TinyArgs {
  SellView A;
  const double* Q;
  const double* fb;   // may be null
  PullLattice lat;
  int n, n_blocks, steps;
  double *x, *r, *p, *z;
  CgScalars* sc;
};

// sums of kN values over the workgroup, the same in every thread
template <int kN>
__device__ __forceinline__ void tiny_sums(double (&v)[kN], double (*red)[kTinyWaves], int w,
                                          int l) {
#pragma unroll
  for (int k = 0; k < kN; ++k) {
    v[k] = wave_sum_last(v[k]);
    if (l == 63) red[k][w] = v[k];
  }
  __syncthreads();
#pragma unroll
  for (int k = 0; k < kN; ++k) {
    v[k] = red[k][0];
    for (int u = 1; u < kTinyWaves; ++u) v[k] += red[k][u];
  }
}

template <int P, int kDim>
__global__ __launch_bounds__(64 * kTinyWaves) void k_cg_tiny(const TinyArgs T) {
  constexpr int kM = kDim == 2 ? (P + 1) * (P + 1) : (P + 1) * (P + 1) * (P + 1);
  constexpr int kBpw = 64 / kM;
  extern __shared__ __align__(16) double lds[];
  __shared__ double red_q[1][kTinyWaves], red_z[3][kTinyWaves];
  __shared__ CgScalars S;
  const int n = T.n, tid = threadIdx.x, l = tid & 63;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  double *p = lds, *q = p + n, *r = q + n, *z = r + n, *y = z + n;
  double* rB = y + (int64_t)T.n_blocks * kM + 64 * w;   // of this wave
  if (tid == 0) S = *T.sc;
  double x[kTinyElems];
#pragma unroll
  for (int e = 0; e < kTinyElems; ++e) {
    const int i = tid + 64 * kTinyWaves * e;
    if (i >= n) continue;
    p[i] = T.p[i];
    r[i] = T.r[i];
    x[e] = T.x[i];
  }
  __syncthreads();
  if (S.done) return;
  bool pulled = false;
  for (int it = 0; it < T.steps; ++it) {
    double pq[1] = {0.0};
    for (int s = w; s < T.A.n_slices; s += kTinyWaves)
      pq[0] += sell_slice_product<P, false>(T.A, T.A.slices[s], l, GatherX{p}, q);
    const double rz = S.rzn;
    tiny_sums<1>(pq, red_q, w, l);   // q is complete
    const bool ok = pq[0] > 0.0 && rz > 0.0;
    const double alpha = rz / pq[0];
    if (tid == 0) {
      S.pq = pq[0];
      S.rz = rz;
      S.iter += 1;
      if (ok) S.alpha = alpha;
      else S.done = (pq[0] != pq[0] || rz != rz) ? 4 : 3;
    }
    if (!ok) break;
    // block products on r - alpha q
    const int lb = l / kM, i = l % kM;
    for (int t = w; t * kBpw < T.n_blocks; t += kTinyWaves) {
      const int blk = t * kBpw + lb;
      const bool active = lb < kBpw && blk < T.n_blocks;
      double v[kM / 2 + 1];
      small_rows<double, kM>(T.Q + (active ? blk : 0) * sym_block_stride_dev(kM), i, v);
      const int64_t dof = active ? lattice_cell_node(T.lat, blk, i) : 0;
      const double rv = fma(-alpha, q[dof], r[dof]);
      // the wave's own entries: no other wave reads or writes them
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
      __builtin_amdgcn_wave_barrier();
      if (active) rB[l] = rv;
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
      __builtin_amdgcn_wave_barrier();
      const int g0 = (active ? lb : 0) * kM;
      const double out = small_product<double, kM>(v, rB + g0, i, g0);
      if (active) y[blk * kM + i] = out;
    }
    __syncthreads();
    // pull, x, r, z
    pulled = true;
    double acc[3] = {0.0, 0.0, 0.0};
    const int j0 = opaque(tid);   // its offsets are not held across steps
#pragma unroll
    for (int e = 0; e < kTinyElems; ++e) {
      const int j = j0 + 64 * kTinyWaves * e;
      if (j >= n) continue;
      const double fb = T.fb ? T.fb[j] : 0.0;
      double v[8];
      pull_lattice_load(y, T.lat, kM, 1, (uint32_t)j, 0, v);
      const double s = pull_sum8(v);
      const double rn = fma(-alpha, q[j], r[j]);
      x[e] = fma(alpha, p[j], x[e]);
      r[j] = rn;
      const double zn = T.fb ? fma(fb, rn, s) : s;
      z[j] = zn;
      acc[0] = fma(rn, zn, acc[0]);
      acc[1] = fma(zn, zn, acc[1]);
      acc[2] = fma(rn, rn, acc[2]);
    }
    tiny_sums<3>(acc, red_z, w, l);
    if (tid == 0) cg_beta_store(&S, acc[0], acc[1], acc[2]);
    const double beta = acc[0] / rz;
#pragma unroll
    for (int e = 0; e < kTinyElems; ++e) {
      const int j = tid + 64 * kTinyWaves * e;
      if (j < n) p[j] = fma(beta, p[j], z[j]);
    }
    __syncthreads();
    if (S.done) break;
  }
  __syncthreads();
#pragma unroll
  for (int e = 0; e < kTinyElems; ++e) {
    const int i = tid + 64 * kTinyWaves * e;
    if (i >= n) continue;
    T.p[i] = p[i];
    T.r[i] = r[i];
    T.x[i] = x[e];
    if (pulled) T.z[i] = z[i];
  }
  if (tid == 0) *T.sc = S;
}

bool tiny_fits(const fc_precond_s& pc) {
  const fc_problem_s& pb = *pc.pb;
  return spmv_has_sell(pb.A) && pc.lat.dim > 0 && pb.bdim == 1 && pc.n_blocks > 0 &&
         pc.m == pc.nn && tiny_sizes(pb.A.nnzb, pb.n_dofs, pc.n_blocks, pc.m);
}

template <int P, int kDim>
static hipError_t launch_tiny(const TinyArgs& t, size_t lds, hipStream_t s) {
  const hipError_t e = hipFuncSetAttribute((const void*)k_cg_tiny<P, kDim>,
                                           hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL((k_cg_tiny<P, kDim>), dim3(1), dim3(64 * kTinyWaves), lds, s, t);
  return hipGetLastError();
}

hipError_t launch_tiny_steps(const fc_precond_s& pc, double* x, double* r, double* p, double* z,
                             CgScalars* sc, int steps, hipStream_t s) {
  TinyArgs t{};
  t.A = sell_view(pc.pb->A);
  t.Q = pc.Q;
  t.fb = pc.n_fallback ? pc.fallback : nullptr;
  t.lat = pc.lat;
  t.n = (int)pc.pb->n_dofs;
  t.n_blocks = (int)pc.n_blocks;
  t.steps = steps;
  t.x = x;
  t.r = r;
  t.p = p;
  t.z = z;
  t.sc = sc;
  const size_t lds = tiny_lds(t.n, t.n_blocks, pc.m);
  switch (10 * pc.lat.dim + pc.lat.p) {
    case 21: return launch_tiny<1, 2>(t, lds, s);
    case 22: return launch_tiny<2, 2>(t, lds, s);
    case 23: return launch_tiny<3, 2>(t, lds, s);
    case 24: return launch_tiny<4, 2>(t, lds, s);
    case 31: return launch_tiny<1, 3>(t, lds, s);
    case 32: return launch_tiny<2, 3>(t, lds, s);
  }
  return hipErrorInvalidValue;
}

}  // namespace fc
