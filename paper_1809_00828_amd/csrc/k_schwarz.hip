// Application of the additive Schwarz preconditioner
//     z = S r = sum_B R_B^T P_B R_B r  (+ diagonal scaling)   (Sec. 3.1, Eq. 6)
// with the element-block local inverses P_B kept as dense blocks instead of
// being summed into one global sparse S (Algorithm 1 prolongates them into
// S; keeping them apart lets the gather, the block product and the scatter
// stream each block once).
//
// Phase 1 (one pass over the local inverses): per block, gather
// r_B = R_B r into LDS and write y_B = P_B r_B.
//   * FP64.  P_B is symmetric, so only its m(m+1)/2
//     distinct entries are stored, as "wrapped diagonals":
//         Q_B[k][i] = P_B[i][(i + k) mod m],   k = 0 .. floor(m/2).
//     Thread i then needs, for every k, Q_B[k][i] (the entry P[i][i+k]) and
//     Q_B[k][(i - k) mod m] (the entry P[i][i-k] by symmetry): both are
//     reads of the same stored row k, one of them rotated, so every wave
//     load is a contiguous segment, no cross-lane reduction is needed, and
//     HBM delivers each stored entry once (the rotated read hits the cache
//     line the direct read of a neighbouring thread brought in).  When m is
//     even the row k = m/2 holds every pair twice and is used once.  For
//     m <= 64 (one lane per column) the stored rows are kept in pairs,
//     rows 2j and 2j + 1 interleaved column by column, so a lane reads two
//     of its entries with one load (sym_offset).
//   * FP32: the same wrapped diagonals of the diagonally scaled inverse
//     D^{1/2} P_B D^{1/2} rounded to FP32 (FP32 accumulation), applied as
//     D^{-1/2} (.) D^{-1/2}; blocks whose rounded copy is not certified
//     positive definite are skipped there and done from the FP64 copy.
//   * BF16: the scaled Cholesky factor of the same matrix, two triangular
//     passes through LDS (positive semi-definite however rounded).
//   Every block reads its own stored inverse once per apply.
// Phase 2 (pull): every unknown sums the y_B entries of the blocks that
// contain it, in a fixed order (no atomics, bitwise reproducible), and adds
// its diagonal-scaling term.
#include <algorithm>
#include <cstdlib>
#include <vector>

#include "dev_common.h"
#include "k_schwarz.h"
#include "routes.h"
#include "schwarz_dev.h"

namespace fc {

// m > 64, symmetric layout staged through LDS in chunks of kRows stored rows, for
// blocks of up to kMaxM.  Bound by HBM: 0.21 GB of blocks of 81 in 41 us (5.2 TB/s),
// of 125 (20^3 cells, p = 4) 95 us with the pull, of 192 4.9 GB in 0.81 ms (6.2
// TB/s).  With 16 KB of LDS a workgroup and every thread's own entry of
// each row for m <= 128: 61 and 113 us.  Rows a chunk: staged_rows (routes.h).
template <typename T, int kRows, int kMaxM>
__global__ __launch_bounds__(256) void k_schwarz_sym_staged(
    const T* __restrict__ P, int64_t block_stride, const int32_t* __restrict__ elem_nodes,
    const int32_t* __restrict__ block_elem, int nn, int bd, int m,
    const double* __restrict__ r, const double* __restrict__ q, const double* __restrict__ isd,
    CgScalars* sc, const AlphaIn ai, double* __restrict__ y, int64_t n_blocks,
    const int32_t* __restrict__ list, const int32_t* __restrict__ skip) {
  using A = typename Acc<T>::type;
  // the gathered residual is kept in the accumulation type: an FP32 copy
  // rounds it to FP32 at every use anyway, and half-width entries halve the
  // LDS traffic of the rotated reads
  __shared__ A rB[kMaxM];
  __shared__ __align__(16) T tile[kRows * kMaxM];
  __shared__ double red[16];
  if (alpha_stopped(sc, ai.np > 0, blockIdx.x == 0)) return;
  // list: the workgroups handle only the listed blocks; skip: blocks
  // flagged there are left to another launch
  const int64_t blk = list ? (int64_t)list[blockIdx.x] : xcd_remap(blockIdx.x, gridDim.x);
  const bool skipped = skip && skip[blk];
  if (skipped && blockIdx.x != 0) return;   // the first workgroup stores alpha
  schwarz_staged_block<T, kRows>(
      P + blk * block_stride, skipped ? nullptr : y + blk * m, m, r, q, isd, sc, ai,
      blockIdx.x == 0, rB, tile, red,
      [&](int i) { return block_dof(elem_nodes, block_elem[blk], nn, bd, i); });
}

// m <= 64 (schwarz_small_tile)
template <typename T, int kM, bool kLat>
__global__ __launch_bounds__(256) void k_schwarz_small(
    const T* __restrict__ P, int64_t block_stride, const int32_t* __restrict__ elem_nodes,
    const int32_t* __restrict__ block_elem, int nn, int bd, int m_arg,
    const double* __restrict__ r, const double* __restrict__ q, const double* __restrict__ isd,
    CgScalars* sc, const AlphaIn ai, double* __restrict__ y, int64_t n_blocks,
    const PullLattice lat) {
  __shared__ double rB[4][64], red[16];
  if (alpha_stopped(sc, ai.np > 0, blockIdx.x == 0)) return;
  schwarz_small_tile<T, kM, kLat>(
      P, block_stride, m_arg, r, q, isd, sc, ai, blockIdx.x == 0, y, n_blocks, lat,
      xcd_remap(blockIdx.x, gridDim.x), rB, red,
      [&](int64_t blk, int i) { return block_dof(elem_nodes, block_elem[blk], nn, bd, i); });
}

// Factored low-precision product y_B = D^{-1/2} Lt (Lt^T (D^{-1/2} r_B)) with
// Lt packed by subdiagonals (k_setup.hip).  The whole packed factor of a
// block is staged in LDS with 16-byte loads, then both triangular passes
// read it from LDS:
//   t_j = sum_d Lt[off_d + j] r_{j+d}        (lane j, d = 0 .. m-1-j)
//   y_i = sum_d Lt[off_d + i - d] t_{i-d}    (lane i, d = 0 .. i)
// Each pass reads consecutive LDS words across lanes.  FP32 accumulation.
template <typename T>
__device__ __forceinline__ void stage_packed(const T* __restrict__ src, T* dst, int64_t count,
                                             int tid, int nt) {
  // 16-byte chunks where the block start is 16-byte aligned, else scalar
  const uintptr_t addr = reinterpret_cast<uintptr_t>(src);
  constexpr int V = 16 / sizeof(T);
  if ((addr % 16) == 0) {
    const int64_t nv = count / V;
    typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
    const u32x4* s4 = reinterpret_cast<const u32x4*>(src);
    u32x4* d4 = reinterpret_cast<u32x4*>(dst);
    for (int64_t c = tid; c < nv; c += nt) d4[c] = __builtin_nontemporal_load(s4 + c);
    for (int64_t c = nv * V + tid; c < count; c += nt) dst[c] = src[c];
  } else {
    for (int64_t c = tid; c < count; c += nt) dst[c] = __builtin_nontemporal_load(src + c);
  }
}

template <typename T>
__device__ __forceinline__ float ld_f32(const T* p) {
  if constexpr (sizeof(T) == 4)
    return *p;
  else
    return bf16_to_f32(*p);
}

// One block per workgroup (m > 64) or several per wave (m <= 64): the
// caller sets up rb (scaled gathered residual) and the staged factor Lb.
template <typename T>
__device__ __forceinline__ float chol_pass1(const T* Lb, const float* rb, int m, int j) {
  float t0 = 0.f, t1 = 0.f;
  int64_t off = 0;
  int d = 0;
  for (; d + 1 <= m - 1 - j; d += 2) {
    t0 = fmaf(ld_f32(Lb + off + j), rb[j + d], t0);
    off += m - d;
    t1 = fmaf(ld_f32(Lb + off + j), rb[j + d + 1], t1);
    off += m - d - 1;
  }
  if (d <= m - 1 - j) t0 = fmaf(ld_f32(Lb + off + j), rb[j + d], t0);
  return t0 + t1;
}

template <typename T>
__device__ __forceinline__ float chol_pass2(const T* Lb, const float* tb, int m, int i) {
  float y0 = 0.f, y1 = 0.f;
  int64_t off = 0;
  int d = 0;
  for (; d + 1 <= i; d += 2) {
    y0 = fmaf(ld_f32(Lb + off + i - d), tb[i - d], y0);
    off += m - d;
    y1 = fmaf(ld_f32(Lb + off + i - d - 1), tb[i - d - 1], y1);
    off += m - d - 1;
  }
  if (d <= i) y0 = fmaf(ld_f32(Lb + off + i - d), tb[i - d], y0);
  return y0 + y1;
}

constexpr int kCholLdsBytes = 75000;   // FP32 factor of m = 192: 74,112 bytes

template <typename T>
__global__ __launch_bounds__(256) void k_schwarz_chol_large(
    const T* __restrict__ L, const int32_t* __restrict__ elem_nodes,
    const int32_t* __restrict__ block_elem, int nn, int bd, int m,
    const double* __restrict__ r, const double* __restrict__ q, const double* __restrict__ isd,
    const CgScalars* __restrict__ sc, double* __restrict__ y, int64_t n_blocks) {
  extern __shared__ __align__(16) unsigned char dyn_lds[];
  __shared__ float rb[256], tb[256];
  if (cg_stopped(sc)) return;
  const int64_t blk = xcd_remap(blockIdx.x, gridDim.x);
  if (blk >= n_blocks) return;
  const double alpha = (sc && q) ? sc->alpha : 0.0;
  const int i = threadIdx.x;
  const int64_t per = (int64_t)m * (m + 1) / 2;
  T* Lb = reinterpret_cast<T*>(dyn_lds);
  stage_packed<T>(L + blk * per, Lb, per, i, blockDim.x);
  const int64_t e = block_elem[blk];
  int64_t dof = 0;
  double s = 1.0;
  if (i < m) {
    dof = (int64_t)elem_nodes[e * nn + i / bd] * bd + (i % bd);
    s = isd[dof];
    rb[i] = (float)(gather_r(r, q, alpha, dof) * s);
  }
  __syncthreads();
  if (i < m) tb[i] = chol_pass1<T>(Lb, rb, m, i);
  __syncthreads();
  if (i < m) y[blk * m + i] = (double)chol_pass2<T>(Lb, tb, m, i) * s;
}

template <typename T>
__global__ __launch_bounds__(256) void k_schwarz_chol_small(
    const T* __restrict__ L, const int32_t* __restrict__ elem_nodes,
    const int32_t* __restrict__ block_elem, int nn, int bd, int m,
    const double* __restrict__ r, const double* __restrict__ q, const double* __restrict__ isd,
    const CgScalars* __restrict__ sc, double* __restrict__ y, int64_t n_blocks) {
  extern __shared__ __align__(16) unsigned char dyn_lds[];
  __shared__ float rb[4][64], tb[4][64];
  if (cg_stopped(sc)) return;
  const double alpha = (sc && q) ? sc->alpha : 0.0;
  const int bpw = 64 / m;
  const int w = threadIdx.x / 64, l = threadIdx.x % 64;
  const int lb = l / m, i = l % m;
  const int64_t tile = xcd_remap(blockIdx.x, gridDim.x);
  const int64_t blk0 = tile * 4 * bpw;                 // first block of the workgroup
  const int64_t nwb = std::min<int64_t>(4 * bpw, n_blocks - blk0);
  const int64_t per = (int64_t)m * (m + 1) / 2;
  T* Ls = reinterpret_cast<T*>(dyn_lds);
  if (nwb > 0) stage_packed<T>(L + blk0 * per, Ls, nwb * per, threadIdx.x, blockDim.x);
  const int64_t blk = (tile * 4 + w) * bpw + lb;
  const bool active = lb < bpw && blk < n_blocks;
  int64_t dof = 0;
  double s = 1.0;
  if (active) {
    const int64_t e = block_elem[blk];
    dof = (int64_t)elem_nodes[e * nn + i / bd] * bd + (i % bd);
    s = isd[dof];
    rb[w][l] = (float)(gather_r(r, q, alpha, dof) * s);
  }
  __syncthreads();
  const T* Lb = Ls + (blk - blk0) * per;
  if (active) tb[w][l] = chol_pass1<T>(Lb, &rb[w][lb * m], m, i);
  __syncthreads();
  if (active) y[blk * m + i] = (double)chol_pass2<T>(Lb, &tb[w][lb * m], m, i) * s;
}

template <typename T>
static hipError_t phase1_chol(const fc_precond_s& pc, const T* L, const double* r,
                              const double* q, const CgScalars* sc, hipStream_t s) {
  const fc_problem_s& pb = *pc.pb;
  if (pc.n_blocks == 0) return hipSuccess;
  const int m = pc.m;
  const int64_t per = (int64_t)m * (m + 1) / 2;
  if (m > 64) {
    const int threads = 64 * ((m + 63) / 64);
    const size_t lds = (size_t)per * sizeof(T);
    (void)hipFuncSetAttribute((const void*)k_schwarz_chol_large<T>,
                              hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    hipLaunchKernelGGL(k_schwarz_chol_large<T>, dim3((unsigned)pc.n_blocks), dim3(threads), lds,
                       s, L, block_nodes(pc), pc.block_elem, pc.nn, pc.bdim, m, r, q, pc.isd, sc,
                       pc.y, pc.n_blocks);
  } else {
    const int bpw = 64 / m;
    const int64_t per_wg = 4 * (int64_t)bpw;
    const int64_t nwg = (pc.n_blocks + per_wg - 1) / per_wg;
    const size_t lds = (size_t)(per_wg * per) * sizeof(T);
    (void)hipFuncSetAttribute((const void*)k_schwarz_chol_small<T>,
                              hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    hipLaunchKernelGGL(k_schwarz_chol_small<T>, dim3((unsigned)nwg), dim3(256), lds, s, L,
                       block_nodes(pc), pc.block_elem, pc.nn, pc.bdim, m, r, q, pc.isd, sc, pc.y,
                       pc.n_blocks);
  }
  return hipGetLastError();
}

// Phase 2: z_i = sum over blocks containing i of y_B[slot] + fb_i * r_i.  kLat:
// every cell is a block, and a node's blocks follow from its lattice indices.
// fb may be null (no unknown needs the diagonal scaling).
template <bool kLat>
__global__ __launch_bounds__(256) void k_schwarz_pull(
    const double* __restrict__ y, const int32_t* __restrict__ inv_ptr,
    const int32_t* __restrict__ inv_idx, const double* __restrict__ fb, int bd, const FastDiv dbd,
    int m, const PullLattice L, uint32_t n_dofs, const double* __restrict__ r,
    double* __restrict__ z) {
  const uint32_t i = xcd_remap(blockIdx.x, gridDim.x) * 256 + threadIdx.x;
  if (i >= n_dofs) return;
  const uint32_t node = fdiv(i, dbd);
  const int c = (int)(i - node * (uint32_t)bd);
  double s;
  if constexpr (kLat) {
    double v[8];
    pull_lattice_load(y, L, m, bd, node, c, v);
    s = pull_sum8(v);
  } else {
    s = pull_mapped_sum(y, inv_ptr, inv_idx, node, c);
  }
  z[i] = fb ? fma(fb[i], r[i], s) : s;
}

// FP32 copy of the local inverses in the same storage: the diagonally scaled
// D^{1/2} P_B D^{1/2} (D = diag(A) on the block's unknowns, isd = D^{-1/2}),
// which removes the 1/alpha dynamic range of fictitious functions before
// rounding; the apply undoes the scaling in FP64.
__global__ void k_pack_f32(const double* __restrict__ Q, float* __restrict__ Q32, int m,
                           int64_t n_blocks, const double* __restrict__ isd,
                           const int32_t* __restrict__ elem_nodes,
                           const int32_t* __restrict__ block_elem, int nn, int bd) {
  const int64_t per = sym_block_stride_dev(m);
  const int64_t total = per * n_blocks;
  for (int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; t < total;
       t += (int64_t)gridDim.x * blockDim.x) {
    const int64_t blk = t / per;
    const int64_t rem = t - blk * per;
    const int k = (int)(rem / m), i = (int)(rem - (int64_t)k * m);
    int j = i + k;
    if (j >= m) j -= m;
    const int64_t dst = blk * per + sym_offset(k, i, m);
    const int64_t e = block_elem[blk];
    const int64_t di = block_dof(elem_nodes, e, nn, bd, i);
    const int64_t dj = block_dof(elem_nodes, e, nn, bd, j);
    Q32[dst] = (di < 0 || dj < 0) ? 0.0f : (float)(Q[dst] / (isd[di] * isd[dj]));
  }
}

int64_t sym_block_stride(int m) { return sym_block_stride_dev(m); }

hipError_t launch_pack_f32(const fc_precond_s& pc, hipStream_t s) {
  if (pc.n_blocks == 0) return hipSuccess;
  hipLaunchKernelGGL(k_pack_f32, dim3(8192), dim3(256), 0, s, pc.Q, pc.Q32, pc.m, pc.n_blocks,
                     pc.isd, block_nodes(pc), pc.block_elem, pc.nn, pc.bdim);
  return hipGetLastError();
}

// element nodes that differ from the lattice's (counted with an atomic only
// where one occurs)
__global__ void k_check_cells(const int32_t* __restrict__ nodes, int nn, int64_t n_el,
                              const PullLattice L, unsigned long long* __restrict__ bad) {
  for (int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; t < n_el * nn;
       t += (int64_t)gridDim.x * blockDim.x) {
    const int64_t e = t / nn;
    if (nodes[t] != lattice_cell_node(L, (int)e, (int)(t - e * nn))) atomicAdd(bad, 1ull);
  }
}

hipError_t schwarz_check_cells(const fc_problem_s& pb, const PullLattice L, bool* ok,
                               hipStream_t s) {
  *ok = false;
  unsigned long long* bad = nullptr;
  hipError_t e = dev_malloc(&bad, sizeof(*bad));
  if (e != hipSuccess) return e;
  unsigned long long hbad = 1;
  e = hipMemsetAsync(bad, 0, sizeof(*bad), s);
  if (e == hipSuccess) {
    hipLaunchKernelGGL(k_check_cells, dim3(2048), dim3(256), 0, s, pb.elem_nodes, pb.nn, pb.n_el,
                       L, bad);
    e = hipGetLastError();
  }
  if (e == hipSuccess) e = hipMemcpyAsync(&hbad, bad, sizeof(hbad), hipMemcpyDeviceToHost, s);
  if (e == hipSuccess) e = hipStreamSynchronize(s);
  (void)hipFree(bad);
  *ok = e == hipSuccess && hbad == 0;
  return e;
}

__global__ void k_inv_sqrt_diag(const double* __restrict__ d, double* __restrict__ isd, int64_t n) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * blockDim.x)
    isd[i] = d[i] > 0.0 ? 1.0 / sqrt(d[i]) : 1.0;
}

hipError_t launch_inv_sqrt_diag(const fc_problem_s& pb, double* isd, hipStream_t s) {
  hipLaunchKernelGGL(k_inv_sqrt_diag, dim3(1024), dim3(256), 0, s, pb.diag, isd, pb.n_dofs);
  return hipGetLastError();
}

template <typename T>
static void launch_staged(const fc_precond_s& pc, const T* Q, int64_t n_launch,
                          const double* r, const double* q, const double* isd,
                          CgScalars* sc, const AlphaIn ai, const int32_t* list,
                          const int32_t* skip, hipStream_t s) {
  const dim3 g((unsigned)n_launch), b(64 * ((pc.m + 63) / 64));
#define FC_STAGED(ROWS, MAXM)                                                                \
  hipLaunchKernelGGL((k_schwarz_sym_staged<T, ROWS, MAXM>), g, b, 0, s, Q,                   \
                     sym_block_stride(pc.m), block_nodes(pc), pc.block_elem, pc.nn, pc.bdim, \
                     pc.m, r, q, isd, sc, ai, pc.y, pc.n_blocks, list, skip)
#define FC_STAGED_ROWS(ROWS, MAXM) \
  case ROWS: FC_STAGED(ROWS, MAXM); break;
  const int rows = staged_rows(sizeof(T) == 8, pc.m, n_launch);
  if constexpr (sizeof(T) == 8) {
    if (pc.m <= 96) {
      switch (rows) { FC_STAGED_ROWS(6, 96) FC_STAGED_ROWS(24, 96) }
    } else if (pc.m <= 128) {
      switch (rows) { FC_STAGED_ROWS(4, 128) FC_STAGED_ROWS(16, 128) }
    } else {
      FC_STAGED(8, 192);
    }
  } else {
    if (pc.m <= 96) {
      switch (rows) { FC_STAGED_ROWS(8, 96) FC_STAGED_ROWS(24, 96) }
    } else if (pc.m <= 128) {
      switch (rows) { FC_STAGED_ROWS(8, 128) FC_STAGED_ROWS(24, 128) }
    } else {
      switch (rows) { FC_STAGED_ROWS(4, 192) FC_STAGED_ROWS(12, 192) FC_STAGED_ROWS(24, 192) }
    }
  }
#undef FC_STAGED_ROWS
#undef FC_STAGED
}

template <typename T>
static hipError_t phase1(const fc_precond_s& pc, const T* Q, const double* r, const double* q,
                         CgScalars* sc, const AlphaIn ai, hipStream_t s) {
  const double* isd = sizeof(T) == 8 ? nullptr : pc.isd;
  if (pc.n_blocks == 0) return hipSuccess;
  const int64_t stride = sym_block_stride(pc.m);
  if (pc.m > 64) {
    launch_staged<T>(pc, Q, pc.n_blocks, r, q, isd, sc, ai, nullptr,
                     sizeof(T) == 4 ? pc.unsafe_flag32 : nullptr, s);
  } else {
    const int bpw = 64 / pc.m;
    const int64_t per_wg = 4 * (int64_t)bpw;
    const int64_t nwg = (pc.n_blocks + per_wg - 1) / per_wg;
    // the block sizes of scalar and vector problems at p = 1..3 (2-D and
    // 3-D) have their own compiled kernels
    const bool lat = pc.lat.dim > 0 && pc.bdim == 1;
#define FC_SMALL_LAUNCH(KM)                                                                    \
  do {                                                                                         \
    if (lat && KM > 0)                                                                         \
      hipLaunchKernelGGL((k_schwarz_small<T, KM, true>), dim3((unsigned)nwg), dim3(256),       \
                         0, s, Q, stride, block_nodes(pc), pc.block_elem, pc.nn, pc.bdim, pc.m, \
                         r, q, isd, sc, ai, pc.y, pc.n_blocks, pc.lat);                        \
    else                                                                                       \
      hipLaunchKernelGGL((k_schwarz_small<T, KM, false>), dim3((unsigned)nwg),                 \
                         dim3(256), 0, s, Q, stride, block_nodes(pc), pc.block_elem, pc.nn,    \
                         pc.bdim, pc.m, r, q, isd, sc, ai, pc.y, pc.n_blocks, pc.lat);         \
  } while (0)
#define FC_SMALL_CASE(KM) \
  case KM: FC_SMALL_LAUNCH(KM); break;
    switch (pc.m) {
      FC_SMALL_SIZES(FC_SMALL_CASE)
      default: FC_SMALL_LAUNCH(0); break;
    }
#undef FC_SMALL_CASE
#undef FC_SMALL_LAUNCH
  }
  return hipGetLastError();
}

// FP64 symmetric product for the listed blocks (those whose FP32 copy is
// not used), one workgroup per block.
__global__ __launch_bounds__(256) void k_schwarz_sym_list(
    const double* __restrict__ Q, int64_t stride, const int32_t* __restrict__ list,
    const int32_t* __restrict__ elem_nodes, const int32_t* __restrict__ block_elem, int nn,
    int bd, int m, const double* __restrict__ r, const double* __restrict__ q,
    const CgScalars* __restrict__ sc, double* __restrict__ y) {
  __shared__ double rB[256];
  if (cg_stopped(sc)) return;
  const int64_t blk = list[blockIdx.x];
  const double alpha = (sc && q) ? sc->alpha : 0.0;
  const int i = threadIdx.x;
  if (i < m) {
    const int64_t e = block_elem[blk];
    const int64_t dof = block_dof(elem_nodes, e, nn, bd, i);
    rB[i] = dof >= 0 ? gather_r(r, q, alpha, dof) : 0.0;
  }
  __syncthreads();
  if (i < m) y[blk * m + i] = sym_row<double>(Q + blk * stride, rB, m, i);
}

bool schwarz_takes_alpha(const fc_precond_s& pc, int precision) {
  return pc.n_blocks > 0 && precision != 2;
}

hipError_t launch_schwarz_phase1(const fc_precond_s& pc, int precision, const double* r,
                                 const double* q, CgScalars* sc, const AlphaIn ai,
                                 hipStream_t s) {
  switch (precision) {
    case 0:
      return phase1<double>(pc, pc.Q, r, q, sc, ai, s);
    case 1: {
      if (!pc.Q32 || !pc.Q) return hipErrorInvalidValue;
      hipError_t e = phase1<float>(pc, pc.Q32, r, q, sc, ai, s);
      if (e != hipSuccess || pc.n_unsafe32 == 0) return e;
      // the first launch has stored alpha
      if (pc.m > 64)
        launch_staged<double>(pc, pc.Q, pc.n_unsafe32, r, q, nullptr, sc, AlphaIn{}, pc.unsafe32,
                              nullptr, s);
      else
        hipLaunchKernelGGL(k_schwarz_sym_list, dim3((unsigned)pc.n_unsafe32),
                           dim3(64 * ((pc.m + 63) / 64)), 0, s, pc.Q, sym_block_stride(pc.m),
                           pc.unsafe32, block_nodes(pc), pc.block_elem, pc.nn, pc.bdim, pc.m, r, q,
                           sc, pc.y);
      return hipGetLastError();
    }
    case 2:
      if (!pc.Lbf) return hipErrorInvalidValue;
      return phase1_chol<uint16_t>(pc, pc.Lbf, r, q, sc, s);
  }
  return hipErrorInvalidValue;
}

hipError_t launch_schwarz_pull(const fc_precond_s& pc, const double* r, double* z,
                               hipStream_t s) {
  const int64_t n = pc.pb->n_dofs;
  if (n == 0) return hipSuccess;
  const dim3 g((unsigned)((n + 255) / 256)), b(256);
  const double* fb = pc.n_fallback ? pc.fallback : nullptr;
  const FastDiv dbd = make_fastdiv((uint32_t)pc.bdim);
  if (pc.lat.dim > 0)
    hipLaunchKernelGGL(k_schwarz_pull<true>, g, b, 0, s, pc.y, pc.inv_ptr, pc.inv_idx, fb, pc.bdim,
                       dbd, pc.m, pc.lat, (uint32_t)n, r, z);
  else
    hipLaunchKernelGGL(k_schwarz_pull<false>, g, b, 0, s, pc.y, pc.inv_ptr, pc.inv_idx, fb,
                       pc.bdim, dbd, pc.m, pc.lat, (uint32_t)n, r, z);
  return hipGetLastError();
}

hipError_t launch_schwarz_apply(const fc_precond_s& pc, const double* r, double* z,
                                hipStream_t s) {
  hipError_t e = launch_schwarz_phase1(pc, 0, r, nullptr, nullptr, AlphaIn{}, s);
  if (e != hipSuccess) return e;
  return launch_schwarz_pull(pc, r, z, s);
}

}  // namespace fc
