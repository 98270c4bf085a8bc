// Set-up of the additive Schwarz preconditioner on the device
// (Algorithm 1 of the paper, Sec. 4.3):
//   extractSubMatrix      A_B = R_B A R_B^T gathered from the BSR matrix
//   computePseudoInverse  the stabilised local inverse of Eqs. (9)-(11):
//                         eigen-decompose A_B, drop eigenvalues at or below
//                         eps * max eigenvalue, sum 1/lambda v v^T
//   diagonal scaling      1/A_ll for every unknown whose entry S_ll is zero
//
// Local inverses are computed in one of two ways, both FP64:
//  * a certified direct inverse.  The block is inverted by the symmetric
//    sweep operator in registers: a column per lane, one to four blocks per
//    wave, for m <= 64, 16 x 16 tiles on the FP64 matrix cores for 64 < m <=
//    192.  The result is accepted only when every pivot is
//    positive and trace(P) * ||A_B||_inf * eps * 4 < 1.  Since
//    lambda_min >= 1/trace(A_B^-1) and lambda_max <= ||A_B||_inf, that
//    certificate proves no eigenvalue lies within a factor 4 of the
//    threshold, so the pseudo-inverse equals the inverse.
//  * cyclic two-sided Jacobi eigen-decomposition (parallel round-robin
//    ordering, m/2 disjoint rotations per step), then
//    P_B = V diag(1/lambda_+) V^T: for the blocks that fail the
//    certificate, and for every block of the unstabilised inverse when
//    m <= 64.  The block and its eigenvectors stay in LDS when they fit,
//    else in global memory.
#include <algorithm>

#include "k_setup.h"
#include "schwarz_dev.h"

namespace fc {

// ---------------------------------------------------------- extraction
__global__ __launch_bounds__(256) void k_block_extract(
    const int32_t* __restrict__ rowptr, const int32_t* __restrict__ col,
    const double* __restrict__ val, const int32_t* __restrict__ elem_nodes,
    const int32_t* __restrict__ block_elem, const int32_t* __restrict__ list, int64_t b0, int nn,
    int bd, int m, double* __restrict__ out) {
  const int64_t blk = list ? (int64_t)list[blockIdx.x] : b0 + blockIdx.x;
  const int64_t e = block_elem[blk];
  const int32_t* en = elem_nodes + e * nn;
  double* Ab = out + blockIdx.x * (int64_t)m * m;
  const int bb = bd * bd;
  for (int t = threadIdx.x; t < nn * nn; t += blockDim.x) {
    const int a = t / nn, b = t % nn;
    const int32_t na = en[a], nb = en[b];
    if (na < 0 || nb < 0) {
      // padding of a boundary vertex patch: zero rows and columns, whose
      // zero eigenvalues the threshold of Eq. 11 drops
      for (int i = 0; i < bd; ++i)
        for (int j = 0; j < bd; ++j) Ab[(int64_t)(a * bd + i) * m + (b * bd + j)] = 0.0;
      continue;
    }
    const int32_t lo = rowptr[na], hi = rowptr[na + 1];
    int32_t l = lo, h = hi - 1, found = -1;
    while (l <= h) {
      int32_t mid = (l + h) >> 1;
      int32_t c = col[mid];
      if (c == nb) {
        found = mid;
        break;
      }
      if (c < nb) l = mid + 1;
      else h = mid - 1;
    }
    const int64_t L = hi - lo;
    for (int i = 0; i < bd; ++i)
      for (int j = 0; j < bd; ++j) {
        double v = 0.0;
        if (found >= 0) v = val[(int64_t)lo * bb + (int64_t)(i * bd + j) * L + (found - lo)];
        Ab[(int64_t)(a * bd + i) * m + (b * bd + j)] = v;
      }
  }
}

// ------------------------------------------------------- Jacobi eigen
// Pair `pi` of round-robin step `step` over mp (even) players.
__device__ __forceinline__ void rr_pair(int pi, int step, int mp, int* p, int* q) {
  auto player = [&](int pos) { return pos == 0 ? 0 : 1 + (pos - 1 + step) % (mp - 1); };
  int a = player(pi), b = player(mp - 1 - pi);
  *p = a < b ? a : b;
  *q = a < b ? b : a;
}

constexpr int kMaxJacobiM = 192;

// In: A_B of the workgroup's block in P (row-major m x m).  Out: P_B in place.
// With kLds the block and eigenvectors live in dynamic LDS (m <= 64), otherwise
// in `work` (2*m*m doubles per workgroup).  sel: the blocks' numbers, for
// `dropped`.
template <bool kLds>
__global__ __launch_bounds__(256) void k_jacobi_pinv(
    double* __restrict__ P, int m, const int32_t* __restrict__ sel,
    double* __restrict__ work, double eps, int stabilize,
    int32_t* __restrict__ dropped) {
  extern __shared__ double dyn[];
  __shared__ double cs[kMaxJacobiM / 2 + 1], sn[kMaxJacobiM / 2 + 1];
  __shared__ int pp[kMaxJacobiM / 2 + 1], qq[kMaxJacobiM / 2 + 1];
  __shared__ double invl[kMaxJacobiM];
  __shared__ double red[16];
  __shared__ int rotated;
  const int64_t blk = sel[blockIdx.x];
  double* Ab = P + blockIdx.x * (int64_t)m * m;
  const int ld = kLds ? m + 1 : m;
  double* A = kLds ? dyn : work + (int64_t)blockIdx.x * 2 * m * m;
  double* V = A + (int64_t)m * ld;
  const int tid = threadIdx.x, nt = blockDim.x;
  for (int t = tid; t < m * m; t += nt) {
    const int i = t / m, j = t % m;
    A[i * ld + j] = Ab[t];
    V[i * ld + j] = (i == j) ? 1.0 : 0.0;
  }
  __syncthreads();
  const int mp = m + (m & 1), np = mp / 2;
  for (int sweep = 0; sweep < 40; ++sweep) {
    if (tid == 0) rotated = 0;
    __syncthreads();
    for (int step = 0; step < mp - 1; ++step) {
      for (int pi = tid; pi < np; pi += nt) {
        int p, q;
        rr_pair(pi, step, mp, &p, &q);
        double c = 1.0, s = 0.0;
        if (q < m) {
          const double app = A[p * ld + p], aqq = A[q * ld + q], apq = A[p * ld + q];
          if (apq != 0.0 && fabs(apq) > 2.220446049250313e-16 * sqrt(fabs(app * aqq))) {
            const double tau = (aqq - app) / (2.0 * apq);
            const double t = (tau >= 0.0 ? 1.0 : -1.0) / (fabs(tau) + sqrt(1.0 + tau * tau));
            c = 1.0 / sqrt(1.0 + t * t);
            s = t * c;
            rotated = 1;
          }
        }
        cs[pi] = c;
        sn[pi] = s;
        pp[pi] = p;
        qq[pi] = q;
      }
      __syncthreads();
      // rows p, q of J^T A
      for (int t = tid; t < np * m; t += nt) {
        const int pi = t / m, j = t % m;
        const double s = sn[pi];
        if (s == 0.0) continue;
        const double c = cs[pi];
        const int p = pp[pi], q = qq[pi];
        const double apj = A[p * ld + j], aqj = A[q * ld + j];
        A[p * ld + j] = c * apj - s * aqj;
        A[q * ld + j] = s * apj + c * aqj;
      }
      __syncthreads();
      // columns p, q of (J^T A) J and of V J
      for (int t = tid; t < np * m; t += nt) {
        const int pi = t / m, i = t % m;
        const double s = sn[pi];
        if (s == 0.0) continue;
        const double c = cs[pi];
        const int p = pp[pi], q = qq[pi];
        const double aip = A[i * ld + p], aiq = A[i * ld + q];
        A[i * ld + p] = c * aip - s * aiq;
        A[i * ld + q] = s * aip + c * aiq;
        const double vip = V[i * ld + p], viq = V[i * ld + q];
        V[i * ld + p] = c * vip - s * viq;
        V[i * ld + q] = s * vip + c * viq;
      }
      __syncthreads();
    }
    if (!rotated) break;
    __syncthreads();
  }
  // threshold of Eq. (11) relative to the largest eigenvalue of the block
  double lmax = -1e308;
  for (int k = tid; k < m; k += nt) lmax = fmax(lmax, A[k * ld + k]);
  {
    double v = lmax;
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v = fmax(v, __shfl_xor(v, o, 64));
    if (tid % 64 == 0) red[tid / 64] = v;
    __syncthreads();
    v = -1e308;
    for (int w = 0; w < nt / 64; ++w) v = fmax(v, red[w]);
    lmax = v;
    __syncthreads();
  }
  int ndrop = 0;
  for (int k = tid; k < m; k += nt) {
    const double lam = A[k * ld + k];
    bool keep = stabilize ? (lmax > 0.0 && lam > eps * lmax) : (lam != 0.0);
    invl[k] = keep ? 1.0 / lam : 0.0;
    ndrop += keep ? 0 : 1;
  }
  __syncthreads();
  {
    double nd = block_sum((double)ndrop, red);
    if (tid == 0 && dropped) dropped[blk] = (int32_t)nd;
  }
  for (int t = tid; t < m * m; t += nt) {
    const int i = t / m, j = t % m;
    double acc = 0.0;
    for (int k = 0; k < m; ++k) acc = fma(V[i * ld + k] * invl[k], V[j * ld + k], acc);
    Ab[t] = acc;
  }
}

// ------------------------------------------------- certified sweep inverse
// Sweep operator on a symmetric matrix: sweeping every pivot turns A into
// -A^{-1}.  Both kernels below read A_B straight from the lattice matrix (a
// dense copy otherwise), keep the block in registers through all pivots and
// write the stored rows of the apply copy Q (sym_offset); a block that fails a
// pivot or the certificate is flagged in need_eig and left to the
// eigen-decomposition.

// Rows of A through the nodes of one cell: the entry of row a in the column of
// node b starts at base and lies at gx + len0 gy + len01 gz - pos0 of the L
// entries of every component pair.
struct BlockRow {
  int64_t base;
  int32_t pos0, len0, len01, L;
};

struct BlockSrc {
  const double* val;          // lattice matrix, or
  const double* dense;        // [count][m][m], block b0 first
  const int32_t* block_elem;
  LatticeInfo lat;
  PullLattice cells;
  FastDiv dbd;
  int bd;
};

// Row table entry and lattice indices of local node a of cell e.
__device__ __forceinline__ void block_row(const BlockSrc& S, int32_t e, int a, BlockRow* row,
                                          int4* g) {
  int c[3] = {0, 0, 0};
  uint32_t ee = (uint32_t)e, ll = (uint32_t)a;
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    if (k < S.cells.dim) {
      const uint32_t eq = fdiv(ee, S.cells.dn), lq = fdiv(ll, S.cells.dp1);
      const int cell = (int)(ee - eq * (uint32_t)S.cells.n);
      const int l = (int)(ll - lq * (uint32_t)(S.cells.p + 1));
      ee = eq;
      ll = lq;
      c[k] = cell * S.cells.p + (l == 0 ? 0 : l == 1 ? S.cells.p : l - 1);
    }
  }
  const RowBox b = row_box_at(c, S.lat);
  row->base = lattice_row_start_at(c, b, S.lat);
  row->len0 = b.len[0];
  row->len01 = b.len[0] * b.len[1];
  row->L = row->len01 * b.len[2];
  row->pos0 = b.lo[0] + b.len[0] * (b.lo[1] + b.len[1] * b.lo[2]);
  *g = int4{c[0], c[1], c[2], 0};
}

__device__ __forceinline__ double block_entry(const BlockSrc& S, const BlockRow& r, int ci,
                                              const int4& g, int cj) {
  const int pos = g.x + r.len0 * g.y + r.len01 * g.z - r.pos0;
  return S.val[r.base * (S.bd * S.bd) + (int64_t)(ci * S.bd + cj) * r.L + pos];
}

// m > 64: blocked sweep on the FP64 matrix cores.  The upper tiles (16 x 16,
// NT (NT + 1) / 2 of them) of the symmetric block stay in the accumulators of
// eight waves.  Per panel of 16 pivots the panel's row of tiles, P, goes to LDS
// and one wave factors the diagonal tile, D = L G L^T, keeping E = L^{-1}; then
// with B = E P, four v_mfma_f64_16x16x4 steps a tile,
//     A_IJ -= B_I^T G^{-1} B_J,   A_KJ = E^T G^{-1} B_J,   A_KK = -E^T G^{-1} E.
// (D^{-1} P in place of the factored form would be one product less, but loses
// the condition number of D in the update instead of its root: thin cut cells
// came out indefinite.)  Padding rows are rows of the identity.
// Operand layouts (one wave, lane l, c = l % 16, g = l / 16): A[c][4s + g] and
// B[4s + g][c] for step s, D[4r + g][c] in register r.
// Bound by the chain panel (1,200 cycles) -> diagonal tile (4,500) -> B (2,000) ->
// update (7,300, of them 5,100 matrix instructions) with one block of 192 per
// compute unit: 1.78 ms for the 4,096 blocks of elasticity 16^3 cells, p = 3 (58
// GFLOP, 33 TFLOP/s).  A rank-one update per pivot on the VALU, with a barrier
// each (4,000 cycles a pivot, 576 of them arithmetic), took 5.13 ms, on top of
// 0.71 ms extraction and 1.05 ms packing.
typedef double d4 __attribute__((ext_vector_type(4)));

template <int K>
__device__ __forceinline__ double bcast16(double v) {   // lane K of every 16
  return __longlong_as_double(
      __builtin_amdgcn_update_dpp(0ll, __double_as_longlong(v), 0x150 + K, 0xf, 0xf, false));
}

// 1 / d by two Newton steps from the hardware's estimate, within an ulp: half
// the dependent operations of the exactly rounded division.
__device__ __forceinline__ double recip(double d) {
  double r = __builtin_amdgcn_rcp(d);
  r = fma(r, fma(-d, r, 1.0), r);
  return fma(r, fma(-d, r, 1.0), r);
}

// v of the lane with the same c in group G, in every group.
template <int G>
__device__ __forceinline__ double bcast_group(double v) {
  typedef unsigned int u2 __attribute__((ext_vector_type(2)));
  const long long b = __double_as_longlong(v);
  unsigned int o[2];
#pragma unroll
  for (int k = 0; k < 2; ++k) {
    unsigned int u = (unsigned int)(b >> (32 * k));
    const u2 p = __builtin_amdgcn_permlane16_swap(u, u, false, false);   // odd and even groups
    u = p[G & 1];
    const u2 q = __builtin_amdgcn_permlane32_swap(u, u, false, false);   // lower and upper half
    o[k] = q[G >> 1];
  }
  return __longlong_as_double(((long long)o[1] << 32) | (long long)o[0]);
}

// Pivots K .. 15 of a 16 x 16 tile x in D layout (one wave): x becomes upper
// triangular (G L^T), e, from the identity, L^{-1}, and lane c of every 16
// holds the pivot G_cc in gi.  All moves between lanes are VALU ones, and nothing
// branches: through LDS permutes a pivot took twice as long.
template <int K>
__device__ __forceinline__ void factor_tile(d4& x, d4& e, double& gi, int c, int g) {
  if constexpr (K < 16) {
    constexpr int rk = K / 4, gk = K % 4;
    const double xk = bcast_group<gk>(x[rk]);   // row K, column c
    const double d = bcast16<K>(xk);
    if (c == K) gi = d;
    const double rinv = recip(d);
    if constexpr (K < 15) {
      const double ek = bcast_group<gk>(e[rk]);
#pragma unroll
      for (int r = rk; r < 4; ++r) {
        double f = bcast16<K>(x[r]) * rinv;   // L_{row, K}, row 4r + g > K
        if (r == rk && g <= gk) f = 0.0;
        x[r] = fma(-f, xk, x[r]);
        e[r] = fma(-f, ek, e[r]);
      }
    }
    factor_tile<K + 1>(x, e, gi, c, g);
  }
}

template <int NT, int NW, bool kLat>
__global__ __launch_bounds__(64 * NW, 4) void k_sweep_large(const BlockSrc S, int64_t b0, int m,
                                                        double eps, int stabilize,
                                                        double* __restrict__ Q,
                                                        int32_t* __restrict__ need_eig) {
  constexpr int kTiles = NT * (NT + 1) / 2, kTQ = (kTiles + NW - 1) / NW;
  // LDS row of a panel: 17 mod 32 doubles, so that neither the rows' reads nor
  // the transposed writes meet in a bank
  constexpr int kS = 16 * NT + 17;
  __shared__ __align__(16) double buf[2 * 16 * kS];
  __shared__ double E[16][17], GE[16][17], gi[16];   // L^{-1}, G^{-1} L^{-1}, 1 / G
  __shared__ double red[16];
  __shared__ int bad;
  // the row table lies where the panels come later
  BlockRow* rows = reinterpret_cast<BlockRow*>(buf);
  int4* cols = reinterpret_cast<int4*>(buf + 192 * sizeof(BlockRow) / sizeof(double));
  double* Pan = buf;                                 // P, then B = E P: [16][kS]
  double* Wn = buf + 16 * kS;                        // -G^{-1} B
  const int64_t blk = b0 + blockIdx.x;
  const int tid = threadIdx.x, w = __builtin_amdgcn_readfirstlane(tid / 64), l = tid % 64;
  int c = l % 16, g = l / 16;
  int tI[kTQ], tJ[kTQ];
#pragma unroll
  for (int q = 0; q < kTQ; ++q) {
    int t = w + NW * q, I = 0;
    const bool on = t < kTiles;
    if (!on) t = 0;
    while (t >= NT - I) t -= NT - I++;
    tI[q] = on ? I : -1;
    tJ[q] = on ? I + t : -1;
  }
  if constexpr (kLat) {
    const int nn = (int)fdiv((uint32_t)m, S.dbd);
    if (tid < nn) block_row(S, S.block_elem[blk], tid, &rows[tid], &cols[tid]);
    __syncthreads();
  }
  d4 acc[kTQ];
#pragma unroll
  for (int q = 0; q < kTQ; ++q) {
    c = opaque(c);
    g = opaque(g);
    const int j = 16 * tJ[q] + c;
    int4 gj{0, 0, 0, 0};
    int cj = 0;
    if constexpr (kLat) {
      const int b = (int)fdiv((uint32_t)(j < m ? max(j, 0) : 0), S.dbd);
      gj = cols[b];
      cj = j - b * S.bd;
    }
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int i = 16 * tI[q] + 4 * r + g;
      double v = i == j ? 1.0 : 0.0;
      if (tI[q] >= 0 && i < m && j < m) {
        if constexpr (kLat) {
          const int a = (int)fdiv((uint32_t)i, S.dbd);
          v = block_entry(S, rows[a], i - a * S.bd, gj, cj);
        } else {
          v = S.dense[(blockIdx.x * (int64_t)m + i) * m + j];
        }
      }
      acc[q][r] = v;
    }
    __builtin_amdgcn_sched_barrier(0);
  }
  if constexpr (kLat) __syncthreads();
  // ||A_B||_inf: a tile's row sums and, above the diagonal, its column sums
  // (the rows of the transposed tile), then every row's tiles in order
  if (tid == 0) bad = 0;
#pragma unroll
  for (int q = 0; q < kTQ; ++q) {
    if (tI[q] < 0) continue;
    double cs = 0.0;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const double v = fabs(acc[q][r]);
      cs += v;
      const double rs = row16_sum_last(v);
      if (c == 15) buf[tJ[q] * (16 * NT) + 16 * tI[q] + 4 * r + g] = rs;
    }
    cs += __shfl_xor(cs, 16, 64);
    cs += __shfl_xor(cs, 32, 64);
    if (g == 0 && tI[q] != tJ[q]) buf[tI[q] * (16 * NT) + 16 * tJ[q] + c] = cs;
    __builtin_amdgcn_sched_barrier(0);
  }
  __syncthreads();
  double anorm = 0.0;
  if (tid < m)
#pragma unroll
    for (int t = 0; t < NT; ++t) anorm += buf[t * (16 * NT) + tid];
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) anorm = fmax(anorm, __shfl_xor(anorm, o, 64));
  if (l == 0) red[w] = anorm;
  __syncthreads();
  anorm = red[0];
#pragma unroll
  for (int t = 1; t < NW; ++t) anorm = fmax(anorm, red[t]);
  for (int K = 0; K < NT; ++K) {
    c = opaque(c);
    g = opaque(g);
    // the panel: rows K, columns of every tile
#pragma unroll
    for (int q = 0; q < kTQ; ++q) {
      if (tI[q] == K) {
#pragma unroll
        for (int r = 0; r < 4; ++r) Pan[(4 * r + g) * kS + 16 * tJ[q] + c] = acc[q][r];
      } else if (tJ[q] == K) {
#pragma unroll
        for (int r = 0; r < 4; ++r) Pan[c * kS + 16 * tI[q] + 4 * r + g] = acc[q][r];
      }
    }
    __syncthreads();
    if (w == K % NW) {
      d4 x, e;
      double piv = 0.0;
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        x[r] = Pan[(4 * r + g) * kS + 16 * K + c];
        e[r] = 4 * r + g == c ? 1.0 : 0.0;
      }
      factor_tile<0>(x, e, piv, c, g);
      if (stabilize ? !(piv > 0.0) : !(piv < 0.0 || piv > 0.0)) bad = 1;   // (NaN too)
      const double inv = recip(piv);
      if (g == 0) gi[c] = inv;
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        E[4 * r + g][c] = e[r];
        GE[4 * r + g][c] = e[r] * __shfl(inv, 4 * r + g, 64);
      }
    }
    __syncthreads();
    if (bad) break;
    for (int J = w; J < NT; J += NW) {
      if (J == K) continue;
      d4 t{0.0, 0.0, 0.0, 0.0};
#pragma unroll
      for (int s = 0; s < 4; ++s)
        t = __builtin_amdgcn_mfma_f64_16x16x4f64(E[c][4 * s + g],
                                                 Pan[(4 * s + g) * kS + 16 * J + c], t, 0, 0, 0);
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        Pan[(4 * r + g) * kS + 16 * J + c] = t[r];   // only this wave reads these columns now
        Wn[(4 * r + g) * kS + 16 * J + c] = -gi[4 * r + g] * t[r];
      }
    }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < kTQ; ++q) {
      const int I = tI[q], J = tJ[q];
      if (I < 0) continue;
      if (I != K && J != K) {
#pragma unroll
        for (int s = 0; s < 4; ++s)
          acc[q] = __builtin_amdgcn_mfma_f64_16x16x4f64(Pan[(4 * s + g) * kS + 16 * I + c],
                                                        Wn[(4 * s + g) * kS + 16 * J + c], acc[q],
                                                        0, 0, 0);
      } else {
        // rows K: E^T (G^{-1} B_J), columns K: B_I^T (G^{-1} E), tile K: E^T (G^{-1} E)
        d4 t{0.0, 0.0, 0.0, 0.0};
#pragma unroll
        for (int s = 0; s < 4; ++s) {
          const double av = I == K ? E[4 * s + g][c] : Pan[(4 * s + g) * kS + 16 * I + c];
          const double bv = J == K ? GE[4 * s + g][c] : -Wn[(4 * s + g) * kS + 16 * J + c];
          t = __builtin_amdgcn_mfma_f64_16x16x4f64(av, bv, t, 0, 0, 0);
        }
        const bool diag = I == J;
#pragma unroll
        for (int r = 0; r < 4; ++r) acc[q][r] = diag ? -t[r] : t[r];
      }
      __builtin_amdgcn_sched_barrier(0);   // one tile's operands at a time: registers
    }
    __syncthreads();   // the panel is read before the next one overwrites it
  }
  if (bad) {
    if (tid == 0) need_eig[blk] = 1;
    return;
  }
  double tr = 0.0;
#pragma unroll
  for (int q = 0; q < kTQ; ++q) {
    if (tI[q] < 0 || tI[q] != tJ[q]) continue;
#pragma unroll
    for (int r = 0; r < 4; ++r)
      if (4 * r + g == c && 16 * tI[q] + c < m) tr -= acc[q][r];
  }
  tr = block_sum(tr, red);
  const bool ok = !stabilize || (tr > 0.0 && tr * anorm * eps * 4.0 < 1.0);
  if (tid == 0) need_eig[blk] = ok ? 0 : 1;
  if (!ok) return;
  // the stored rows k = (j - i) mod m <= m/2, a few at a time through LDS so
  // that they leave as contiguous runs
  const int h = m / 2;
  const bool even = (m & 1) == 0;
  const int per = 2 * 16 * kS / m;
  double* Qb = Q + blk * ((int64_t)(h + 1) * m);
  for (int k0 = 0; k0 <= h; k0 += per) {
    const int cnt = min(per, h + 1 - k0);
    __syncthreads();
    c = opaque(c);
    g = opaque(g);
#pragma unroll
    for (int q = 0; q < kTQ; ++q) {
      if (tI[q] < 0) continue;
      const int j = 16 * tJ[q] + c;
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int i = 16 * tI[q] + 4 * r + g, dl = j - i;
        if (j >= m || dl < 0) continue;
        const double v = -acc[q][r];
        const int k = (dl <= h ? dl : m - dl) - k0;
        if (k >= 0 && k < cnt) {
          buf[k * m + (dl <= h ? i : j)] = v;
          if (even && dl == h) buf[k * m + j] = v;   // that row holds each pair twice
        }
      }
      __builtin_amdgcn_sched_barrier(0);
    }
    __syncthreads();
    for (int t = tid; t < cnt * m; t += 64 * NW) Qb[(int64_t)k0 * m + t] = buf[t];
  }
}

// m <= W (16, 32 or 64 lanes per block, 64 / W blocks per wave): lane j holds
// column j; the pivot row (by symmetry the pivot column) is broadcast through
// LDS within the wave, without a barrier.  KM >= m: rows and columns past m are
// those of the identity, whose pivots change nothing.  The rows are renamed by
// one place per pivot, so that the pivot is always row 0 and the loop over the
// pivots needs no unrolling (the unrolled kernel's code did not fit the
// instruction cache at m = 64).
// Bound by the VALU: 0.66 ms for the 110,592 blocks of 27 of 48^3 cells, p = 2.
// One block per wave, the pivot row read across lanes one entry at a time, took
// 1.19 ms, on top of 0.92 ms extraction and 0.28 ms packing.
template <int W, int KM, bool kLat>
__global__ __launch_bounds__(256) void k_sweep_small(const BlockSrc S, int64_t b0, int64_t count,
                                                     int m, double eps, double* __restrict__ Q,
                                                     int32_t* __restrict__ need_eig) {
  constexpr int NB = 256 / W;        // blocks per workgroup
  constexpr int kR = 16;             // rows per output round
  __shared__ double pivot[NB][2 * KM];
  __shared__ double stage[NB][kR * KM];
  __shared__ BlockRow rows[kLat ? NB : 1][kLat ? KM : 1];
  __shared__ int4 cols[kLat ? NB : 1][kLat ? KM : 1];
  const int sb = threadIdx.x / W, j = threadIdx.x % W;
  const int64_t loc = (int64_t)blockIdx.x * NB + sb;
  const bool on = loc < count;
  const int64_t blk = b0 + (on ? loc : 0);
  double a[KM];
  if constexpr (kLat) {
    const int nn = (int)fdiv((uint32_t)m, S.dbd);
    const int32_t e = S.block_elem[blk];
    if (j < nn) block_row(S, e, j, &rows[sb][j], &cols[sb][j]);
    __builtin_amdgcn_wave_barrier();   // a block's lanes are of one wave
    const int jc = j < m ? j : 0;
    const int bn = (int)fdiv((uint32_t)jc, S.dbd), cj = jc - bn * S.bd;
    const int4 gj = cols[sb][bn];
#pragma unroll
    for (int i = 0; i < KM; ++i) {
      a[i] = i == j ? 1.0 : 0.0;
      if (i < m) {
        const int an = (int)fdiv((uint32_t)i, S.dbd);
        const double v = block_entry(S, rows[sb][an], i - an * S.bd, gj, cj);
        a[i] = j < m ? v : 0.0;
      }
    }
  } else {
    const double* Ab = S.dense + (on ? loc : 0) * (int64_t)m * m;
#pragma unroll
    for (int i = 0; i < KM; ++i)
      a[i] = i < m && j < m ? Ab[(int64_t)i * m + j] : i == j ? 1.0 : 0.0;
  }
  // ||A_B||_inf: the column sums equal the row sums of the symmetric block
  double cs = 0.0;
#pragma unroll
  for (int i = 0; i < KM; ++i) cs += i < m ? fabs(a[i]) : 0.0;
  if (j >= m) cs = 0.0;
#pragma unroll
  for (int o = W / 2; o > 0; o >>= 1) cs = fmax(cs, __shfl_xor(cs, o, W));
  const double anorm = cs;
  bool bad = false;
#pragma unroll 1
  for (int k = 0; k < KM; ++k) {
    const double bj = a[0];   // row k, column j
    if (j < KM) {
      pivot[sb][j] = bj;
      pivot[sb][j + KM] = bj;
    }
    __builtin_amdgcn_wave_barrier();
    const double* pv = &pivot[sb][k];
    const double d = pv[0];
    bad = bad || !(d > 0.0);   // the same for every lane of the block
    const double rinv = 1.0 / d;
#pragma unroll
    for (int i = 1; i < KM; ++i) {
      const double bi = pv[i];   // row k, column k + i = column k, row k + i
      a[i - 1] = j == k ? bi * rinv : fma(-(bi * bj), rinv, a[i]);
    }
    a[KM - 1] = j == k ? -rinv : bj * rinv;
    __builtin_amdgcn_wave_barrier();
  }
  // trace of A_B^-1 = minus the trace of the swept block
  double tr = 0.0;
#pragma unroll
  for (int i = 0; i < KM; ++i)
    if (i == j && i < m) tr = -a[i];
#pragma unroll
  for (int o = W / 2; o > 0; o >>= 1) tr += __shfl_xor(tr, o, W);
  bad = bad || !(tr > 0.0 && tr * anorm * eps * 4.0 < 1.0);
  if (on && j == 0) need_eig[blk] = bad ? 1 : 0;
  const bool out = on && !bad;
  // 16 rows at a time to LDS, and their stored entries (k, i) = P[i][(i + k)
  // mod m] from there: pairs of stored rows side by side, an odd last one alone
  const int h = m / 2, npair = (h + 1) & ~1;
  double* Qb = Q + blk * ((int64_t)(h + 1) * m);
  double* st = stage[sb];
#pragma unroll
  for (int i0 = 0; i0 < KM; i0 += kR) {
    if (i0 >= m) break;
    __builtin_amdgcn_wave_barrier();
#pragma unroll
    for (int u = 0; u < kR; ++u)
      if (i0 + u < KM && j < KM) st[u * KM + j] = -a[i0 + u < KM ? i0 + u : 0];
    __builtin_amdgcn_wave_barrier();
    const int nr = min(kR, m - i0);
    for (int t = j; t < npair * kR; t += W) {
      const int u = (t % (2 * kR)) / 2, k = 2 * (t / (2 * kR)) + (t & 1);
      if (u < nr && out) {
        int q = i0 + u + k;
        if (q >= m) q -= m;
        Qb[(int64_t)(k & ~1) * m + 2 * (i0 + u) + (k & 1)] = st[u * KM + q];
      }
    }
    if (npair <= h && j < kR) {
      if (j < nr && out) {
        int q = i0 + j + h;
        if (q >= m) q -= m;
        Qb[(int64_t)h * m + i0 + j] = st[j * KM + q];
      }
    }
  }
}

// ------------------------------------------- factored low-precision copy
// P_B = L L^T (lower Cholesky factor of the FP64 local inverse; a pivot at
// or below 1e-14 * max diag(P_B) zeroes its column, which is exact for the
// null modes of a pseudo-inverse).  The stored factor is the diagonally
// scaled Lt = D^{1/2} L (D = diag(A) on the block, isd = D^{-1/2}), so
// Lt Lt^T = D^{1/2} P_B D^{1/2}, packed by subdiagonals:
//     diagonal d (i - j = d) at offset d*m - d*(d-1)/2, entry j.
// However it is rounded, Lt Lt^T stays positive semi-definite, which is
// what keeps CG with an FP32/BF16 preconditioner meaningful.
// Thread (ti, tj) of a GRID x GRID grid holds the T x T tile at rows
// ti*T.., columns tj*T..; the pivot row is broadcast through LDS.
__device__ __forceinline__ uint16_t f32_to_bf16(float f) {
  uint32_t u = __float_as_uint(f);
  u += 0x7fffu + ((u >> 16) & 1u);
  return (uint16_t)(u >> 16);
}

// kCheck: factor fl32(D^{1/2} P_B D^{1/2}) instead (the FP32 rounding of
// the diagonally scaled inverse) and only report, in unsafe[blk], whether a
// pivot fell to 1e-10 of the largest diagonal entry: where it does not, the
// rounded matrix is positive definite with margin and may stand in for P_B.
template <int GRID, int T, bool kCheck>
__global__ __launch_bounds__(GRID * GRID) void k_chol_pack(
    const double* __restrict__ Q, int m, const double* __restrict__ isd,
    const int32_t* __restrict__ elem_nodes, const int32_t* __restrict__ block_elem, int nn,
    int bd, uint16_t* __restrict__ Lbf, int32_t* __restrict__ unsafe) {
  __shared__ double rowbuf[2][GRID * T];
  __shared__ double red[16];
  __shared__ double sc[GRID * T];
  const int64_t blk = blockIdx.x;
  const double* Qb = Q + blk * sym_block_stride_dev(m);
  const int tid = threadIdx.x, ti = tid / GRID, tj = tid % GRID;
  const int64_t e = block_elem[blk];
  for (int i = tid; i < m; i += GRID * GRID) {
    const int64_t dof = (int64_t)elem_nodes[e * nn + i / bd] * bd + (i % bd);
    sc[i] = 1.0 / isd[dof];   // sqrt(A_ii)
  }
  __syncthreads();   // the check scales every tile entry by sc[i] sc[j]
  double a[T][T];
  double dmax = 0.0;
#pragma unroll
  for (int r = 0; r < T; ++r)
#pragma unroll
    for (int c = 0; c < T; ++c) {
      const int i = ti * T + r, j = tj * T + c;
      a[r][c] = (i < m && j < m) ? Qb[sym_entry(i, j, m)] : 0.0;
      if (kCheck && i < m && j < m) a[r][c] = (double)(float)(a[r][c] * sc[i] * sc[j]);
      if (i == j && i < m) dmax = fmax(dmax, a[r][c]);
    }
  {
    double v = dmax;
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v = fmax(v, __shfl_xor(v, o, 64));
    if (tid % 64 == 0) red[tid / 64] = v;
    __syncthreads();
    v = 0.0;
    for (int w = 0; w < (GRID * GRID + 63) / 64; ++w) v = fmax(v, red[w]);
    dmax = v;
  }
  const double tiny = (kCheck ? 1e-10 : 1e-14) * dmax;
  bool bad = false;
  for (int k = 0; k < m; ++k) {
    double* buf = rowbuf[k & 1];
    if (ti == k / T) {
      const int r = k % T;
#pragma unroll
      for (int rr = 0; rr < T; ++rr)
        if (rr == r) {
#pragma unroll
          for (int c = 0; c < T; ++c) buf[tj * T + c] = a[rr][c];
        }
    }
    __syncthreads();
    const double d = buf[k];
    const bool live = d > tiny;
    bad = bad || !live;
    const double lkk = live ? sqrt(d) : 0.0;
    const double rl = live ? 1.0 / lkk : 0.0;
    // L[i][k] below the pivot (zero elsewhere, so the rank-one update below
    // leaves every entry outside the trailing block as it is), then column
    // k of L.  Entries above the diagonal are never stored or read again.
    double li[T], lj[T];
#pragma unroll
    for (int r = 0; r < T; ++r) {
      const int i = ti * T + r;
      li[r] = (i > k && i < m) ? buf[i] * rl : 0.0;
    }
#pragma unroll
    for (int c = 0; c < T; ++c) {
      const int j = tj * T + c;
      lj[c] = (j > k && j < m) ? buf[j] * rl : 0.0;
    }
#pragma unroll
    for (int r = 0; r < T; ++r)
#pragma unroll
      for (int c = 0; c < T; ++c) a[r][c] = fma(-li[r], lj[c], a[r][c]);
    if (tj == k / T) {
      const int ck = k % T;
#pragma unroll
      for (int c = 0; c < T; ++c)
        if (c == ck) {
#pragma unroll
          for (int r = 0; r < T; ++r) a[r][c] = (ti * T + r == k) ? lkk : li[r];
        }
    }
  }
  __syncthreads();
  if constexpr (kCheck) {
    if (tid == 0) unsafe[blk] = bad ? 1 : 0;
    return;
  }
  // write the scaled lower triangle by subdiagonals
  const int64_t per = (int64_t)m * (m + 1) / 2;
#pragma unroll
  for (int r = 0; r < T; ++r)
#pragma unroll
    for (int c = 0; c < T; ++c) {
      const int i = ti * T + r, j = tj * T + c;
      if (i >= m || j > i) continue;
      const int dg = i - j;
      const int64_t pos = blk * per + (int64_t)dg * m - (int64_t)dg * (dg - 1) / 2 + j;
      const double v = a[r][c] * sc[i];
      Lbf[pos] = f32_to_bf16((float)v);
    }
}

hipError_t launch_chol_pack(fc_precond_s& pc, hipStream_t s, int32_t* unsafe) {
  const int m = pc.m;
  const int64_t nb = pc.n_blocks;
  if (nb == 0) return hipSuccess;
  dim3 g((unsigned)nb);
  const fc_problem_s& pb = *pc.pb;
#define FC_CHOL(GR, TT)                                                                     \
  if (unsafe)                                                                               \
    hipLaunchKernelGGL((k_chol_pack<GR, TT, true>), g, dim3(GR * GR), 0, s, pc.Q, m, pc.isd, \
                       block_nodes(pc), pc.block_elem, pc.nn, pc.bdim, nullptr, unsafe);       \
  else                                                                                      \
    hipLaunchKernelGGL((k_chol_pack<GR, TT, false>), g, dim3(GR * GR), 0, s, pc.Q, m,        \
                       pc.isd, block_nodes(pc), pc.block_elem, pc.nn, pc.bdim, pc.Lbf, nullptr)
  if (m <= 8) FC_CHOL(8, 1);
  else if (m <= 16) FC_CHOL(8, 2);
  else if (m <= 32) FC_CHOL(8, 4);
  else if (m <= 64) FC_CHOL(8, 8);
  else if (m <= 96) FC_CHOL(32, 3);
  else if (m <= 128) FC_CHOL(32, 4);
  else if (m <= 160) FC_CHOL(32, 5);
  else FC_CHOL(32, 6);
#undef FC_CHOL
  return hipGetLastError();
}

// ---------------------------------------------------- diagonal / fallback
__global__ void k_diag(const int32_t* __restrict__ rowptr, const int32_t* __restrict__ col,
                       const double* __restrict__ val, int bd, int64_t n_rows,
                       double* __restrict__ diag) {
  const int64_t row = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (row >= n_rows) return;
  const int32_t lo = rowptr[row], hi = rowptr[row + 1];
  int32_t l = lo, h = hi - 1, found = -1;
  while (l <= h) {
    int32_t mid = (l + h) >> 1;
    int32_t c = col[mid];
    if (c == row) {
      found = mid;
      break;
    }
    if (c < row) l = mid + 1;
    else h = mid - 1;
  }
  const int64_t L = hi - lo;
  for (int c = 0; c < bd; ++c)
    diag[row * bd + c] =
        found >= 0 ? val[(int64_t)lo * bd * bd + (int64_t)(c * bd + c) * L + (found - lo)] : 0.0;
}

// Diagonals of the local inverses in the layout of the block outputs.
__global__ __launch_bounds__(256) void k_block_diag(const double* __restrict__ Q, int m,
                                                    const FastDiv dm, uint32_t total,
                                                    double* __restrict__ d) {
  const uint32_t t = blockIdx.x * 256 + threadIdx.x;
  if (t >= total) return;
  const uint32_t blk = fdiv(t, dm);
  const int i = (int)(t - blk * (uint32_t)m);
  d[t] = Q[(int64_t)blk * sym_block_stride_dev(m) + sym_offset(0, i, m)];
}

// Algorithm 1 diagonal scaling: S_ll == 0 -> 1/A_ll (only where A_ll > 0).
// S_ll is the pull of the blocks' diagonals d.
template <bool kLat>
__global__ __launch_bounds__(256) void k_fallback(
    const double* __restrict__ d, const int32_t* __restrict__ inv_ptr,
    const int32_t* __restrict__ inv_idx, const double* __restrict__ diag, int m, int bd,
    const FastDiv dbd, const PullLattice L, uint32_t n_dofs, double* __restrict__ fb,
    unsigned long long* __restrict__ count) {
  const uint32_t i = blockIdx.x * 256 + threadIdx.x;
  if (i >= n_dofs) return;
  const uint32_t node = fdiv(i, dbd);
  const int c = (int)(i - node * (uint32_t)bd);
  double s;
  if constexpr (kLat) {
    double v[8];
    pull_lattice_load(d, L, m, bd, node, c, v);
    s = pull_sum8(v);
  } else {
    s = pull_mapped_sum(d, inv_ptr, inv_idx, node, c);
  }
  const double a = diag[i];
  const bool fall = (s == 0.0) && (a > 0.0);
  fb[i] = fall ? 1.0 / a : 0.0;
  if (fall) atomicAdd(count, 1ull);
}

// ------------------------------------------------------ node-to-block map
// Counted, scanned and filled on the device: on the host the two passes over
// (block, node) pairs and the upload took 4 ms at 48^3 cells, p = 2 (3.0M
// pairs), as long as all kernels of the build.  Entries land in the order of
// the atomics and are then sorted per node, so the map does not depend on it.
__global__ void k_map_count(const int32_t* __restrict__ nodes,
                            const int32_t* __restrict__ block_elem, int nn, int64_t total,
                            int32_t* __restrict__ count) {
  for (int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; t < total;
       t += (int64_t)gridDim.x * blockDim.x) {
    const int64_t b = t / nn;
    const int32_t node = nodes[(int64_t)block_elem[b] * nn + (t - b * nn)];
    if (node >= 0) atomicAdd(count + node, 1);
  }
}

// Exclusive scan of runs of 1,024 entries: pass 0 leaves the runs' sums, one
// workgroup scans those (pass 1), pass 2 writes the offsets (and zeroes the
// counts, which become fill positions).
__device__ __forceinline__ int32_t scan256(int32_t v, int32_t* lds /* 4 */) {
  const int l = threadIdx.x % 64, w = threadIdx.x / 64;
  int32_t x = v;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const int32_t y = __shfl_up(x, o, 64);
    if (l >= o) x += y;
  }
  __syncthreads();
  if (l == 63) lds[w] = x;
  __syncthreads();
  for (int k = 0; k < w; ++k) x += lds[k];
  return x;   // inclusive
}

template <int kPass>
__global__ __launch_bounds__(256) void k_map_scan(int32_t* __restrict__ count, int64_t n,
                                                  int32_t* __restrict__ sums, int nruns,
                                                  int32_t* __restrict__ ptr) {
  __shared__ int32_t lds[4];
  if constexpr (kPass == 1) {
    int32_t carry = 0;
    for (int r0 = 0; r0 < nruns; r0 += 256) {
      const int r = r0 + threadIdx.x;
      const int32_t v = r < nruns ? sums[r] : 0;
      const int32_t x = scan256(v, lds);
      if (r < nruns) sums[r] = carry + x - v;
      carry += lds[0] + lds[1] + lds[2] + lds[3];
      __syncthreads();
    }
  } else {
    const int64_t i0 = (int64_t)blockIdx.x * 1024 + threadIdx.x * 4;
    int32_t v[4], t = 0;
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      v[u] = i0 + u < n ? count[i0 + u] : 0;
      t += v[u];
    }
    const int32_t x = scan256(t, lds);
    if constexpr (kPass == 0) {
      if (threadIdx.x == 255) sums[blockIdx.x] = x;
    } else {
      int32_t o = sums[blockIdx.x] + x - t;
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        if (i0 + u < n) {
          ptr[i0 + u] = o;
          count[i0 + u] = 0;
        }
        o += v[u];
      }
    }
  }
}

__global__ void k_map_fill(const int32_t* __restrict__ nodes,
                           const int32_t* __restrict__ block_elem, int nn, int m, int bd,
                           int64_t total, const int32_t* __restrict__ ptr,
                           int32_t* __restrict__ fill, int32_t* __restrict__ idx) {
  for (int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; t < total;
       t += (int64_t)gridDim.x * blockDim.x) {
    const int64_t b = t / nn;
    const int a = (int)(t - b * nn);
    const int32_t node = nodes[(int64_t)block_elem[b] * nn + a];
    if (node >= 0) idx[ptr[node] + atomicAdd(fill + node, 1)] = (int32_t)(b * m + a * bd);
  }
}

__global__ __launch_bounds__(256) void k_map_sort(const int32_t* __restrict__ ptr, int64_t n_nodes,
                                                  int32_t* __restrict__ idx) {
  const int64_t node = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (node >= n_nodes) return;
  const int32_t lo = ptr[node], hi = ptr[node + 1];
  for (int32_t e = lo + 1; e < hi; ++e) {
    const int32_t v = idx[e];
    int32_t k = e;
    for (; k > lo && idx[k - 1] > v; --k) idx[k] = idx[k - 1];
    idx[k] = v;
  }
}

__global__ void k_zero_i32(int32_t* __restrict__ a, int64_t n) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * blockDim.x)
    a[i] = 0;
}

int64_t map_scan_blocks(int64_t n) { return (n + 1023) / 1024; }

hipError_t launch_build_map(const fc_precond_s& pc, int64_t n_nodes, int32_t* ptr, int32_t* idx,
                            int32_t* work, int32_t* sums, hipStream_t s) {
  const int64_t n = n_nodes + 1, total = pc.n_blocks * pc.nn;
  const int nruns = (int)map_scan_blocks(n);
  const dim3 b(256), runs((unsigned)nruns);
  const dim3 g((unsigned)std::min<int64_t>((total + 255) / 256, 8192));
  const dim3 gz((unsigned)std::min<int64_t>((n + 255) / 256, 1024));
  if (total == 0) {   // no block: every node's entries are empty
    hipLaunchKernelGGL(k_zero_i32, gz, b, 0, s, ptr, n);
    return hipGetLastError();
  }
  hipLaunchKernelGGL(k_zero_i32, gz, b, 0, s, work, n);
  hipLaunchKernelGGL(k_map_count, g, b, 0, s, block_nodes(pc), pc.block_elem, pc.nn, total, work);
  hipLaunchKernelGGL(k_map_scan<0>, runs, b, 0, s, work, n, sums, nruns, ptr);
  hipLaunchKernelGGL(k_map_scan<1>, dim3(1), b, 0, s, work, n, sums, nruns, ptr);
  hipLaunchKernelGGL(k_map_scan<2>, runs, b, 0, s, work, n, sums, nruns, ptr);
  hipLaunchKernelGGL(k_map_fill, g, b, 0, s, block_nodes(pc), pc.block_elem, pc.nn, pc.m, pc.bdim,
                     total, ptr, work, idx);
  hipLaunchKernelGGL(k_map_sort, dim3((unsigned)((n_nodes + 255) / 256)), b, 0, s, ptr, n_nodes,
                     idx);
  return hipGetLastError();
}

__global__ void k_cast_f32(const double* __restrict__ in, float* __restrict__ out, int64_t n) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * blockDim.x)
    out[i] = (float)in[i];
}

// ---------------------------------------------------------- launchers
hipError_t launch_block_extract(const fc_precond_s& pc, const int32_t* list, int64_t b0,
                                int64_t count, double* dense, hipStream_t s) {
  if (count == 0) return hipSuccess;
  const DeviceBsr& A = pc.pb->A;
  hipLaunchKernelGGL(k_block_extract, dim3((unsigned)count), dim3(256), 0, s, A.rowptr, A.col,
                     A.val, block_nodes(pc), pc.block_elem, list, b0, pc.nn, pc.bdim, pc.m, dense);
  return hipGetLastError();
}

// P_B of the listed blocks (dense) into their places in Q
__global__ __launch_bounds__(256) void k_pack_list(const double* __restrict__ P,
                                                   const int32_t* __restrict__ list, int m,
                                                   double* __restrict__ Q) {
  const double* Pb = P + blockIdx.x * (int64_t)m * m;
  double* Qb = Q + list[blockIdx.x] * sym_block_stride_dev(m);
  for (int t = threadIdx.x; t < (m / 2 + 1) * m; t += 256) {
    const int k = t / m, i = t - k * m;
    const int j = i + k < m ? i + k : i + k - m;
    Qb[sym_offset(k, i, m)] = Pb[(int64_t)i * m + j];
  }
}

hipError_t launch_jacobi(fc_precond_s& pc, const int32_t* sel, int64_t count, double* dense,
                         double* work, int32_t* dropped, hipStream_t s) {
  if (count == 0) return hipSuccess;
  const int m = pc.m;
  hipError_t e = launch_block_extract(pc, sel, 0, count, dense, s);
  if (e != hipSuccess) return e;
  // one wave per block for small blocks, four waves otherwise
  const int threads = m <= 32 ? 64 : 256;
  const size_t lds = sizeof(double) * 2 * (size_t)m * (m + 1);
  if (!jacobi_needs_work(m)) {
    (void)hipFuncSetAttribute((const void*)k_jacobi_pinv<true>,
                              hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    hipLaunchKernelGGL(k_jacobi_pinv<true>, dim3((unsigned)count), dim3(threads), lds, s,
                       dense, m, sel, nullptr, pc.eps, pc.stabilize, dropped);
  } else {
    if (!work) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_jacobi_pinv<false>, dim3((unsigned)count), dim3(threads), 0, s,
                       dense, m, sel, work, pc.eps, pc.stabilize, dropped);
  }
  hipLaunchKernelGGL(k_pack_list, dim3((unsigned)count), dim3(256), 0, s, dense, sel, m, pc.Q);
  return hipGetLastError();
}

bool jacobi_needs_work(int m) {
  const size_t lds = sizeof(double) * 2 * (size_t)m * (m + 1);
  int dev = 0, limit = 0;
  (void)hipGetDevice(&dev);
  if (hipDeviceGetAttribute(&limit, hipDeviceAttributeMaxSharedMemoryPerBlock, dev) != hipSuccess)
    limit = 65536;
  const size_t static_lds = 6 * 1024;   // rotation tables and reductions
  return !(m <= 64 && lds + static_lds <= (size_t)limit);
}

bool sweep_reads_lattice(const fc_precond_s& pc) {
  return pc.pb->cells.dim > 0 && pc.pb->A.lat.dim > 0 && !pc.bnodes;
}

// One instance for each of 9, 24, 25 and 27, and one for every other size up to 8,
// 16, 32 and 64 (padded with rows of the identity: plane elasticity's 18 and 50
// among them).
template <bool kLat>
static void sweep_small(const BlockSrc& S, const fc_precond_s& pc, int64_t b0, int64_t count,
                        int32_t* need_eig, hipStream_t s) {
  const int m = pc.m;
#define FC_SWEEP(W, KM)                                                                        \
  hipLaunchKernelGGL((k_sweep_small<W, KM, kLat>),                                             \
                     dim3((unsigned)((count + 256 / W - 1) / (256 / W))), dim3(256), 0, s, S,  \
                     b0, count, m, pc.eps, pc.Q, need_eig)
  switch (m) {
    case 9: FC_SWEEP(16, 9); break;
    case 24: FC_SWEEP(32, 24); break;
    case 25: FC_SWEEP(32, 25); break;
    case 27: FC_SWEEP(32, 27); break;
    default:
      if (m <= 8) FC_SWEEP(16, 8);
      else if (m <= 16) FC_SWEEP(16, 16);
      else if (m <= 32) FC_SWEEP(32, 32);
      else FC_SWEEP(64, 64);
  }
#undef FC_SWEEP
}

template <bool kLat>
static void sweep_large(const BlockSrc& S, const fc_precond_s& pc, int64_t b0, int64_t count,
                        int32_t* need_eig, hipStream_t s) {
  const dim3 g((unsigned)count);
#define FC_SWEEP(NT, NW)                                                                       \
  hipLaunchKernelGGL((k_sweep_large<NT, NW, kLat>), g, dim3(64 * NW), 0, s, S, b0, pc.m,       \
                     pc.eps, pc.stabilize, pc.Q, need_eig)
  // waves per block: sixteen where the tiles of one workgroup fill a compute
  // unit's registers (1.8 against 2.8 ms with eight at 192), fewer where several
  // workgroups fit and hide each other's diagonal tiles (m = 81, 8,000 blocks:
  // four waves 0.51 ms, eight 0.68, two 1.02; m = 125, 4,096 blocks: eight 0.57
  // ms, four 0.72, twelve 0.85)
  if (pc.m <= 96) FC_SWEEP(6, 4);
  else if (pc.m <= 128) FC_SWEEP(8, 8);
  else if (pc.m <= 160) FC_SWEEP(10, 16);
  else FC_SWEEP(12, 16);
#undef FC_SWEEP
}

hipError_t launch_sweep(fc_precond_s& pc, int64_t b0, int64_t count, double* dense,
                        int32_t* need_eig, hipStream_t s) {
  if (count == 0) return hipSuccess;
  const fc_problem_s& pb = *pc.pb;
  const BlockSrc S{pb.A.val, dense,  pc.block_elem, pb.A.lat, pb.cells,
                   make_fastdiv((uint32_t)pc.bdim), pc.bdim};
  const bool lat = sweep_reads_lattice(pc);
  if (!lat) {
    hipError_t e = launch_block_extract(pc, nullptr, b0, count, dense, s);
    if (e != hipSuccess) return e;
  }
  if (pc.m > 192) return hipErrorInvalidValue;
  if (pc.m <= 64) {
    if (lat) sweep_small<true>(S, pc, b0, count, need_eig, s);
    else sweep_small<false>(S, pc, b0, count, need_eig, s);
  } else {
    if (lat) sweep_large<true>(S, pc, b0, count, need_eig, s);
    else sweep_large<false>(S, pc, b0, count, need_eig, s);
  }
  return hipGetLastError();
}

hipError_t launch_diag(const fc_problem_s& pb, hipStream_t s) {
  const int64_t n = pb.A.n_rows;
  if (n == 0) return hipSuccess;
  hipLaunchKernelGGL(k_diag, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s,
                     pb.A.rowptr, pb.A.col, pb.A.val, pb.bdim, n, pb.diag);
  return hipGetLastError();
}

hipError_t launch_fallback(const fc_problem_s& pb, fc_precond_s& pc,
                           unsigned long long* d_count, hipStream_t s) {
  const uint32_t n = (uint32_t)pb.n_dofs;
  const int64_t total = pc.n_blocks * pc.m;
  const dim3 g((n + 255) / 256), b(256);
  const FastDiv dbd = make_fastdiv((uint32_t)pc.bdim);
  if (total > 0)
    hipLaunchKernelGGL(k_block_diag, dim3((unsigned)((total + 255) / 256)), b, 0, s, pc.Q, pc.m,
                       make_fastdiv((uint32_t)pc.m), (uint32_t)total, pc.y);
  if (pc.lat.dim > 0)
    hipLaunchKernelGGL(k_fallback<true>, g, b, 0, s, pc.y, pc.inv_ptr, pc.inv_idx, pb.diag, pc.m,
                       pc.bdim, dbd, pc.lat, n, pc.fallback, d_count);
  else
    hipLaunchKernelGGL(k_fallback<false>, g, b, 0, s, pc.y, pc.inv_ptr, pc.inv_idx, pb.diag, pc.m,
                       pc.bdim, dbd, pc.lat, n, pc.fallback, d_count);
  return hipGetLastError();
}

// FP32 copy of the matrix values, same layout (k_cast_f32 above)
hipError_t launch_cast_matrix(const DeviceBsr& A, hipStream_t s) {
  const int64_t n = A.nnzb * A.bdim * A.bdim;
  if (!A.val32 || n == 0) return hipSuccess;
  hipLaunchKernelGGL(k_cast_f32, dim3(4096), dim3(256), 0, s, A.val, A.val32, n);
  return hipGetLastError();
}

}  // namespace fc
