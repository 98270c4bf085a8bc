// Internal structures of libfc shared by the HIP translation units.
#pragma once
#include <hip/hip_runtime.h>

#include <cstdint>
#include <string>
#include <vector>

#include "fc.h"

namespace fc {

void set_error(const std::string& msg);

#define FC_HIP(call)                                                         \
  do {                                                                       \
    hipError_t e_ = (call);                                                  \
    if (e_ != hipSuccess) {                                                  \
      ::fc::set_error(std::string(#call) + ": " + hipGetErrorString(e_));    \
      return FC_E_DEVICE;                                                    \
    }                                                                        \
  } while (0)

// Scalars of one PCG run kept on the device so the iteration never waits on
// the host.  Dots are reduced per workgroup into `partial`, which a later
// kernel sums in a fixed order, so every run is bitwise reproducible.  Kernels
// of many workgroups derive alpha and beta from the partials themselves; only
// their first workgroup writes scalars, and none that the same kernel reads: the
// waves of a workgroup that starts late would otherwise part at the stop test.
// So the stop has two flags.  The kernels that take alpha test `done` and write
// `halt`, those that take beta test `halt` and write `done`, each passing on what
// it found set: the products between beta and alpha test `done`, the pull between
// alpha and beta `halt`, and what may run in either place both.
struct CgScalars {
  double rz;        // (r, z) of the iterate the step starts from
  double pq;        // (p, A p)
  double alpha, beta;
  double zz;        // (z, z) of the newest z
  double rr;        // (r, r) of the newest r
  double crit;      // newest relative criterion
  double tol;
  int64_t iter;     // products with A done
  int64_t maxit;
  int32_t done;     // 0 running, 1 converged, 2 maxit, 3 breakdown, 4 non-finite
  int32_t halt;     // the same between a step's alpha and its beta
  double rzn;       // (r, z) of the newest iterate (rz of the next step)
  double zn0, rn0;  // ||z_0||, ||r_0||: the denominators of the stop test
  double* history;  // optional per-iteration criterion
  int32_t stop;     // FC_STOP_*
  int32_t pad;
};
static_assert(sizeof(CgScalars) == 128, "one cache line each in a batch's array");

// Tensor-product lattice behind a matrix assembled from a problem
// description (dim = 0 otherwise): the block columns of every row are the
// lattice box spanned by the supports through the row's node, so they can
// be computed instead of read.
// Division of 32-bit unsigned numbers by an invariant d (Granlund and
// Montgomery, division by invariant integers using multiplication): with
// l = ceil(log2 d) and m = floor(2^32 (2^l - d) / d) + 1, the quotient is
// (t + ((n - t) >> min(l, 1))) >> max(l - 1, 0), t = (m n) >> 32.
struct FastDiv {
  uint32_t d = 1, m = 1, s1 = 0, s2 = 0;
};

inline FastDiv make_fastdiv(uint32_t d) {
  FastDiv f;
  f.d = d;
  uint32_t l = 0;
  while ((uint64_t(1) << l) < d) ++l;
  f.m = (uint32_t)(((uint64_t(1) << 32) * ((uint64_t(1) << l) - d)) / d + 1);
  f.s1 = l > 0 ? 1u : 0u;
  f.s2 = l > 0 ? l - 1 : 0u;
  return f;
}

struct LatticeInfo {
  int32_t dim = 0, n1 = 0, p = 0;
  FastDiv dn1, dp;   // division by n1 and by p
};

inline LatticeInfo make_lattice_info(int32_t dim, int32_t n1, int32_t p) {
  LatticeInfo l;
  l.dim = dim;
  l.n1 = n1;
  l.p = p;
  l.dn1 = make_fastdiv((uint32_t)n1);
  l.dp = make_fastdiv((uint32_t)p);
  return l;
}

// Lattice of the element blocks when every cell of a problem set up from a
// description is a block, in cell order (dim = 0 otherwise): the pull then
// finds the blocks holding a node from its lattice indices instead of the
// node-to-block map.
struct PullLattice {
  int32_t dim = 0, n = 0, p = 0, n1 = 0;
  FastDiv dn, dp, dp1, dn1;   // division by n, p, p + 1 and n1
};

inline PullLattice make_pull_lattice(int32_t dim, int32_t n, int32_t p) {
  PullLattice l;
  l.dim = dim;
  l.n = n;
  l.p = p;
  l.n1 = p * n + 1;
  l.dn = make_fastdiv((uint32_t)n);
  l.dp = make_fastdiv((uint32_t)p);
  l.dp1 = make_fastdiv((uint32_t)(p + 1));
  l.dn1 = make_fastdiv((uint32_t)l.n1);
  return l;
}

// A slice of the sliced copy: 64 rows of class cls (bit d: the indices along
// direction d are interior vertices), rows 64 chunk .. of its enumeration.  Its
// entries are stored in pairs: entries 2j and 2j + 1 of lane l at
// val[off + 128 j + 2 l] and the next word, an odd last entry alone at
// off + 128 j + l (zero for lanes past the class's end).
struct SellSlice {
  int64_t off;
  int32_t cls, chunk;
};

struct SellView {
  const double* val = nullptr;
  const SellSlice* slices = nullptr;
  int32_t n_slices = 0, dim = 0, n1 = 0;
  uint32_t nv = 0, nn = 0;   // interior vertices and other indices per direction
  FastDiv dv, dn;            // division by nv and nn
};

struct DeviceBsr {
  int32_t bdim = 1;
  int64_t n_rows = 0;      // block rows
  int64_t nnzb = 0;
  int32_t max_row = 0;     // longest block row
  int32_t group = 0;       // SpMV lanes per block row, fixed at set-up from the row lengths
  LatticeInfo lat;         // set when the columns were verified to be the lattice box
  int32_t* rowptr = nullptr;
  int32_t* col = nullptr;
  double* val = nullptr;   // row-SoA layout
  float* val32 = nullptr;  // optional FP32 copy, same layout
  // mixed-precision products: block rows read in FP64 (rows_hi) and from
  // the FP32 copy (rows_lo), ascending
  int32_t* rows_hi = nullptr;
  int32_t* rows_lo = nullptr;
  int64_t n_hi = 0, n_lo = 0;
  // Sliced copy of a scalar lattice matrix (degree p <= 4; spmv_dev.h)
  double* sell_val = nullptr;
  SellSlice* sell_slices = nullptr;
  int64_t n_slices = 0;
  int32_t sell_nv = 0;     // interior vertices per direction
};

inline SellView sell_view(const DeviceBsr& A) {
  SellView v;
  v.val = A.sell_val;
  v.slices = A.sell_slices;
  v.n_slices = (int32_t)A.n_slices;
  v.dim = A.lat.dim;
  v.n1 = A.lat.n1;
  v.nv = (uint32_t)A.sell_nv;
  v.nn = (uint32_t)(A.lat.n1 - A.sell_nv);
  v.dv = make_fastdiv(v.nv > 0 ? v.nv : 1);
  v.dn = make_fastdiv(v.nn);
  return v;
}

// hipMalloc for everything else the library holds: out of memory, the buffers kept
// for reuse are given back first.
hipError_t dev_malloc(void** p, size_t bytes);
template <class T>
hipError_t dev_malloc(T** p, size_t bytes) {
  return dev_malloc(reinterpret_cast<void**>(p), bytes);
}

// Device memory that outlives no problem but is reused from one preconditioner
// to the next (dev_pool.hip).  pool_free: idle says that nothing on the device uses
// p any more; without it p is not kept, or not before device_idle() has succeeded.
hipError_t pool_malloc(void** p, size_t bytes);
void pool_free(void* p, bool idle);
void pool_problem_created();
void pool_problem_destroyed();

// The current device's stream for copies of calls that take none (made once, held
// until the process ends).  Work on the legacy stream would break every graph
// capture in progress in the process, and fail itself.
hipError_t own_stream(hipStream_t* s);
// Copy on it, done when this returns.  Waits for no other stream.
hipError_t copy_now(void* dst, const void* src, size_t bytes, hipMemcpyKind kind);

// Waits for all work on the device; graph captures in progress on other threads
// (and, in relaxed mode, on this one) go on.
hipError_t device_idle();

// Per-workgroup (p, q) partials a kernel derives the step length from; np = 0:
// the step length is in CgScalars already.
struct AlphaIn {
  const double* partial = nullptr;
  int np = 0;
};

struct SolverWs;
void solver_ws_destroy(SolverWs* ws, bool idle);   // idle: as pool_free
struct CoarseCtx;
void coarse_destroy(CoarseCtx* c);

}  // namespace fc

struct fc_problem_s {
  int device = 0;
  int32_t dim = 0, p = 0, n = 0;   // lattice (0 when built from a matrix)
  int32_t bdim = 1, nn = 0, m = 0;
  int64_t n_nodes = 0, n_dofs = 0, n_el = 0;
  fc::DeviceBsr A;
  double* rhs = nullptr;           // [n_dofs]
  int32_t* elem_nodes = nullptr;   // [n_el*nn]
  std::vector<double> eta;         // host copy [n_el]
  std::vector<int32_t> elem_nodes_host;
  double* diag = nullptr;          // A_ll [n_dofs]
  fc::PullLattice cells;           // set when the elements are a lattice's cells, in order
};

struct fc_precond_s {
  fc_problem pb = nullptr;
  int device = 0;
  int32_t m = 0, nn = 0, bdim = 1;
  int64_t n_blocks = 0;
  int32_t block_kind = FC_BLOCK_ELEMENT;
  int32_t* block_elem = nullptr;   // [n_blocks] element of each block (patch: its index)
  int32_t* bnodes = nullptr;       // vertex patches: [n_blocks][nn] node lists, -1 padding
  double* Q = nullptr;             // FP64 local inverses, wrapped-diagonal symmetric storage
  float* Q32 = nullptr;            // optional FP32 copy of D^1/2 P D^1/2, same storage
  int32_t* unsafe32 = nullptr;     // blocks whose FP32 copy is not safely positive
  int32_t* unsafe_flag32 = nullptr; // the same as one flag per block
  int64_t n_unsafe32 = 0;          //   (applied from the FP64 copy instead)
  uint16_t* Lbf = nullptr;         // optional BF16 scaled Cholesky factors
  double* isd = nullptr;           // [n_dofs] 1/sqrt(A_ll), scaling of Q32/Lbf
  int32_t* inv_ptr = nullptr;      // [n_nodes+1] node -> (block, local node); null where
  int32_t* inv_idx = nullptr;      // `lat` is set; entries: block*m + local_node*bdim
  double* fallback = nullptr;      // [n_dofs] 1/A_ll where S_ll = 0, else 0
  fc::PullLattice lat;             // set when every cell is a block (lattice pull)
  double* y = nullptr;             // [n_blocks*m] block outputs (workspace)
  int64_t n_fallback = 0, n_eig = 0, n_dropped = 0;
  std::vector<int32_t> dropped;    // host copy: eigenvalues dropped per block
  double eps = 1e-13;
  int32_t stabilize = 1;
  fc::SolverWs* ws = nullptr;      // PCG workspace, created on first solve
  fc::CoarseCtx* coarse = nullptr; // learned coarse correction, when attached
};

namespace fc {

// Node lists of the preconditioner's blocks: the element lists of the
// problem, or the patch lists of a vertex-patch preconditioner.
inline const int32_t* block_nodes(const fc_precond_s& pc) {
  return pc.bnodes ? pc.bnodes : pc.pb->elem_nodes;
}

// ---- launchers (each returns hipSuccess or the first launch error) ----
// y = A x  (and optionally partial dots (x, y) per workgroup)
hipError_t launch_spmv(const DeviceBsr& A, const double* x, double* y,
                       hipStream_t s);
// lanes per block row of A's products, from its mean row length
int spmv_group_for(const DeviceBsr& A);
// verify on the device that A's columns are the lattice boxes of (dim, n1,
// p); if so record it in A.lat, so the SpMV computes columns instead of
// reading them
hipError_t spmv_enable_lattice(DeviceBsr& A, int dim, int n1, int p, hipStream_t s);

// z = S r
hipError_t launch_schwarz_apply(const fc_precond_s& pc, const double* r,
                                double* z, hipStream_t s);

// drop the captured solver chunk (its kernels hold buffers about to change)
void solver_invalidate_graph(fc_precond_s& pc);

}  // namespace fc
