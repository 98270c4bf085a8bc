// Preconditioner set-up launchers.
#pragma once
#include "fc_internal.h"

namespace fc {
// A_B of `count` blocks, listed or b0, b0 + 1, .., into dense [count][m][m]
hipError_t launch_block_extract(const fc_precond_s& pc, const int32_t* list, int64_t b0,
                                int64_t count, double* dense, hipStream_t s);
// Pseudo-inverses of the listed blocks by eigen-decomposition into pc.Q; dense:
// [count][m][m] scratch, work: [count][2][m][m] where jacobi_needs_work
hipError_t launch_jacobi(fc_precond_s& pc, const int32_t* sel, int64_t count, double* dense,
                         double* work, int32_t* dropped, hipStream_t s);
// Blocks of a launch of it, of `count`.  Blocks take sweeps of their own number, so
// every launch ends in a tail: up to m = 64 as many as 256 MB of dense copies hold.
// Unstabilised inverse, 110,592 blocks of 27: 47.8 ms, 57.7 in launches of 2,048;
// 13,824 of 8: 0.34 / 0.60.  Above 64 a block fills a compute unit for long enough:
// 2,048, which at 192 take 0.6 GB of dense copies and 1.2 GB of work.
inline int64_t jacobi_chunk(int m, int64_t count) {
  const int64_t most = m <= 64 ? (int64_t(1) << 25) / ((int64_t)m * m) : 2048;
  return most < count ? most : count;
}
// true when the Jacobi eigen path keeps its blocks in global memory
bool jacobi_needs_work(int m);
// Certified direct inverses of blocks b0 .. b0 + count - 1 into pc.Q; blocks
// that fail are flagged.  dense: [count][m][m] scratch unless
// sweep_reads_lattice(pc)
hipError_t launch_sweep(fc_precond_s& pc, int64_t b0, int64_t count, double* dense,
                        int32_t* need_eig, hipStream_t s);
bool sweep_reads_lattice(const fc_precond_s& pc);
// Scaled Cholesky factors of the local inverses in BF16 into pc.Lbf (needs
// pc.isd); with `unsafe` instead only flag the blocks whose FP32-rounded
// scaled inverse is not safely positive definite
hipError_t launch_chol_pack(fc_precond_s& pc, hipStream_t s, int32_t* unsafe = nullptr);
hipError_t launch_diag(const fc_problem_s& pb, hipStream_t s);
// The node-to-block map: ptr [n_nodes + 1] and idx (room for n_blocks * nn
// entries), the entries of a node in block order.  work: [n_nodes + 1] and the
// sums of map_scan_blocks(n_nodes + 1) runs.
int64_t map_scan_blocks(int64_t n);
hipError_t launch_build_map(const fc_precond_s& pc, int64_t n_nodes, int32_t* ptr, int32_t* idx,
                            int32_t* work, int32_t* sums, hipStream_t s);
// Algorithm 1's diagonal scaling (uses pc.y for the blocks' diagonals)
hipError_t launch_fallback(const fc_problem_s& pb, fc_precond_s& pc,
                           unsigned long long* d_count, hipStream_t s);
// A.val32 = FP32 copy of A.val (same layout)
hipError_t launch_cast_matrix(const DeviceBsr& A, hipStream_t s);
}  // namespace fc
