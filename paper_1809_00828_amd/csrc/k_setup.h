// Preconditioner set-up launchers.
#pragma once
#include "fc_internal.h"

namespace fc {
hipError_t launch_jacobi(fc_precond_s& pc, const int32_t* sel, int64_t count,
                         double* work, int32_t* dropped, hipStream_t s);
// true when the Jacobi eigen path keeps its blocks in global memory
bool jacobi_needs_work(int m);
hipError_t launch_sweep(fc_precond_s& pc, int32_t* need_eig, hipStream_t s);
// the same certified sweep for m <= 64 (one wave per block)
hipError_t launch_sweep_small(fc_precond_s& pc, int32_t* need_eig, hipStream_t s);
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
