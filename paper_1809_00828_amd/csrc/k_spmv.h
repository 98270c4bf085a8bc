// SpMV launch helpers used by the solver.
#pragma once
#include "fc_internal.h"

namespace fc {
// There is a sliced copy; the FP64 product alone takes it.
bool spmv_has_sell(const DeviceBsr& A);
bool spmv_uses_sell(const DeviceBsr& A);
// A step's p update may join the sliced product (launch_spmv_beta); the product of such
// steps, and of those that cannot join, takes the sliced copy (routes.h).
bool spmv_step_joins(const DeviceBsr& A);
bool spmv_step_uses_sell(const DeviceBsr& A);
// (p, q) partials the product can leave, one per workgroup; 0: it has too many
// workgroups, and the dot is a pass of its own.
int spmv_dot_blocks(const DeviceBsr& A, bool sell);
// q = A p on the sliced copy or the rows, with one partial (p, q) per workgroup in
// partial[0 .. spmv_dot_blocks(A, sell)) unless partial is null (skipped when sc->done is
// set)
hipError_t launch_spmv_pq(const DeviceBsr& A, const double* p, double* q, CgScalars* sc,
                          double* partial, bool sell, hipStream_t s);
// q = A p on the sliced copy with p = z + beta p_old, stored in p_new; beta from the
// pull's np partial sets, (p, q) partials as above.
hipError_t launch_spmv_beta(const DeviceBsr& A, const double* z, const double* p_old,
                            double* p_new, double* q, CgScalars* sc, double* partial,
                            const double* sets, int np, hipStream_t s);
// q = A p with the rows A.rows_hi from the FP64 values and p, and the rows
// A.rows_lo from the FP32 copy and p32 = fl32(p) (skipped when sc->done is
// set)
hipError_t launch_spmv_mixed(const DeviceBsr& A, const double* p, const float* p32, double* q,
                             const CgScalars* sc, hipStream_t s);
}  // namespace fc
