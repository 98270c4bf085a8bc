// Schwarz apply launchers used by the solver.
#pragma once
#include "fc_internal.h"

namespace fc {
// Phase 1 only: y_B = P_B R_B (r - alpha q) for every block (q may be NULL,
// then r is gathered as is).  precision 0 = FP64, 1 = FP32, 2 = BF16 copy of
// the local inverses.  Skipped when sc->done is set (sc may be NULL).  With
// ai.np > 0 (schwarz_takes_alpha) every workgroup derives alpha from the (p, q)
// partials, and the first one stores it.
hipError_t launch_schwarz_phase1(const fc_precond_s& pc, int precision, const double* r,
                                 const double* q, CgScalars* sc, const AlphaIn ai, hipStream_t s);
// Whether the block products of this precision can derive alpha themselves.
bool schwarz_takes_alpha(const fc_precond_s& pc, int precision);
// Phase 2 only: z = sum_B R_B^T y_B + fallback * r.
hipError_t launch_schwarz_pull(const fc_precond_s& pc, const double* r, double* z,
                               hipStream_t s);
// Elements per block of the wrapped-diagonal symmetric layout, (m/2+1)*m.
int64_t sym_block_stride(int m);
// pc.Q32 = FP32 copy of pc.Q, diagonally scaled (needs pc.isd).
hipError_t launch_pack_f32(const fc_precond_s& pc, hipStream_t s);
// Whether the elements of pb are the cells of the lattice L, in order, with
// their nodes in the cells' local tensor order; synchronises s.
hipError_t schwarz_check_cells(const fc_problem_s& pb, const PullLattice L, bool* ok,
                               hipStream_t s);
// isd = 1/sqrt(diag(A)) (1 where the diagonal is not positive).
hipError_t launch_inv_sqrt_diag(const fc_problem_s& pb, double* isd, hipStream_t s);
}  // namespace fc
