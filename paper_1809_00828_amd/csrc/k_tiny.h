// CG steps of a tiny problem in one workgroup (k_tiny.hip).
#pragma once
#include "fc_internal.h"

namespace fc {
// Bytes of matrix and local inverses a step reads, at most.  Measured, in us a step
// against separate launches: 2-D p = 3, 0.29 MB 7.3 / 15.3, 0.74 MB 13.1 / 15.3;
// p = 4, 0.45 MB 10.8 / 16.2, 1.0 MB 20.4 / 16.1; 3-D p = 1, 0.72 MB 15.2 / 16.7;
// p = 2, 0.47 MB 11.9 / 19.5, 0.9 MB 19.6 / 19.8.
constexpr size_t kTinyBytes = size_t(768) << 10;
// Steps of a launch, in units of check_every and at most (16 ms): the stop is tested
// on the device.
constexpr int kTinyChunks = 4, kTinySteps = 1024;
// FP64 steps of pc can run in one workgroup.
bool tiny_fits(const fc_precond_s& pc);
// Up to `steps` steps from r, p and sc (after the start); stops like the others.
hipError_t launch_tiny_steps(const fc_precond_s& pc, double* x, double* r, double* p, double* z,
                             CgScalars* sc, int steps, hipStream_t s);
}  // namespace fc
