// CG steps of a tiny problem in one workgroup (k_tiny.hip).
#pragma once
#include "fc_internal.h"

namespace fc {
// Steps of a launch, in units of check_every and at most (16 ms): the stop is tested
// on the device.
constexpr int kTinyChunks = 4, kTinySteps = 1024;
// FP64 steps of pc can run in one workgroup (sizes: tiny_sizes, routes.h).
bool tiny_fits(const fc_precond_s& pc);
// Up to `steps` steps from r, p and sc (after the start); stops like the others.
hipError_t launch_tiny_steps(const fc_precond_s& pc, double* x, double* r, double* p, double* z,
                             CgScalars* sc, int steps, hipStream_t s);
}  // namespace fc
