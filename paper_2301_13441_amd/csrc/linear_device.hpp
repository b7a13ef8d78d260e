// Device-resident view of a linear model, passed by value to the kernel.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

#include "linear_plan.hpp"

namespace linear_impl {

enum { TRANSFORM = 255, SCORES_PAST = 256, LABELS_PAST = 512 };  // LinDev::finish

struct LinDev {
    const double *weight;  // [n_features rounded up to a multiple of 32][kp]: float64, zero-padded
    const double *bias;    // [kp]
    int32_t n_features, n_outputs, kp;
    int32_t finish;  // LINEAR_TRANSFORM_*, and per launch SCORES_PAST and LABELS_PAST: one register, of which many outputs spill some
    int32_t output;
    int64_t lds_limit;  // bytes of LDS that a workgroup may have
};

// Lets the kernels have `lds_limit` bytes of LDS on the current device.
hipError_t init_linear_kernels(int64_t lds_limit);

hipError_t launch_linear(const LinDev &m, const float *X, int64_t n_rows, float *scores, int32_t *labels,
                         hipStream_t stream);

}  // namespace linear_impl
