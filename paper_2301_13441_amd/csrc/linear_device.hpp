// Device-resident view of a linear model, passed by value to the kernel.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

#include "linear_plan.hpp"

namespace linear_impl {

struct LinDev {
    const double *weight;  // [n_features rounded up to a multiple of 32][kp]: float64, zero-padded
    const double *bias;    // [kp]
    int32_t n_features, n_outputs, kp;
    int32_t transform, output;
    int32_t scores_past, labels_past;  // set per launch (LinearPlan)
    int64_t lds_limit;  // bytes of LDS that a workgroup may have
};

// Lets the kernels have `lds_limit` bytes of LDS on the current device.
hipError_t init_linear_kernels(int64_t lds_limit);

hipError_t launch_linear(const LinDev &m, const float *X, int64_t n_rows, float *scores, int32_t *labels,
                         hipStream_t stream);

}  // namespace linear_impl
