/*
 * linear_testing.h -- host-only view of what a call on a linear model launches, for the library's tests.
 * Not part of the inference ABI (include/linear.h); no GPU needed.
 */
#ifndef LINEAR_TESTING_H_
#define LINEAR_TESTING_H_

#include <stdint.h>

#include "linear.h"

#ifdef __cplusplus
extern "C" {
#endif

typedef struct linear_launch_t {
    int32_t whole_rows; /* 1: whole rows of a tile in LDS, 0: chunks of 32 features */
    int32_t padded;     /* whole rows: the tile has padding */
    int32_t load_width; /* chunks: floats per load of X */
    int32_t once;       /* chunks: loads of X are non-temporal */
    int32_t lds_bytes;  /* dynamic LDS per workgroup */
    int32_t scores_past, labels_past; /* 1: stored past the L2 */
} linear_launch_t;

/*
 * The launch of a call on n_rows rows whose X, scores and labels are at these addresses (0: not asked for), on a device whose workgroups
 * may have `lds_limit` bytes of LDS.
 * Returns LINEAR_OK, LINEAR_EINVAL (null pointer, counts below 1) or LINEAR_ELIMIT.
 */
int linear_launch_shape(int32_t n_features, int32_t n_outputs, int64_t n_rows, uintptr_t x, uintptr_t scores,
                        uintptr_t labels, int64_t lds_limit, linear_launch_t *out);

#ifdef __cplusplus
}
#endif
#endif /* LINEAR_TESTING_H_ */
