// What a call on a linear model launches: kernel, width of its loads, cache policies.  Host code without HIP, so that the
// rules can be tested without a GPU (include/linear_testing.h).
#pragma once

#include <cstddef>
#include <cstdint>

namespace linear_impl {

constexpr int LANES = 64;
constexpr int CHUNK = 32;      // features per pass of the chunked kernel
constexpr int ROWS_WAVES = 2;  // waves per workgroup of the whole-row kernel
constexpr int PIECE = LANES * 4;  // floats that one load of the whole-row kernel brings to LDS
constexpr int PAD = 4;            // floats left free behind a piece in the padded form
constexpr int STEP = 16;          // features of a step of the padded form
constexpr int ROWS_MAX_FEATURES = 96, ROWS_MAX_OF_THREE = 104, ROWS_MAX_OF_TWO = 156;

// Column counts the kernels are instantiated for; a model uses the smallest one >= n_outputs.
inline int padded_outputs(int n_outputs)
{
    constexpr int sizes[] = {1, 2, 3, 4, 5, 6, 8, 10, 12, 16, 24, 32};
    for (int s : sizes)
        if (s >= n_outputs) return s;
    return 0;
}

// The whole-row kernel, or chunks.  Beyond 96 features multiples of 32 go by chunks, whose lines are whole; of the others
// those of which three workgroups fit a CU (up to 104 features) go by rows, and, with one output, those of which two do (us,
// chunks with the cache / rows: 100 features, one output 243 / 178, 5 classes 178 / 166; 130, one output 271 / 183; 112
// features, 5 classes 189 / 198; 150, 12 classes 217 / 279).
inline bool takes_rows(int n_features, int n_outputs)
{
    if (n_features <= ROWS_MAX_FEATURES) return true;
    return n_features % CHUNK != 0 && n_features <= (n_outputs == 1 ? ROWS_MAX_OF_TWO : ROWS_MAX_OF_THREE);
}

// Rows of a multiple of 16 floats begin in two LDS banks or one and get the padded tile.
inline bool padded_rows(int n_features) { return n_features % STEP == 0; }

// Floats of a wave's tile: 64 rows of F are F / 4 pieces.
constexpr int rows_tile_floats(int n_features, bool padded) { return LANES * n_features + (padded ? n_features / 4 * PAD : 0); }

struct LinearPlan {
    int32_t rows = 0;       // 1: the whole-row kernel, 0: chunks
    int32_t padded = 0;     // whole-row kernel: the padded tile
    int32_t width = 0;      // chunks: floats per load of X
    int32_t once = 0;       // chunks: loads of X are non-temporal
    int32_t lds_bytes = 0;  // dynamic LDS per workgroup
};

// x: the address of X.  lds_limit: bytes of LDS that a workgroup may have; a tile beyond it goes by chunks.
inline LinearPlan plan_linear(int n_features, int n_outputs, uintptr_t x, int64_t lds_limit)
{
    LinearPlan p;
    if (takes_rows(n_features, n_outputs) && x % 16 == 0) {
        p.padded = padded_rows(n_features);
        const int64_t lds = static_cast<int64_t>(sizeof(float)) * ROWS_WAVES * rows_tile_floats(n_features, p.padded);
        if (lds <= lds_limit) {
            p.rows = 1;
            p.lds_bytes = static_cast<int32_t>(lds);
            return p;
        }
        p.padded = 0;
    }
    // chunks: the widest load that every row start and every chunk start is aligned for
    p.width = n_features % 4 == 0 && x % 16 == 0 ? 4 : n_features % 2 == 0 && x % 8 == 0 ? 2 : 1;
    p.once = n_features % CHUNK == 0 && x % 128 == 0;
    return p;
}

}  // namespace linear_impl
