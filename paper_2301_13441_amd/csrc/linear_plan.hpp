// What a call on a linear model launches: kernel, width of its loads, cache policies.  Host code without HIP, so that the
// rules can be tested without a GPU (include/linear_testing.h).
#pragma once

#include <cstddef>
#include <cstdint>

namespace linear_impl {

constexpr int LANES = 64;
constexpr int CHUNK = 32;      // features per pass of the chunked kernel
constexpr int CHUNK_WAVES = 4;  // waves per workgroup of the chunked kernel
constexpr int ROWS_WAVES = 2;   // of the whole-row kernel
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

// The whole-row kernel, or chunks.  Up to 96 features always the former; beyond, multiples of 32 go by chunks, whose lines are
// whole; of the others those of which three row workgroups fit a CU (up to 104 features) and, with one output, those of which
// two do (150M values, us, chunks / rows: 100 features, one output 243 / 178; 130, one output 271 / 183; 100 features, 2 outputs
// 132 / 103, 5 outputs 136 / 128; 112 features, 5 classes 189 / 198; 150, 12 classes 217 / 279) may go by rows.  What decides is how
// the CUs share the workgroups, which own 128 rows and 256 rows:
// - rows that one round of row workgroups holds: chunks leave CUs with one workgroup and others with two (80,000 x 100, 8 outputs
//   18.2 / 14.2; 80,000 x 104, 20 outputs 42.5 / 28.6; 16 outputs 26.8 / 18.9; one output, 20,000 x 130 9.7 / 6.4), but for 7 or 8
//   outputs where every chunk workgroup has a CU to itself (40,000 x 104, 8 outputs 10.6 / 12.6);
// - a rest behind a round of row workgroups costs as much as the round (120,000 x 104, 2 outputs 13.1 / 18.6, 6 outputs 18.1 / 20.5,
//   16 outputs, 100 features 28.6 / 31.8; 120,000 x 98, 4 outputs 14.8 / 17.0), until there are many (250,000 x 100, 2 outputs
//   22.7 / 22.8, 500,000 x 104, 6 outputs 54 / 52); more than 6 outputs stay with chunks (1.44M x 104, 8 outputs 138 / 161, 16 outputs
//   182 / 229, 20 outputs 284 / 351), unless these load less than 16 bytes at a time (1.53M x 98, 20 outputs 375 / 359);
// - one output, rows of a multiple of 8 floats, which begin in few LDS banks, from the second row workgroup of a CU on (90,000 x 112
//   10.6 / 13.4, 140,000 x 152 20.3 / 26.7, 400,000 x 120 41.6 / 45.8, 600,000 x 136 68.4 / 65.7, 1M x 112 82.9 / 80.1).
constexpr int64_t CUS = 256;
constexpr int64_t CHUNK_ROUND = CUS * CHUNK_WAVES * LANES;      // rows of a chunk workgroup for every CU
constexpr int64_t ROWS_ROUND = 3 * CUS * ROWS_WAVES * LANES;    // of three row workgroups
constexpr int64_t MANY_ROUNDS = int64_t{1} << 18, MANY_ROUNDS_OF_TWO = int64_t{1} << 19;  // rows

inline bool takes_rows(int n_features, int n_outputs, int64_t n_rows)
{
    if (n_features <= ROWS_MAX_FEATURES) return true;
    if (n_features % CHUNK == 0) return false;
    if (n_outputs == 1 && n_features > ROWS_MAX_OF_THREE)
        return n_features <= ROWS_MAX_OF_TWO && (n_features % 8 != 0 || n_rows <= CUS * ROWS_WAVES * LANES || n_rows > MANY_ROUNDS_OF_TWO);
    if (n_features > ROWS_MAX_OF_THREE) return false;
    const bool loose = n_features % 4 != 0;  // chunks load these rows by halves or single floats
    if (n_outputs == 1) return true;
    if (n_rows <= ROWS_ROUND) return n_outputs <= 6 || n_outputs > 8 || n_rows > CHUNK_ROUND;
    if (n_outputs <= 6) return n_rows > MANY_ROUNDS || (loose && n_outputs <= 3);
    return loose && n_outputs > 16;
}

// Rows of a multiple of 16 floats begin in two LDS banks or one and get the padded tile.
inline bool padded_rows(int n_features) { return n_features % STEP == 0; }

// Floats of a wave's tile: 64 rows of F are F / 4 pieces.
constexpr int rows_tile_floats(int n_features, bool padded) { return LANES * n_features + (padded ? n_features / 4 * PAD : 0); }

// Scores and labels go past the L2 (device scope): beside X, of which every line is new, written lines that wait in the L2 leave
// it in no order, and every write there costs the reads of X more than its bytes (us, non-temporal or kept / past it: 2M x 128,
// 10 classes 194.4 / 189.1, 169 with no scores written; 8M x 28, sigmoid and label 158.4 / 149.5; 8M x 20, 3 classes 122.9 /
// 118).  One score a row of 64 features or more does not need it, and a label beside it goes past the L2 alone, wherever it begins
// (us, scores non-temporal / past the L2: 4M x 90 213.1 / 212.6, 5.6M x 90 296.2 / 298.4, 667,000 x 150 67.9 / 69.6, 1.56M x 64
// 63.4 / 62.3; with a label, results written over 4M x 90 223.5 / 226.4, 2.2M x 90 124.8 / 126.2, 3.1M x 64 128.6 / 127.2, and in
// new places 4M x 90 224.0 / 235.8, 4.5M x 80 235.8 / 245.6, 5.6M x 64 and five more rows 235.8 / 263.3).
// Two or three scores of a row of 56 features or more, and their label, do not either as long as X is small beside the 256 MB
// cache before the memory, which then serves the reads that the writes would hold up (us, kept / past the L2: two 234,000 x 64
// 13.2 / 14.1, 1.09M x 64 46.1 / 46.8, 1.25M x 80 68.8 / 72.6, 667,000 x 90 42.2 / 44.0, 313,000 x 128 26.1 / 26.9, three 500,000 x
// 80 33.9 / 35.4; from 2^27 floats of X on two 2.3M x 64 99.5 / 96.1, 1.7M x 90 98.1 / 96.6, three 1.9M x 80 114.3 / 111.9; five
// 444,000 x 90 38.1 / 38.7, 625,000 x 64 35.1 / 34.7; two 1M x 48 35.8 / 34.9).
// A wave's 64 scores of one output, or its labels, are whole pieces of 64 bytes only if the first of them begins one.  Elsewhere
// two waves share a piece, which past the L2 goes to memory once for each (one output and label, where labels begin behind the
// scores of an odd number of rows, and results that are not written over and over, us, both past the L2 / labels kept: 20M x 10
// 198 / 165, 16M x 13 196 / 167, 7.1M x 28 163 / 143, 7.5M x 48 273 / 247; two outputs, 31M x 8 249 / 234).  16 bytes per lane
// of a tile's several scores do not mind (5.4M x 28, 5 outputs, 4 to 12 bytes off: 119.9, on the boundary 118.9).  Rows of a few
// features, which are as many bytes as their results, do not gain from the scores alone where their labels are kept (4,734,629 x
// 1, both kept / scores past the L2 21.3 / 22.8, x 3 22.7 / 23.5, x 5 25.9 / 26.1, x 6 27.7 / 27.7, x 10 38.8 / 38.0).
constexpr int TINY_FEATURES = 5;
constexpr int FEW_COLUMNS = 3, FEW_COLUMNS_FEATURES = 56;
constexpr int64_t FEW_COLUMNS_X = int64_t{1} << 27;  // floats
constexpr int FEW_WRITES_FEATURES = 64;
constexpr uintptr_t WRITE_PIECE = 64;

// Chunks that are whole lines are read with the non-temporal policy: nothing reads them again and the caches need not keep them.
// Elsewhere two chunks share a line, and with that policy it came from memory twice (1M x 300, 2 classes 319 us a call, 240 so;
// 1.5M x 200 287 and 221; 2M x 128, 10 classes the other way 191 and 215).  More than 16 outputs take longer than that line and
// do better with it all the same (100M values, with the cache / non-temporal: 17 outputs, 200 features 210 / 191, 112 226 / 197;
// 20 outputs, 132 225 / 211, 300 203.6 / 202.3, 108 232 / 234; 32 outputs, 200 300 / 270; 16 outputs, 132 133 / 149).  So does a
// batch whose chunk workgroups have a CU each, where the L1 still holds the line when the next chunk comes for its rest (50,000 x
// 300, 10 outputs 34.9 / 25.4; 65,536 x 144, one output 12.3 / 9.2; 50,000 x 200, 3 outputs 16.3 / 12.9; 70,000 x 200, one output the
// other way 16.3 / 20.0), unless X is small enough for the L2s to hold it (10,000 x 300, one output 10.9 / 13.2, 30,000 x 132, 3
// outputs 8.5 / 9.6; 30,000 x 200, 10 outputs 21.2 / 19.1); and one whose CUs have two, if the outputs take long to sum up (16
// outputs, 100,000 x 200 42.8 / 36.2, 131,072 x 132 35.9 / 33.0; 12 outputs, 100,000 x 200 34.2 / 31.1; 8 outputs, 100,000 x 112 18.4 /
// 16.1, 131,072 x 112 20.1 / 19.1, 100,000 x 164 24.1 / 25.2, 70,000 x 300 33.1 / 35.5; 3 outputs, 70,000 x 112 11.6 / 11.7), or even
// four (16 outputs, 200,000 x 200 73.4 / 66.9, 300 features 103 / 94.5, 132 47 / 51.6; 8 outputs, 200,000 x 200 46.3 / 51.8).
constexpr int ONCE_OUTPUTS = 16, ONCE_LONG_OUTPUTS = 6, ONCE_LONGER_OUTPUTS = 10, ONCE_LONGEST_OUTPUTS = 12;
constexpr int ONCE_LONGEST_FEATURES = 160;
constexpr int64_t ONCE_X = int64_t{1} << 22, ONCE_LONG_X = 7 * (int64_t{1} << 21);  // floats

inline bool reads_once(int n_features, int n_outputs, int64_t n_rows, uintptr_t x)
{
    if (n_outputs > ONCE_OUTPUTS || (n_features % CHUNK == 0 && x % 128 == 0)) return true;
    const int64_t floats = n_rows * n_features;
    if (n_rows <= CHUNK_ROUND) return floats > ONCE_X;
    if (n_rows <= 2 * CHUNK_ROUND) return n_outputs > ONCE_LONGER_OUTPUTS || (n_outputs > ONCE_LONG_OUTPUTS && floats <= ONCE_LONG_X);
    return n_rows <= 4 * CHUNK_ROUND && n_outputs > ONCE_LONGEST_OUTPUTS && n_features > ONCE_LONGEST_FEATURES;
}

struct LinearPlan {
    int32_t rows = 0;       // 1: the whole-row kernel, 0: chunks
    int32_t padded = 0;     // whole-row kernel: the padded tile
    int32_t width = 0;      // chunks: floats per load of X
    int32_t once = 0;       // chunks: loads of X are non-temporal
    int32_t lds_bytes = 0;  // dynamic LDS per workgroup
    int32_t scores_past = 0, labels_past = 0;  // 1: stored past the L2
};

// x, scores, labels: addresses, 0 of what is not asked for.  lds_limit: bytes of LDS that a workgroup may have; a tile beyond it goes by chunks.
inline LinearPlan plan_linear(int n_features, int n_outputs, int64_t n_rows, uintptr_t x, uintptr_t scores, uintptr_t labels, int64_t lds_limit)
{
    LinearPlan p;
    const bool few_writes = n_features >= FEW_WRITES_FEATURES;
    const bool kept = n_outputs > 1 && n_outputs <= FEW_COLUMNS && n_features >= FEW_COLUMNS_FEATURES && n_rows * n_features < FEW_COLUMNS_X;
    const bool tiny = n_features <= TINY_FEATURES && labels % WRITE_PIECE != 0;
    p.scores_past = scores && (n_outputs > 1 ? !kept : scores % WRITE_PIECE == 0 && !few_writes && !tiny);
    p.labels_past = labels && !kept && (labels % WRITE_PIECE == 0 || (n_outputs == 1 && few_writes));
    if (takes_rows(n_features, n_outputs, n_rows) && x % 16 == 0) {
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
    p.once = p.width == 4 && reads_once(n_features, n_outputs, n_rows, x);
    return p;
}

}  // namespace linear_impl
