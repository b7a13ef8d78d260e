// Device helpers shared by the walk kernels (forest_kernels_walk.hip, forest_kernels_deep.hip): LDS by
// byte address, and the tile of float32 features.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

#include "forest_device.hpp"
#include "forest_kernel_common.hpp"

namespace forest_impl {

typedef uint32_t Vec4 __attribute__((ext_vector_type(4)));
typedef uint32_t Vec2 __attribute__((ext_vector_type(2)));

// LDS by byte address: the kernels have no static LDS, so the dynamic part begins at 0 (checked at
// start-up) and addresses are plain integers with the level's offset as an immediate.
template <typename T>
__device__ __forceinline__ T lds_read(uint32_t at)
{
    return *reinterpret_cast<const __attribute__((address_space(3))) T *>(at);
}
template <typename T>
__device__ __forceinline__ void lds_write(uint32_t at, T v)
{
    *reinterpret_cast<__attribute__((address_space(3))) T *>(at) = v;
}

typedef float FloatRun4 __attribute__((ext_vector_type(4), aligned(4)));
#if defined(__HIP_DEVICE_COMPILE__)
typedef const __attribute__((address_space(1))) FloatRun4 *GlobalRuns;
typedef const __attribute__((address_space(1))) Vec4 *GlobalVec4;
typedef const __attribute__((address_space(4))) uint32_t *WalkTop;
typedef const __attribute__((address_space(4))) int32_t *WalkTable;
typedef const __attribute__((address_space(1))) char *GlobalBytes;
typedef const __attribute__((address_space(1))) float *GlobalFloats;
typedef const __attribute__((address_space(1))) int32_t *GlobalInts;
#else
typedef const FloatRun4 *GlobalRuns;
typedef const Vec4 *GlobalVec4;
typedef const uint32_t *WalkTop;  // host pass: the kernel body is only parsed
typedef const int32_t *WalkTable;
typedef const char *GlobalBytes;
typedef const float *GlobalFloats;
typedef const int32_t *GlobalInts;
#endif

typedef uint32_t LooseVec4 __attribute__((ext_vector_type(4), aligned(4)));

// Bit BIT of the lane and the index of two registers change places: lane l of b with bit BIT clear and lane l ^ 1 << BIT of a.
template <int BIT>
__device__ __forceinline__ void exchange_lane_bit(float &a, float &b, int lane)
{
    const uint32_t x = __float_as_uint(a), y = __float_as_uint(b);
    if constexpr (BIT < 2) {
        constexpr int perm = BIT == 0 ? 0xB1 : 0x4E;  // lanes [1, 0, 3, 2] or [2, 3, 0, 1] of every four
        const uint32_t from_b = __builtin_amdgcn_mov_dpp(static_cast<int>(y), perm, 0xf, 0xf, true);
        const uint32_t from_a = __builtin_amdgcn_mov_dpp(static_cast<int>(x), perm, 0xf, 0xf, true);
        a = __uint_as_float(lane >> BIT & 1 ? from_b : x);
        b = __uint_as_float(lane >> BIT & 1 ? y : from_a);
    } else {
        static_assert(BIT == 4 || BIT == 5, "halves and quarters of a wave");
        const auto r = BIT == 4 ? __builtin_amdgcn_permlane16_swap(x, y, false, false) : __builtin_amdgcn_permlane32_swap(x, y, false, false);
        a = __uint_as_float(r[0]);
        b = __uint_as_float(r[1]);
    }
}

// How the lanes of a wave take eight rows' 128 bytes in one load: bits 1 to 3 the row, bits 0, 4 and 5 the four of features.  A line goes whole,
// and the bits that pairs of registers exchange in one instruction are features.
__device__ __forceinline__ int line_row(int lane) { return (lane >> 1) & 7; }
__device__ __forceinline__ int line_four(int lane) { return (lane & 1) | (lane >> 3 & 6); }

// The X tile of a workgroup: rows [row0, row0 + 64 NR) as float32, row group g, feature f and row r of the
// group at xbase + g * group_stride + f * stride + 4 r.  It is filled in pieces of 8 L rows x 32 features, L loads of
// eight rows' 128 bytes, non-temporally (ONCE) or not (keeps_lines, forest_plan.hpp).  A line that is asked for in
// two halves is read twice so, and what waits for it holds up the other loads of the CU, which return in order (16 rows' 64
// bytes a load and no exchange: 103,069 rows of 300 deep trees, 90 features 72.2 us, so 69.5; 100 trees of depth 6, 64 features,
// 300,000 rows 44.9 / 41.2, 300 features, 100,000 rows 61.7 / 55.6).  But of narrow rows lines make few pieces, which
// few waves load and exchange while the others wait: 8 features, 1M rows 93.8 / 98.0.  So rows of fewer than lines_from features go by 64
// bytes of 16 rows: of 17, and of 33 for leaf ids of few trees, which are little but the fill, in workgroups of one and two row groups (2 trees of
// depth 8, two columns, 25 features, 800,000 rows 29.8 / 42.0 us; 12 of depth 5, 32 features, 300,000 rows 17.3 / 20.7).  The lanes exchange what they loaded until 16 rows are written at a time, for 16 of 32 LDS banks.
// The four features of a lane that would reach beyond the row are the row's last four (written twice, with the same values), and
// the rows beyond the batch are its last row, so that every load is whole and none waits for another: a lane's features
// one by one under a mask of their own cost a second round trip to memory, and the addresses as 64-bit products more
// instructions than the loads (256 features, 4M rows of 128 deep trees: 2.89 -> 2.80 ms a call).  NAN_IS_INF: a NaN is stored as +Inf.
template <int NR, int P, bool NAN_IS_INF, bool LINES, bool ONCE, bool ONE_BLOCK = false>
__device__ __forceinline__ void fill_pieces(const float *X, int64_t row0, int64_t n_rows, int F, uint32_t xbase, uint32_t group_stride,
                                            uint32_t stride, int wave, int lane)
{
    constexpr int L = !LINES ? 1 : NR == 1 ? 2 : 4, LOAD_ROWS = LINES ? 8 : 16, ROWS = LOAD_ROWS * L, FEATURES = LINES ? 32 : 16, G = P / L;  // G pieces on their way at a time
    const char *tile = reinterpret_cast<const char *>(X + row0 * F);
    const int rows = n_rows - row0 < NR * TILE ? static_cast<int>(n_rows - row0) : NR * TILE;
    const int blocks = ONE_BLOCK ? 1 : (F + FEATURES - 1) / FEATURES, pieces = blocks * (NR * TILE / ROWS);
    const int begin = pieces * wave / WALK_WAVES, end = pieces * (wave + 1) / WALK_WAVES;
    const uint32_t pitch = static_cast<uint32_t>(F) * 4;
    // a lane's row and four of features as loaded, and, of register 0, after the exchange
    const int r = LINES ? line_row(lane) : lane & 15, c = LINES ? line_four(lane) : lane >> 4;
    const int after_r = LINES ? (lane >> 1) & (ROWS - 1) : r, after_c = !LINES ? c : L == 2 ? (lane & 1) | (lane >> 5) * 4 : lane & 1;
    int at_rows = begin / blocks, at_block = begin - at_rows * blocks;  // the piece
    for (int t = begin; t < end; t += G) {
        FloatRun4 v[G][L];
        uint32_t to[G];
        int block[G];
#pragma unroll
        for (int g = 0; g < G; ++g) {
            if (t + g < end) {  // wave-uniform
                const int f = min(at_block * FEATURES + c * 4, F - 4), first = at_rows * ROWS;
#pragma unroll
                for (int u = 0; u < L; ++u) {
                    const auto from = (GlobalRuns)((GlobalBytes)tile + (static_cast<uint32_t>(min(first + u * LOAD_ROWS + r, rows - 1)) * pitch + static_cast<uint32_t>(f) * 4));
                    v[g][u] = ONCE ? __builtin_nontemporal_load(from) : *from;
                }
                to[g] = xbase + static_cast<uint32_t>(first >> 6) * group_stride + static_cast<uint32_t>((first & 63) + after_r) * 4;
                block[g] = at_block;
                if (++at_block == blocks) {
                    at_block = 0;
                    ++at_rows;
                }
            }
        }
#pragma unroll
        for (int g = 0; g < G; ++g) {
            if (t + g < end) {
                uint32_t at[L];
#pragma unroll
                for (int k = 0; k < L; ++k) at[k] = to[g] + static_cast<uint32_t>(min(block[g] * FEATURES + (after_c + 2 * k) * 4, F - 4)) * stride;
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    float x[L];
#pragma unroll
                    for (int k = 0; k < L; ++k) x[k] = v[g][k][i];
                    if constexpr (L > 1) exchange_lane_bit<4>(x[0], x[1], lane);
                    if constexpr (L == 4) {
                        exchange_lane_bit<4>(x[2], x[3], lane);
                        exchange_lane_bit<5>(x[0], x[2], lane);
                        exchange_lane_bit<5>(x[1], x[3], lane);
                    }
#pragma unroll
                    for (int k = 0; k < L; ++k) lds_write<float>(at[k] + i * stride, NAN_IS_INF ? fminf(x[k], __builtin_inff()) : x[k]);
                }
            }
        }
    }
}

template <int NR, int P, bool NAN_IS_INF>
__device__ __forceinline__ void tile_fill(const float *X, int64_t row0, int64_t n_rows, int x_tile, int lines_from, uint32_t xbase, uint32_t group_stride,
                                          uint32_t stride, int wave, int lane)
{
    const int F = x_tile & (KEEP_X - 1);
    if (F >= lines_from) {
        if (x_tile & KEEP_X) fill_pieces<NR, P, NAN_IS_INF, true, false>(X, row0, n_rows, F, xbase, group_stride, stride, wave, lane);
        else fill_pieces<NR, P, NAN_IS_INF, true, true>(X, row0, n_rows, F, xbase, group_stride, stride, wave, lane);
    } else if (F > 16) {
        fill_pieces<NR, P, NAN_IS_INF, false, true>(X, row0, n_rows, F, xbase, group_stride, stride, wave, lane);
    } else if (F >= 4) {
        fill_pieces<NR, P, NAN_IS_INF, false, true, true>(X, row0, n_rows, F, xbase, group_stride, stride, wave, lane);
    } else {  // a lane per row
        const float *tile = X + row0 * F;
        const int rows = n_rows - row0 < NR * TILE ? static_cast<int>(n_rows - row0) : NR * TILE;
        for (int g = wave; g < NR; g += WALK_WAVES)
            for (int f = 0; f < F; ++f) {
                const float x = tile[min(g * TILE + lane, rows - 1) * F + f];
                lds_write<float>(xbase + g * group_stride + f * stride + lane * 4, NAN_IS_INF ? fminf(x, __builtin_inff()) : x);
            }
    }
}

// The same tile on its way to registers while the one before is walked.  A piece is 64 rows x 32 features: eight loads of
// eight rows' 128 bytes, one piece a wave at most (ahead_pieces, forest_plan.hpp).  Waves beyond the last piece load and store nothing:
// with the last piece once more for each of them, on the path that bounds the kernel, a tile was asked for up to twice: 128
// features, 66,000 rows of 20 trees of depth 9 20.5 us (so 16.0), 1M rows 177 (134), of 300 such trees 763 (722), of 128 trees of depth 12
// 557 (514).  F >= 4.
template <int NR, bool ONCE>
struct TileAhead {
    static constexpr int LOADS = 8;
    FloatRun4 v[LOADS];

    struct Piece {
        int group, feature;  // row group, first feature
    };
    static __device__ __forceinline__ Piece piece(int F, int wave)
    {
        const int blocks = ahead_pieces(F, 1);
        static_assert(NR <= 2, "one comparison");
        const int group = NR == 1 ? 0 : wave >= blocks;
        return Piece{group, (wave - group * blocks) * 32};
    }
    // A lane's row and four of features in a load: bits 0, 1 and 4 the four.
    static __device__ __forceinline__ int row_of(int lane) { return (lane >> 2 & 3) | (lane >> 3 & 4); }
    static __device__ __forceinline__ int four_of(int lane) { return (lane & 3) | (lane >> 2 & 4); }
    // The tile whose first row `tile` points at and which has `rows` rows.
    __device__ __forceinline__ void request(const float *tile, int rows, int F, int wave, int lane)
    {
        if (wave >= ahead_pieces(F, NR)) return;  // wave-uniform, here and below: the exchanges have all their lanes
        const Piece p = piece(F, wave);
        asm volatile("" : "+v"(lane));
        const int f = min(p.feature + four_of(lane) * 4, F - 4);
#pragma unroll
        for (int u = 0; u < LOADS; ++u) {
            const int row = min(p.group * TILE + u * 8 + row_of(lane), rows - 1);
            const auto from = (GlobalRuns)((GlobalBytes)tile + static_cast<uint32_t>(row * F + f) * 4);
            v[u] = ONCE ? __builtin_nontemporal_load(from) : *from;
        }
    }
    __device__ __forceinline__ void store(int F, uint32_t xbase, uint32_t group_stride, uint32_t stride, int wave, int lane) const
    {
        if (wave >= ahead_pieces(F, NR)) return;
        asm volatile("" : "+v"(lane));
        const Piece p = piece(F, wave);
        // after the exchange a lane has the features of one row, register k four of them from 4 k
        const uint32_t row = xbase + static_cast<uint32_t>(p.group) * group_stride + static_cast<uint32_t>(four_of(lane) * 8 + row_of(lane)) * 4;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            float x[LOADS];
#pragma unroll
            for (int k = 0; k < LOADS; ++k) x[k] = v[k][i];
#pragma unroll
            for (int k = 0; k < LOADS; k += 2) exchange_lane_bit<0>(x[k], x[k + 1], lane);
#pragma unroll
            for (int k = 0; k < LOADS; ++k)
                if (!(k & 2)) exchange_lane_bit<1>(x[k], x[k + 2], lane);
#pragma unroll
            for (int k = 0; k < LOADS / 2; ++k) exchange_lane_bit<4>(x[k], x[k + 4], lane);
#pragma unroll
            for (int k = 0; k < LOADS; ++k)
                lds_write<float>(row + (static_cast<uint32_t>(min(p.feature + k * 4, F - 4)) + i) * stride, x[k]);
        }
    }
};

// The ids of n trees from `begin` of a row, counted from a workgroup's first: those of four with one store.  The row's place
// comes from 32-bit factors (from the row of the batch, a 64-bit product, leaf ids of 262,144 rows of 128 x depth 6 took
// 60.4 us instead of 55.4).  THROUGH: past the L2 (ids_go_through, forest_plan.hpp), but for two or three ids of a wave.  A form of
// the kernels of its own: chosen per store, the other form's descriptor cost every kernel four scalar registers, of which they
// spill some (20 trees of depth 8, 500,000 rows: 63.9 -> 62.9 us; of depth 6, 100,000 rows: 13.6 -> 13.2).
template <bool THROUGH>
struct IdStore {
    int32_t *first;  // of the workgroup's first row, wave-uniform
    int T;

    __device__ __forceinline__ void operator()(int li, int begin, int n, Vec4 id) const
    {
        const uint64_t at = static_cast<uint64_t>(static_cast<uint32_t>(li)) * static_cast<uint32_t>(T) + static_cast<uint32_t>(begin);
        if (n == 4 && begin + 4 <= T) {
            if constexpr (THROUGH)
                __builtin_amdgcn_raw_buffer_store_b128(id, __builtin_amdgcn_make_buffer_rsrc(first, 0, 0x7fffffff, 0x00027000), static_cast<int>(at) * 4, 0, 16 /* sc1 */);
            else
                *reinterpret_cast<LooseVec4 *>(first + at) = id;  // one value: of four, three would be stored by the path below and one alone (101 trees, 100,000 rows 28.8 us, so 26.8)
        } else if (THROUGH && n == 1) {
            if (begin < T) __hip_atomic_store(first + at, static_cast<int32_t>(id[0]), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        } else {
#pragma unroll
            for (int j = 0; j < 4; ++j)
                if (j < n && begin + j < T) first[at + j] = static_cast<int32_t>(id[j]);
        }
    }
};

// The first row of a workgroup: the first workgroups of a launch own groups x 64 rows, those after them last x 64 (choose_tail, forest_plan.hpp).
__device__ __forceinline__ int64_t first_row(const DevModel &m, int groups, int last, bool &after)
{
    const int64_t block = blockIdx.x;
    after = groups != last && block >= m.full_workgroups;
    return after ? (m.full_workgroups * groups + (block - m.full_workgroups) * last) * TILE : block * groups * TILE;
}

// The column sums of one wave's run of trees for NR row groups: the running column's, those of the columns before it.
template <int NR, int COLUMNS>
struct ColumnSums {
    static constexpr int DONE = COLUMNS > 1 ? COLUMNS - 1 : 1;
    double acc[NR], done[DONE][NR];
    int first = 0, column = 0, n_done = 0, done_column[DONE] = {};

    __device__ __forceinline__ void begin(int c)
    {
        first = column = c;
#pragma unroll
        for (int r = 0; r < NR; ++r) acc[r] = 0.0;
    }
    __device__ __forceinline__ void change(int c)  // the column of the values added next
    {
#pragma unroll
        for (int k = DONE - 1; k > 0; --k) {
            done_column[k] = done_column[k - 1];
#pragma unroll
            for (int r = 0; r < NR; ++r) done[k][r] = done[k - 1][r];
        }
        done_column[0] = column;
        ++n_done;
        column = c;
#pragma unroll
        for (int r = 0; r < NR; ++r) {
            done[0][r] = acc[r];
            acc[r] = 0.0;
        }
    }
};

// The rows of a walk kernel's workgroup from its waves' sums, which meet in LDS in the order of the waves.  A wave's run
// of trees feeds consecutive columns (the trees are sorted by column), so the sum of (wave, column) has the slot wave +
// column to itself and every wave fills its own slots, zeros for columns of its range that no tree feeds, behind one
// barrier.  LDS: slots [WAVES + K - 1][ROWS], sums [K][ROWS], the waves' first columns and how many follow.  A split launch
// stores the sums as they come.  (All slots cleared by all threads first, and a split launch's rows stored by a thread each,
// was two barriers and a serial loop more: 10,007 rows of 250 x depth 8, 5 columns, 17.8 us a call against 17.2.)
// What bounds it is the round trips to LDS: a sum's slots are read together, of several columns only those of the waves
// that feed the column, which a ballot finds.  One wave's slot after the other under a test of its own was 16 trips in turn
// (calls, us: 1,021 rows of 2000 x depth 6, 10 columns 15.35 -> 14.72; 10,007 rows of 250 x depth 8, 5 columns 16.20 -> 15.38;
// 103,069 rows of 300 irregular trees of depth 9 83.2 -> 80.8; 1M rows of 500 x depth 8 624 -> 621; 500,000 rows of
// 2000 x depth 6, 10 columns 831 -> 824, where all 16 slots of every column would take 844).
template <int NR, int WAVES, int COLUMNS>
__device__ __forceinline__ void finish_columns(const DevModel &m, char *smem, int wave, int lane, bool any, const ColumnSums<NR, COLUMNS> &sums,
                                               int64_t row0, int64_t n_rows, float *scores, int32_t *labels)
{
    constexpr int ROWS = NR * TILE;
    const int K = m.n_outputs;
    double *slot = reinterpret_cast<double *>(smem);
    double *sum = slot + static_cast<size_t>(WAVES + K - 1) * ROWS;
    int32_t *fed = reinterpret_cast<int32_t *>(sum + static_cast<size_t>(K) * ROWS);
    __syncthreads();
    const auto at = [&](int k, int r) -> double & { return slot[(wave + k) * ROWS + r * TILE + lane]; };
    if constexpr (COLUMNS == 1) {
#pragma unroll
        for (int r = 0; r < NR; ++r) at(0, r) = sums.acc[r];
    } else {
        if (lane == 0) {
            fed[2 * wave] = any ? sums.first : K;
            fed[2 * wave + 1] = sums.column - sums.first;
        }
        if (any) {
            if (sums.column - sums.first > sums.n_done)
                for (int k = sums.first; k < sums.column; ++k)
#pragma unroll
                    for (int r = 0; r < NR; ++r) at(k, r) = 0.0;
#pragma unroll
            for (int k = 0; k < COLUMNS - 1; ++k)
                if (k < sums.n_done) {
#pragma unroll
                    for (int r = 0; r < NR; ++r) at(sums.done_column[k], r) = sums.done[k][r];
                }
#pragma unroll
            for (int r = 0; r < NR; ++r) at(sums.column, r) = sums.acc[r];
        }
    }
    __syncthreads();
    for (int i = threadIdx.x; i < K * ROWS; i += WAVES * TILE) {
        const int k = i / ROWS, li = i - k * ROWS;
        double s = 0.0;
        if constexpr (COLUMNS == 1) {
            double v[WAVES];
#pragma unroll
            for (int w = 0; w < WAVES; ++w) v[w] = slot[w * ROWS + li];
#pragma unroll
            for (int w = 0; w < WAVES; ++w) s += v[w];
        } else {
            // k is one for the wave: a lane per wave of the workgroup finds out which of them feed it
            const int w = lane & (WAVES - 1);
            uint32_t waves = static_cast<uint32_t>(__ballot(static_cast<uint32_t>(k - fed[2 * w]) <= static_cast<uint32_t>(fed[2 * w + 1]))) & ((1u << WAVES) - 1);
            while (waves) {
                double v[4];
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    v[j] = 0.0;
                    if (waves) v[j] = slot[(__builtin_ctz(waves) + uniform(k)) * ROWS + li];
                    waves &= waves - 1;  // 0 stays 0
                }
#pragma unroll
                for (int j = 0; j < 4; ++j) s += v[j];
            }
        }
        if (m.n_splits == 1) sum[i] = s;
        else if (row0 + li < n_rows) m.partial[(static_cast<int64_t>(blockIdx.y) * m.split_rows + row0 + li) * K + k] = s;
    }
    if (m.n_splits > 1) return;
    if (K > 1) __syncthreads();  // one column: a thread finishes the row that it summed
    for (int li = threadIdx.x; li < ROWS; li += WAVES * TILE)
        if (row0 + li < n_rows) finish_values(m, sum + li, ROWS, row0 + li, scores, labels);
}

}  // namespace forest_impl
