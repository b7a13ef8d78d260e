// Walk kernels (gfx950): trees of depth up to 8 with scalar leaves, one node per level and row.
//
// The paper's three operators answer "which leaf does the row reach" by testing every internal
// node (step (1) and (2) of Fig. 2) and selecting the leaf whose path agrees (step (3)).  Only the
// tests on the row's own path decide that selection.  Here the first two levels are still evaluated
// whole -- their three nodes are the same for every row, so they come through scalar loads and
// their comparisons cost no per-lane look-up -- and below that a lane tests the one node of each
// level that its path meets: two LDS reads (node, feature value) and four vector instructions per
// (row, level) instead of half a vector instruction per (row, node).
//
// A workgroup of 16 waves owns NR x 64 rows, NR per lane, whose features it holds in LDS as float32
// ([feature][row]: the lanes of a wave read one column each of their own row, which falls into 32
// different banks whatever the features are).  Every wave walks its own run of trees for all the
// rows, a stage (1 or 2 KB of whole trees) at a time: the next stage is on its way to registers
// while this one is walked in LDS, and no wave waits for another between the first and the last
// tree.  A node is 8 bytes, {threshold, byte offset of the feature in the X tile}, read at once
// (64-bit LDS reads move 256 bytes per clock, 32-bit ones 128).  Its slot is numbered by the
// outcomes on the path, first outcome in bit 0, so the address of the next node is the last one's
// with one bit more: the sign of threshold - x, moved to its place by v_and_or_b32.  (The subtraction
// is exact in sign for finite thresholds: it is 0 for equal operands and never underflows to 0
// otherwise.  NaN, which belongs on the right of every threshold, is stored in the tile as +Inf.)
// Leaf values are gathered from global memory, which the LDS traffic leaves idle, and added one
// tree later, in fp64.
//
// Bound: at depth 8 the LDS (89 % busy), at depth 6 the vector ALU (96 %) with the LDS (82 %) behind it.  Per (64 rows,
// tree of depth D): 3 + 2 (D - 2) LDS reads of 2 clocks each, more at levels 6 and 7 whose 64 and 128 nodes share the
// 32 banks.  500 trees of depth 8, 28 features, 1M rows: 2.70 -> 0.63 ms against every node tested
// (forest_kernels_rank.hip); 1000 of depth 6, 50 features: 1.57 -> 0.79 ms.
#include <hip/hip_runtime.h>

#include <cstdint>

#include "forest_device.hpp"
#include "forest_kernel_common.hpp"
#include "forest_walk_common.hpp"

namespace forest_impl {
namespace {

// One tree, all row groups: idx[r] = LDS address of the tree | 8 * (index of the leaf reached).
template <int D, int NR>
__device__ __forceinline__ void walk_tree(uint32_t tree_at, uint32_t xa, WalkTop top, uint32_t (&idx)[NR])
{
    const float t1 = __uint_as_float(top[2]), t2 = __uint_as_float(top[4]), t3 = __uint_as_float(top[6]);
    const uint32_t a1 = xa + top[3], a2 = xa + top[5], a3 = xa + top[7];
    float x1[NR], x2[NR], x3[NR];
#pragma unroll
    for (int r = 0; r < NR; ++r) x1[r] = lds_read<float>(a1 + r * 256);
#pragma unroll
    for (int r = 0; r < NR; ++r) x2[r] = lds_read<float>(a2 + r * 256);
#pragma unroll
    for (int r = 0; r < NR; ++r) x3[r] = lds_read<float>(a3 + r * 256);
#pragma unroll
    for (int r = 0; r < NR; ++r) {
        const uint64_t m1 = __ballot(!(x1[r] <= t1)), m2 = __ballot(!(x2[r] <= t2)), m3 = __ballot(!(x3[r] <= t3));
        const uint64_t second = (m1 & m3) | (~m1 & m2);
        uint32_t b0, b1;
        asm("v_cndmask_b32 %0, 0, 8, %1" : "=v"(b0) : "s"(m1));
        asm("v_cndmask_b32 %0, 0, 16, %1" : "=v"(b1) : "s"(second));
        idx[r] = tree_at | b0 | b1;
    }
#pragma unroll
    for (int l = 2; l < D; ++l) {
        Vec2 node[NR];
        float x[NR];
#pragma unroll
        for (int r = 0; r < NR; ++r) node[r] = lds_read<Vec2>(idx[r] + (8u << l));
#pragma unroll
        for (int r = 0; r < NR; ++r) x[r] = lds_read<float>(xa + node[r].y + r * 256);
#pragma unroll
        for (int r = 0; r < NR; ++r) {
            const int right = __float_as_int(__uint_as_float(node[r].x) - x[r]) >> 31;
            asm("v_and_or_b32 %0, %1, %2, %0" : "+v"(idx[r]) : "v"(right), "s"(8 << l));
        }
    }
}

// What a kernel leaves behind: the sums of one output column, those of several (trees sorted by
// column), or the leaf ids of every tree (a kernel of its own).
enum { WALK_COLUMN = 0, WALK_COLUMNS = 1, WALK_LEAVES = 2 };

template <int D, int NR, int MODE>
__global__ __launch_bounds__(WALK_WAVES * TILE, 8) void forest_walk_kernel(DevModel m, const float *__restrict__ X,
                                                                          int64_t n_rows, float *scores,
                                                                          int32_t *labels, int32_t *)
{
    constexpr int TREE_BYTES = 8 << D, STAGE_TREES = walk_stage_trees(D), STAGE_BYTES = TREE_BYTES * STAGE_TREES;
    constexpr int PIECES = STAGE_BYTES / 1024;  // 16 bytes per lane each
    constexpr int ROWS = NR * TILE;
    static_assert(STAGE_BYTES % 1024 == 0, "whole 16-byte pieces per lane");
    extern __shared__ __align__(1024) char smem[];
    const int lane = threadIdx.x & (TILE - 1), wave = uniform(threadIdx.x >> 6);
    const int64_t row0 = static_cast<int64_t>(blockIdx.x) * ROWS;
    const uint32_t stride = static_cast<uint32_t>(m.walk.groups) * 256, xbase = WALK_WAVES * STAGE_BYTES;
    const uint32_t mine = static_cast<uint32_t>(wave) * STAGE_BYTES;

    // This wave's stages: a contiguous run.
    const int S = m.walk.stages;
    const int unit = static_cast<int>(blockIdx.y) * WALK_WAVES + wave, units = m.n_splits * WALK_WAVES;
    const int s_begin = static_cast<int>(static_cast<int64_t>(S) * unit / units);
    const int s_end = static_cast<int>(static_cast<int64_t>(S) * (unit + 1) / units);

    const char *image = reinterpret_cast<const char *>(m.walk.node);
    Vec4 ahead[PIECES];
    auto fetch = [&](int s) {
        const int64_t at = static_cast<int64_t>(s) * STAGE_BYTES + lane * 16;
#pragma unroll
        for (int i = 0; i < PIECES; ++i) ahead[i] = *reinterpret_cast<const Vec4 *>(image + at + i * 1024);
    };
    if (s_begin < s_end) fetch(s_begin);
    tile_fill<NR, NR == 4 ? 8 : 4, true>(X, row0, n_rows, m.n_features, xbase, 256, stride, wave, lane);
    __syncthreads();

    const uint32_t xa = xbase + lane * 4;
    double acc[NR], done[WALK_MAX_COLUMNS - 1][NR];  // the running column, the columns before it
    int column = 0, done_column[WALK_MAX_COLUMNS - 1], n_done = 0, first_column = 0;
    float value[NR];  // the last tree's leaf values, not yet added
#pragma unroll
    for (int r = 0; r < NR; ++r) {
        acc[r] = 0.0;
        value[r] = 0.0f;
    }
    if (MODE == WALK_COLUMNS && s_begin < s_end)
        column = first_column = ((WalkTable)(image + static_cast<int64_t>(s_begin) * STAGE_BYTES))[0];

    for (int s = s_begin; s < s_end; ++s) {
#pragma unroll
        for (int i = 0; i < PIECES; ++i) lds_write<Vec4>(mine + i * 1024 + lane * 16, ahead[i]);
        if (s + 1 < s_end) fetch(s + 1);
#pragma unroll 1
        for (int q = 0; q < STAGE_TREES; ++q) {
            const int t = s * STAGE_TREES + q;
            const WalkTop top = (WalkTop)(image + static_cast<int64_t>(t) * TREE_BYTES);
            const uint32_t tree_at = mine + q * TREE_BYTES;
            uint32_t idx[NR];
            walk_tree<D, NR>(tree_at, xa, top, idx);
#pragma unroll
            for (int r = 0; r < NR; ++r) acc[r] += static_cast<double>(value[r]);
            if (const int c = static_cast<int>(top[0]); MODE == WALK_COLUMNS && c != column) {
#pragma unroll
                for (int k = WALK_MAX_COLUMNS - 2; k > 0; --k) {
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
            // half an index is the leaf's byte offset; the tree's address in it is taken off the base
            const char *leaves = reinterpret_cast<const char *>(m.walk.leaf) + (static_cast<int64_t>(t) << (D + 2)) - (tree_at >> 1);
            asm volatile("" : "+s"(leaves));  // keeps the base whole, so that the loads take a 32-bit offset
#pragma unroll
            for (int r = 0; r < NR; ++r) value[r] = *(GlobalFloats)((GlobalBytes)leaves + (idx[r] >> 1));
        }
    }
#pragma unroll
    for (int r = 0; r < NR; ++r) acc[r] += static_cast<double>(value[r]);

    // The waves' column sums meet in LDS: a wave's run of trees feeds consecutive columns, so the
    // sum of (wave, column) has the slot wave + column to itself.
    __syncthreads();
    const int K = m.n_outputs;
    double *slot = reinterpret_cast<double *>(smem);                 // [WALK_WAVES + K - 1][ROWS]
    double *sum = slot + static_cast<size_t>(WALK_WAVES + K - 1) * ROWS;  // [K][ROWS]
    int32_t *fed = reinterpret_cast<int32_t *>(sum + static_cast<size_t>(K) * ROWS);  // first and last column of a wave
    for (int i = threadIdx.x; i < (WALK_WAVES + K - 1) * ROWS; i += WALK_WAVES * TILE) slot[i] = 0.0;
    if (lane == 0) {
        fed[2 * wave] = s_begin < s_end ? first_column : 1;
        fed[2 * wave + 1] = s_begin < s_end ? column : 0;
    }
    __syncthreads();
    if (s_begin < s_end) {
#pragma unroll
        for (int r = 0; r < NR; ++r) slot[(wave + column) * ROWS + r * TILE + lane] = acc[r];
#pragma unroll
        for (int k = 0; k < WALK_MAX_COLUMNS - 1; ++k)
            if (k < n_done) {
#pragma unroll
                for (int r = 0; r < NR; ++r) slot[(wave + done_column[k]) * ROWS + r * TILE + lane] = done[k][r];
            }
    }
    __syncthreads();
    for (int i = threadIdx.x; i < K * ROWS; i += WALK_WAVES * TILE) {
        const int k = i / ROWS, li = i - k * ROWS;
        double s = 0.0;
#pragma unroll
        for (int w = 0; w < WALK_WAVES; ++w)
            if (fed[2 * w] <= k && k <= fed[2 * w + 1]) s += slot[(w + k) * ROWS + li];
        sum[i] = s;
    }
    __syncthreads();
    for (int li = threadIdx.x; li < ROWS; li += WALK_WAVES * TILE) {
        const int64_t row = row0 + li;
        finish_summed_row(m, sum, ROWS, li, row, row < n_rows, scores, labels);
    }
}

// The leaf ids of every tree, caller's order.  A row's ids are neighbours in the output and a lane holds those of few
// trees, so the waves take four trees each, side by side, and exchange the ids through their stages before they leave: a
// store then writes whole 256-byte runs of four rows.  Straight from the lanes, 16 bytes at the pitch of a row, 100,003
// rows of 200 x depth 6 took 65.6 us, three quarters of them for the stores; so 42.5, of which the stores are 10 (250,000
// rows of 200 x depth 3: 235 -> 65; 66,000 of 700 x depth 3: 310 -> 98).  Ids of these trees, which have 511 nodes at
// most, fit 16 bits.  What is left of the trees after the last whole round is dealt evenly.  Bound: the walk, with 391
// workgroups for 256 CUs; two shares of the trees, or fewer rows per workgroup, fill the tile more often and took 54.7 and
// 50.4.
template <int D, int NR>
__global__ __launch_bounds__(WALK_WAVES * TILE, 8) void forest_walk_leaves_kernel(DevModel m, const float *__restrict__ X,
                                                                                 int64_t n_rows, float *, int32_t *,
                                                                                 int32_t *leaf_out)
{
    constexpr int TREE_BYTES = 8 << D, STEP = walk_stage_trees(D) < 4 ? walk_stage_trees(D) : 4;  // trees copied at a time
    constexpr int STEP_BYTES = TREE_BYTES * STEP, STAGE_BYTES = walk_stage_bytes(D);
    constexpr int PIECES = (STEP_BYTES + 1023) / 1024;
    constexpr int ROWS = NR * TILE;
    constexpr int EXCHANGE = NR * TILE * 8 <= STAGE_BYTES ? NR : STAGE_BYTES / (TILE * 8);  // row groups that a stage holds the ids of
    static_assert(NR % EXCHANGE == 0, "whole exchanges");
    extern __shared__ __align__(1024) char smem[];
    const int lane = threadIdx.x & (TILE - 1), wave = uniform(threadIdx.x >> 6);
    const int64_t row0 = static_cast<int64_t>(blockIdx.x) * ROWS;
    const int T = m.n_trees;
    const uint32_t stride = static_cast<uint32_t>(m.walk.groups) * 256, xbase = WALK_WAVES * STAGE_BYTES;
    const uint32_t mine = static_cast<uint32_t>(wave) * STAGE_BYTES;
    const int round = 4 * WALK_WAVES, rounds = (T + round - 1) / round;

    const char *image = reinterpret_cast<const char *>(m.walk.node);
    // Trees each wave takes in a round, and the first of this one's.
    const auto share = [&](int k) { return T - k * round >= round ? 4 : (T - k * round + WALK_WAVES - 1) / WALK_WAVES; };
    const auto first_tree = [&](int k) { return k * round + wave * share(k); };
    Vec4 ahead[PIECES];
    const auto fetch = [&](int first) {  // caller's order: a tree sits anywhere
        if (PIECES > 1 || lane * 16 < STEP_BYTES) {
            const int t = min(first + (lane * 16) / TREE_BYTES, T - 1);
            const int64_t at = static_cast<int64_t>(m.walk.position[t]) * TREE_BYTES + (lane * 16) % TREE_BYTES;
#pragma unroll
            for (int i = 0; i < PIECES; ++i) ahead[i] = *reinterpret_cast<const Vec4 *>(image + at + i * 1024);
        }
    };
    int k = static_cast<int>(blockIdx.y);
    if (k < rounds) fetch(first_tree(k));
    tile_fill<NR, NR == 4 ? 8 : 4, true>(X, row0, n_rows, m.n_features, xbase, 256, stride, wave, lane);
    __syncthreads();

    const uint32_t xa = xbase + lane * 4;
    for (; k < rounds; k += m.n_splits) {
        const int n = share(k), first = first_tree(k);
        uint32_t ids[NR][2] = {}, id[NR];  // of up to four trees, 16 bits each; of the last tree, not yet among them
        const auto keep = [&](int j) {
#pragma unroll
            for (int r = 0; r < NR; ++r) ids[r][j >> 1] = (j & 1) ? ids[r][j >> 1] | id[r] << 16 : id[r];
        };
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            if (j < n) {
                if (j % STEP == 0) {
                    if (PIECES > 1 || lane * 16 < STEP_BYTES) {
#pragma unroll
                        for (int i = 0; i < PIECES; ++i) lds_write<Vec4>(mine + i * 1024 + lane * 16, ahead[i]);
                    }
                    if (j + STEP < n) fetch(first + j + STEP);
                    else if (k + m.n_splits < rounds) fetch(first_tree(k + m.n_splits));
                }
                const int at = ((WalkTable)m.walk.position)[min(first + j, T - 1)];
                const WalkTop top = (WalkTop)(image + static_cast<int64_t>(at) * TREE_BYTES);
                const uint32_t tree_at = mine + (j % STEP) * TREE_BYTES;
                uint32_t idx[NR];
                walk_tree<D, NR>(tree_at, xa, top, idx);
                const char *leaves = reinterpret_cast<const char *>(m.walk.leaf_node) + (static_cast<int64_t>(at) << (D + 2)) - (tree_at >> 1);
                asm volatile("" : "+s"(leaves));  // keeps the base whole, so that the loads take a 32-bit offset
                if (j > 0) keep(j - 1);
#pragma unroll
                for (int r = 0; r < NR; ++r) id[r] = static_cast<uint32_t>(*(GlobalInts)((GlobalBytes)leaves + (idx[r] >> 1)));
            }
        }
#pragma unroll
        for (int j = 0; j < 4; ++j)
            if (j == n - 1) keep(j);
        const auto store = [&](int64_t row, int begin, int n, Vec2 id) {
            int32_t *dst = leaf_out + row * T + begin;
            const int32_t v[4] = {static_cast<int32_t>(id.x & 0xffff), static_cast<int32_t>(id.x >> 16),
                                  static_cast<int32_t>(id.y & 0xffff), static_cast<int32_t>(id.y >> 16)};
            if (n == 4 && begin + 4 <= T) {
                *reinterpret_cast<Int4 *>(dst) = Int4{{v[0], v[1], v[2], v[3]}};
            } else {
#pragma unroll
                for (int j = 0; j < 4; ++j)
                    if (j < n && begin + j < T) dst[j] = v[j];
            }
        };
        if (T <= 4) {  // a row's ids share 16 bytes: nothing to gain from an exchange
#pragma unroll
            for (int r = 0; r < NR; ++r)
                if (const int64_t row = row0 + r * TILE + lane; first < T && row < n_rows) leaf_out[row * T + first] = static_cast<int32_t>(ids[r][0]);
            return;
        }
        // A wave leaves the ids of its rows in its stage, those of row i at place i + 4 * wave, so that the 16 lanes
        // that read a row's ids from the 16 stages find them in different banks.
#pragma unroll
        for (int g = 0; g < NR; g += EXCHANGE) {
            constexpr int PLACES = EXCHANGE * TILE;
            if (g > 0) __syncthreads();  // the ids before are out of the stages
#pragma unroll
            for (int r = 0; r < EXCHANGE; ++r)
                lds_write<Vec2>(mine + ((r * TILE + lane + 4 * wave) & (PLACES - 1)) * 8, Vec2{ids[g + r][0], ids[g + r][1]});
            __syncthreads();
            const int from = lane & (WALK_WAVES - 1);  // the wave whose trees this lane writes
            const int begin = k * round + from * n;
#pragma unroll
            for (int i = 0; i < EXCHANGE; ++i) {
                const int li = (wave * EXCHANGE + i) * (TILE / WALK_WAVES) + lane / WALK_WAVES;  // a row of the exchange
                const Vec2 id = lds_read<Vec2>(from * STAGE_BYTES + ((li + 4 * from) & (PLACES - 1)) * 8);
                const int64_t row = row0 + g * TILE + li;
                if (row < n_rows) store(row, begin, n, id);
            }
        }
        __syncthreads();
    }
}

template <int D, int MODE>
KernelFn pick_groups(int groups)
{
    if constexpr (MODE == WALK_LEAVES)
        return groups == 1 ? forest_walk_leaves_kernel<D, 1> : groups == 2 ? forest_walk_leaves_kernel<D, 2> : forest_walk_leaves_kernel<D, 4>;
    else switch (groups) {
        case 1: return forest_walk_kernel<D, 1, MODE>;
        case 2: return forest_walk_kernel<D, 2, MODE>;
        default: return forest_walk_kernel<D, MODE == WALK_COLUMNS ? 2 : 4, MODE>;  // walk_max_groups
    }
}

template <int MODE>
KernelFn pick_depth(int depth, int groups)
{
    switch (depth) {
        case 3: return pick_groups<3, MODE>(groups);
        case 4: return pick_groups<4, MODE>(groups);
        case 5: return pick_groups<5, MODE>(groups);
        case 6: return pick_groups<6, MODE>(groups);
        case 7: return pick_groups<7, MODE>(groups);
        default: return pick_groups<8, MODE>(groups);
    }
}

KernelFn pick(int depth, int groups, int mode)
{
    if (mode == WALK_COLUMN) return pick_depth<WALK_COLUMN>(depth, groups);
    if (mode == WALK_COLUMNS) return pick_depth<WALK_COLUMNS>(depth, groups);
    return pick_depth<WALK_LEAVES>(depth, groups);
}

}  // namespace

hipError_t init_walk_kernels(size_t lds_limit)
{
    for (int mode : {WALK_COLUMN, WALK_COLUMNS, WALK_LEAVES})
        for (int depth = WALK_MIN_DEPTH; depth <= WALK_MAX_DEPTH; ++depth)
            for (int groups = 1; groups <= walk_max_groups(mode == WALK_COLUMNS ? 2 : 1); groups *= 2) {
                const void *fn = reinterpret_cast<const void *>(pick(depth, groups, mode));
                hipFuncAttributes attr;
                if (hipError_t e = hipFuncGetAttributes(&attr, fn); e != hipSuccess) return e;
                if (attr.sharedSizeBytes != 0) return hipErrorInvalidValue;  // the kernels address LDS from 0
                if (hipError_t e = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, static_cast<int>(lds_limit));
                    e != hipSuccess)
                    return e;
            }
    return hipSuccess;
}

hipError_t launch_walk(const DevModel &m, int groups, const float *X, int64_t n_rows, float *scores, int32_t *labels,
                       int32_t *leaf_out, hipStream_t stream)
{
    const int64_t n_blocks = (n_rows + TILE * groups - 1) / (TILE * groups);
    if (n_blocks > 0x7fffffffLL) return hipErrorInvalidValue;
    const dim3 grid(static_cast<unsigned>(n_blocks), static_cast<unsigned>(m.n_splits));
    const size_t lds = walk_lds_bytes(m.walk.depth, m.n_features, m.n_outputs, m.walk.groups);
    const int mode = leaf_out ? WALK_LEAVES : m.n_outputs == 1 ? WALK_COLUMN : WALK_COLUMNS;
    hipLaunchKernelGGL(pick(m.walk.depth, groups, mode), grid, dim3(WALK_WAVES * TILE), lds, stream, m, X,
                       n_rows, scores, labels, leaf_out);
    return hipGetLastError();
}

}  // namespace forest_impl
