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
// tree later, in fp64.  Trees of depth up to 6, of which a stage holds two, are walked two at a time: a level is two LDS
// round trips, and the second tree's fill the first one's (2000 x depth 6, 128 features, two row groups, 500,000 rows:
// 922 -> 828 us; 1000 x depth 6, 50 features, four row groups, 1M rows: 777 -> 758; 1,021 rows of the former, one row
// group: 17.4 -> 15.6 us a call).  Deeper trees would need a second stage in LDS, at the price of a workgroup's place.
//
// Bound: at depth 8 the LDS (90 % busy, vector ALU 79 %), at depth 6 the vector ALU (93 to 98 %) with the LDS (82 to 86 %)
// behind it.  Per (64 rows, tree of depth D): 3 + 2 (D - 2) LDS reads of 2 clocks each, more at levels 6 and 7 whose 64 and 128 nodes share the
// 32 banks (4 and 6 clocks).  500 trees of depth 8, 28 features, 1M rows: 2.70 -> 0.60 ms against every node tested
// (forest_kernels_rank.hip); 1000 of depth 6, 50 features: 1.57 -> 0.71 ms.  Leaf values held as float64, which saves
// their conversion and a shift: 633 and 802 us against 629 and 788.
#include <hip/hip_runtime.h>

#include <cstdint>
#include <type_traits>

#include "forest_device.hpp"
#include "forest_kernel_common.hpp"
#include "forest_walk_common.hpp"

namespace forest_impl {
namespace {

// The first words of a tree, wave-uniform: its output column, its caller's index, the nodes of two levels.
struct TreeHead {
    uint32_t w[8];
};

__device__ __forceinline__ TreeHead tree_head(const char *tree)
{
    TreeHead h;
#pragma unroll
    for (int i = 0; i < 8; ++i) h.w[i] = ((WalkTop)tree)[i];
    return h;
}

// NT trees, TREE_BYTES apart, all row groups: idx[j][r] = LDS address of tree j | 8 * (index of the leaf reached).
template <int D, int NR, int NT>
__device__ __forceinline__ void walk_trees(uint32_t tree_at, uint32_t xa, const TreeHead (&head)[NT], uint32_t (&idx)[NT][NR])
{
    float x1[NT][NR], x2[NT][NR], x3[NT][NR];
#pragma unroll
    for (int j = 0; j < NT; ++j) {
#pragma unroll
        for (int r = 0; r < NR; ++r) x1[j][r] = lds_read<float>(xa + head[j].w[3] + r * 256);
#pragma unroll
        for (int r = 0; r < NR; ++r) x2[j][r] = lds_read<float>(xa + head[j].w[5] + r * 256);
#pragma unroll
        for (int r = 0; r < NR; ++r) x3[j][r] = lds_read<float>(xa + head[j].w[7] + r * 256);
    }
#pragma unroll
    for (int j = 0; j < NT; ++j) {
        const float t1 = __uint_as_float(head[j].w[2]), t2 = __uint_as_float(head[j].w[4]), t3 = __uint_as_float(head[j].w[6]);
#pragma unroll
        for (int r = 0; r < NR; ++r) {
            const uint64_t m1 = __ballot(!(x1[j][r] <= t1)), m2 = __ballot(!(x2[j][r] <= t2)), m3 = __ballot(!(x3[j][r] <= t3));
            const uint64_t second = (m1 & m3) | (~m1 & m2);
            uint32_t b0, b1;
            asm("v_cndmask_b32 %0, 0, 8, %1" : "=v"(b0) : "s"(m1));
            asm("v_cndmask_b32 %0, 0, 16, %1" : "=v"(b1) : "s"(second));
            idx[j][r] = (tree_at + j * (8u << D)) | b0 | b1;
        }
    }
#pragma unroll
    for (int l = 2; l < D; ++l) {
        Vec2 node[NT][NR];
        float x[NT][NR];
#pragma unroll
        for (int j = 0; j < NT; ++j)
#pragma unroll
            for (int r = 0; r < NR; ++r) node[j][r] = lds_read<Vec2>(idx[j][r] + (8u << l));
#pragma unroll
        for (int j = 0; j < NT; ++j)
#pragma unroll
            for (int r = 0; r < NR; ++r) x[j][r] = lds_read<float>(xa + node[j][r].y + r * 256);
#pragma unroll
        for (int j = 0; j < NT; ++j)
#pragma unroll
            for (int r = 0; r < NR; ++r) {
                const int right = __float_as_int(__uint_as_float(node[j][r].x) - x[j][r]) >> 31;
                asm("v_and_or_b32 %0, %1, %2, %0" : "+v"(idx[j][r]) : "v"(right), "s"(8 << l));
            }
    }
}

// What a kernel leaves behind: the sums of one output column, those of several (trees sorted by
// column), or the leaf ids of every tree (a kernel of its own, in two forms).
enum { WALK_COLUMN = 0, WALK_COLUMNS = 1, WALK_LEAVES = 2, WALK_LEAVES_THROUGH = 3, WALK_FEW_LEAVES = 4 };

// The sums of a workgroup's rows, from row0.
template <int D, int NR, int MODE>
__device__ __forceinline__ void walk_rows(const DevModel m, const float *__restrict__ X, int64_t row0, int64_t n_rows, float *scores,
                                          int32_t *labels)
{
    constexpr int TREE_BYTES = 8 << D, STAGE_TREES = walk_stage_trees(D), STAGE_BYTES = TREE_BYTES * STAGE_TREES;
    constexpr int PIECES = STAGE_BYTES / 1024;  // 16 bytes per lane each
    static_assert(STAGE_BYTES % 1024 == 0, "whole 16-byte pieces per lane");
    extern __shared__ __align__(1024) char smem[];
    const int lane = threadIdx.x & (TILE - 1), wave = uniform(threadIdx.x >> 6);
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
    tile_fill<NR, NR == 4 ? 8 : 4, true>(X, row0, n_rows, m.x_tile, 17, xbase, 256, stride, wave, lane);
    __syncthreads();

    const uint32_t xa = xbase + lane * 4;
    constexpr int NT = STAGE_TREES > 1 ? 2 : 1;  // trees walked together
    ColumnSums<NR, MODE == WALK_COLUMNS ? WALK_MAX_COLUMNS : 1> sums;
    sums.begin(MODE == WALK_COLUMNS && s_begin < s_end ? ((WalkTable)(image + static_cast<int64_t>(s_begin) * STAGE_BYTES))[0] : 0);
    float value[NT][NR];  // the last trees' leaf values, not yet added to the running column
#pragma unroll
    for (int j = 0; j < NT; ++j)
#pragma unroll
        for (int r = 0; r < NR; ++r) value[j][r] = 0.0f;
    const auto add_value = [&](int j) {
#pragma unroll
        for (int r = 0; r < NR; ++r) sums.acc[r] += static_cast<double>(value[j][r]);
    };

    for (int s = s_begin; s < s_end; ++s) {
#pragma unroll
        for (int i = 0; i < PIECES; ++i) lds_write<Vec4>(mine + i * 1024 + lane * 16, ahead[i]);
        if (s + 1 < s_end) fetch(s + 1);
#pragma unroll 1
        for (int q = 0; q < STAGE_TREES; q += NT) {
            const int t = s * STAGE_TREES + q;
            TreeHead head[NT];
#pragma unroll
            for (int j = 0; j < NT; ++j) head[j] = tree_head(image + static_cast<int64_t>(t + j) * TREE_BYTES);
            const uint32_t tree_at = mine + q * TREE_BYTES;
            uint32_t idx[NT][NR];
            walk_trees<D, NR, NT>(tree_at, xa, head, idx);
#pragma unroll
            for (int j = 0; j < NT; ++j) add_value(j);
            // half an index is the leaf's byte offset; the tree's address in it is taken off the base
            const char *leaves = reinterpret_cast<const char *>(m.walk.leaf) + (static_cast<int64_t>(t) << (D + 2)) - (tree_at >> 1);
            asm volatile("" : "+s"(leaves));  // keeps the base whole, so that the loads take a 32-bit offset
#pragma unroll
            for (int j = 0; j < NT; ++j) {
                if (const int c = static_cast<int>(head[j].w[0]); MODE == WALK_COLUMNS && c != sums.column) {
                    if (j > 0) {  // the first of the two ends its column
                        add_value(0);
#pragma unroll
                        for (int r = 0; r < NR; ++r) value[0][r] = 0.0f;
                    }
                    sums.change(c);
                }
#pragma unroll
                for (int r = 0; r < NR; ++r) value[j][r] = *(GlobalFloats)((GlobalBytes)leaves + (idx[j][r] >> 1));
            }
        }
    }
#pragma unroll
    for (int j = 0; j < NT; ++j) add_value(j);
    finish_columns<NR, WALK_WAVES>(m, smem, wave, lane, s_begin < s_end, sums, row0, n_rows, scores, labels);
}

template <int D, int NR, int LAST, int MODE>
__global__ __launch_bounds__(WALK_WAVES * TILE, 8) void forest_walk_kernel(DevModel m, const float *__restrict__ X,
                                                                          int64_t n_rows, float *scores,
                                                                          int32_t *labels, int32_t *)
{
    bool after;
    const int64_t row0 = first_row(m, NR, LAST, after);
    if (after) walk_rows<D, LAST, MODE>(m, X, row0, n_rows, scores, labels);
    else walk_rows<D, NR, MODE>(m, X, row0, n_rows, scores, labels);
}

// The leaf ids of every tree, caller's order.  A row's ids are neighbours in the output and a lane holds those of few
// trees, so the waves take four trees each, side by side, and exchange the ids through their stages before they leave: a
// store then writes whole 256-byte runs of four rows.  Straight from the lanes, 16 bytes at the pitch of a row, 100,003
// rows of 200 x depth 6 took 65.6 us, three quarters of them for the stores; so 42.5 (250,000 rows of 200 x depth 3: 235 -> 65;
// 66,000 of 700 x depth 3: 310 -> 98), and 37.7 since a row's place comes from 32 bits and four ids are one value (IdStore; 45.4
// where results are not written over and over).  Ids of these trees, which have 511 nodes at most, fit 16 bits.  What is left of the trees after the last whole round is dealt evenly; waves that get none walk none
// (one tree of depth 7, 3 features, 60,000 rows: 4.6 us a call with 16 waves on it, 3.8).  FEW: of few trees
// (leaves_by_fours, forest_plan.hpp) a wave takes four and stores their ids from its lanes.  Bound: the walk, with 391
// workgroups for 256 CUs; two shares of the trees, or fewer rows per workgroup, fill the tile more often and took 54.7 and
// 50.4 when these took 42.5.
template <int D, int NR, int MODE>
__device__ __forceinline__ void walk_leaves(const DevModel m, const float *__restrict__ X, int64_t row0, int64_t n_rows, int32_t *leaf_out)
{
    constexpr bool FEW = MODE == WALK_FEW_LEAVES;
    constexpr int TREE_BYTES = 8 << D, STEP = walk_stage_trees(D) < 4 ? walk_stage_trees(D) : 4;  // trees copied at a time
    constexpr int STEP_BYTES = TREE_BYTES * STEP, STAGE_BYTES = walk_stage_bytes(D);
    constexpr int PIECES = (STEP_BYTES + 1023) / 1024;
    constexpr int EXCHANGE = NR * TILE * 8 <= STAGE_BYTES ? NR : STAGE_BYTES / (TILE * 8);  // row groups that a stage holds the ids of
    static_assert(NR % EXCHANGE == 0, "whole exchanges");
    extern __shared__ __align__(1024) char smem[];
    const int lane = threadIdx.x & (TILE - 1), wave = uniform(threadIdx.x >> 6);
    const int T = m.n_trees;
    const uint32_t stride = static_cast<uint32_t>(m.walk.groups) * 256, xbase = WALK_WAVES * STAGE_BYTES;
    const uint32_t mine = static_cast<uint32_t>(wave) * STAGE_BYTES;
    const int round = 4 * WALK_WAVES, rounds = FEW ? 1 : (T + round - 1) / round;

    const char *image = reinterpret_cast<const char *>(m.walk.node);
    // Trees each wave takes in a round (at most), and the first of this one's.
    const auto share = [&](int k) { return FEW || T - k * round >= round ? 4 : (T - k * round + WALK_WAVES - 1) / WALK_WAVES; };
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
    int k = FEW ? 0 : static_cast<int>(blockIdx.y);
    if (k < rounds && (!FEW || first_tree(k) < T)) fetch(first_tree(k));
    tile_fill<NR, NR == 4 ? 8 : 4, true>(X, row0, n_rows, m.x_tile, FEW && NR <= 2 ? 33 : 17, xbase, 256, stride, wave, lane);
    __syncthreads();

    const uint32_t xa = xbase + lane * 4;
    for (; k < rounds; k += m.n_splits) {
        const int first = first_tree(k), n = FEW ? min(4, T - first) : share(k);
        if (FEW && n <= 0) return;
        // of up to four trees, 16 bits each where they are exchanged; of the last tree, not yet among them
        uint32_t ids[NR][FEW ? 4 : 2] = {}, id[NR];
        const auto keep = [&](int j) {
#pragma unroll
            for (int r = 0; r < NR; ++r) ids[r][j >> 1] = (j & 1) ? ids[r][j >> 1] | id[r] << 16 : id[r];
        };
        const auto walk = [&](int j, auto trees) {  // trees j and, of two, j + 1
            constexpr int NT = decltype(trees)::value;
            int at[NT];
            TreeHead head[NT];
#pragma unroll
            for (int i = 0; i < NT; ++i) {
                at[i] = ((WalkTable)m.walk.position)[min(first + j + i, T - 1)];
                head[i] = tree_head(image + static_cast<int64_t>(at[i]) * TREE_BYTES);
            }
            const uint32_t tree_at = mine + (j % STEP) * TREE_BYTES;
            uint32_t idx[NT][NR];
            walk_trees<D, NR, NT>(tree_at, xa, head, idx);
            if (!FEW && j > 0) keep(j - 1);
#pragma unroll
            for (int i = 0; i < NT; ++i) {
                if (!FEW && i > 0) keep(j);
                const char *leaves = reinterpret_cast<const char *>(m.walk.leaf_node) + (static_cast<int64_t>(at[i]) << (D + 2)) -
                                     ((tree_at + i * TREE_BYTES) >> 1);
                asm volatile("" : "+s"(leaves));  // keeps the base whole, so that the loads take a 32-bit offset
#pragma unroll
                for (int r = 0; r < NR; ++r) {
                    uint32_t &to = FEW ? ids[r][FEW ? j + i : 0] : id[r];
                    to = static_cast<uint32_t>(*(GlobalInts)((GlobalBytes)leaves + (idx[i][r] >> 1)));
                }
            }
        };
        constexpr int NT = STEP > 1 && NR < 4 ? 2 : 1;  // trees walked together: four row groups' would spill (42.5 -> 44.5 us)
#pragma unroll
        for (int j = 0; j < 4; j += NT) {
            if (j < n && first < T) {
                if (j % STEP == 0) {
                    if (PIECES > 1 || lane * 16 < STEP_BYTES) {
#pragma unroll
                        for (int i = 0; i < PIECES; ++i) lds_write<Vec4>(mine + i * 1024 + lane * 16, ahead[i]);
                    }
                    if (j + STEP < n) fetch(first + j + STEP);
                    else if (!FEW && k + m.n_splits < rounds) fetch(first_tree(k + m.n_splits));
                }
                if (NT > 1 && j + 1 < n) walk(j, std::integral_constant<int, NT>{});
                else walk(j, std::integral_constant<int, 1>{});
            }
        }
#pragma unroll
        for (int j = 0; j < 4; ++j)
            if (!FEW && j == n - 1) keep(j);
        const IdStore<MODE == WALK_LEAVES_THROUGH> store{leaf_out + row0 * T, T};
        if (FEW || T <= 4) {  // straight from the lanes
#pragma unroll
            for (int r = 0; r < NR; ++r) {
                const int64_t row = row0 + r * TILE + lane;
                if (row >= n_rows || first >= T) continue;
                if constexpr (FEW) store(r * TILE + lane, first, 4, Vec4{ids[r][0], ids[r][1], ids[r][2], ids[r][3]});
                else leaf_out[row * T + first] = static_cast<int32_t>(ids[r][0]);
            }
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
                if (row0 + g * TILE + li < n_rows) store(g * TILE + li, begin, n, Vec4{id.x & 0xffff, id.x >> 16, id.y & 0xffff, id.y >> 16});
            }
        }
        __syncthreads();
    }
}

template <int D, int NR, int LAST, int MODE>
__global__ __launch_bounds__(WALK_WAVES * TILE, 8) void forest_walk_leaves_kernel(DevModel m, const float *__restrict__ X,
                                                                                 int64_t n_rows, float *, int32_t *,
                                                                                 int32_t *leaf_out)
{
    if constexpr (NR == LAST) {
        walk_leaves<D, NR, MODE>(m, X, static_cast<int64_t>(blockIdx.x) * (NR * TILE), n_rows, leaf_out);
    } else {
        bool after;
        const int64_t row0 = first_row(m, NR, LAST, after);
        if (after) walk_leaves<D, LAST, MODE>(m, X, row0, n_rows, leaf_out);
        else walk_leaves<D, NR, MODE>(m, X, row0, n_rows, leaf_out);
    }
}

template <int D, int NR, int LAST, int MODE>
KernelFn kernel()
{
    if constexpr (MODE == WALK_FEW_LEAVES) return forest_walk_leaves_kernel<D, NR, NR, MODE>;
    else if constexpr (MODE == WALK_LEAVES || MODE == WALK_LEAVES_THROUGH) return forest_walk_leaves_kernel<D, NR, LAST, MODE>;
    else return forest_walk_kernel<D, NR, LAST, MODE>;
}

// last: as groups where a launch has workgroups of one size.  Only leaf ids have a kernel of their own for that (0.5 %).
template <int D, int MODE>
KernelFn pick_groups(int groups, int last)
{
    constexpr int MOST = MODE == WALK_COLUMNS ? 2 : 4;  // walk_max_groups
    if constexpr (MODE == WALK_LEAVES || MODE == WALK_LEAVES_THROUGH)
        if (last == groups && groups > 1) return groups == 2 ? kernel<D, 2, 2, MODE>() : kernel<D, MOST, MOST, MODE>();
    switch (groups) {
        case 1: return kernel<D, 1, 1, MODE>();
        case 2: return kernel<D, 2, 1, MODE>();
        default: return last == 1 ? kernel<D, MOST, 1, MODE>() : kernel<D, MOST, MOST / 2, MODE>();
    }
}

template <int MODE>
KernelFn pick_depth(int depth, int groups, int last)
{
    switch (depth) {
        case 3: return pick_groups<3, MODE>(groups, last);
        case 4: return pick_groups<4, MODE>(groups, last);
        case 5: return pick_groups<5, MODE>(groups, last);
        case 6: return pick_groups<6, MODE>(groups, last);
        case 7: return pick_groups<7, MODE>(groups, last);
        default: return pick_groups<8, MODE>(groups, last);
    }
}

KernelFn pick(int depth, int groups, int last, int mode)
{
    if (mode == WALK_COLUMN) return pick_depth<WALK_COLUMN>(depth, groups, last);
    if (mode == WALK_COLUMNS) return pick_depth<WALK_COLUMNS>(depth, groups, last);
    if (mode == WALK_LEAVES) return pick_depth<WALK_LEAVES>(depth, groups, last);
    if (mode == WALK_LEAVES_THROUGH) return pick_depth<WALK_LEAVES_THROUGH>(depth, groups, last);
    return pick_depth<WALK_FEW_LEAVES>(depth, groups, last);
}

}  // namespace

hipError_t init_walk_kernels(size_t lds_limit)
{
    for (int mode : {WALK_COLUMN, WALK_COLUMNS, WALK_LEAVES, WALK_LEAVES_THROUGH, WALK_FEW_LEAVES})
        for (int depth = WALK_MIN_DEPTH; depth <= WALK_MAX_DEPTH; ++depth)
            for (int groups = 1; groups <= walk_max_groups(mode == WALK_COLUMNS ? 2 : 1); groups *= 2)
                for (int last = 1; last <= groups; last *= 2) {
                    const void *fn = reinterpret_cast<const void *>(pick(depth, groups, last, mode));
                    hipFuncAttributes attr;
                    if (hipError_t e = hipFuncGetAttributes(&attr, fn); e != hipSuccess) return e;
                    if (attr.sharedSizeBytes != 0) return hipErrorInvalidValue;  // the kernels address LDS from 0
                    if (hipError_t e = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, static_cast<int>(lds_limit));
                        e != hipSuccess)
                        return e;
                }
    return hipSuccess;
}

hipError_t launch_walk(const DevModel &m, int groups, const TailPlan &t, const float *X, int64_t n_rows, float *scores, int32_t *labels,
                       int32_t *leaf_out, hipStream_t stream)
{
    int mode = m.n_outputs == 1 ? WALK_COLUMN : WALK_COLUMNS;
    if (leaf_out) mode = leaves_by_fours(m, groups, n_rows) ? WALK_FEW_LEAVES : ids_go_through(m.n_trees, n_rows, reinterpret_cast<uintptr_t>(leaf_out)) ? WALK_LEAVES_THROUGH : WALK_LEAVES;
    if (t.full + t.after > 0x7fffffffLL) return hipErrorInvalidValue;
    const dim3 grid(static_cast<unsigned>(t.full + t.after), static_cast<unsigned>(m.n_splits));
    const size_t lds = walk_lds_bytes(m.walk.depth, m.n_features, m.n_outputs, m.walk.groups);
    hipLaunchKernelGGL(pick(m.walk.depth, groups, t.groups, mode), grid, dim3(WALK_WAVES * TILE), lds, stream, m, X,
                       n_rows, scores, labels, leaf_out);
    return hipGetLastError();
}

}  // namespace forest_impl
