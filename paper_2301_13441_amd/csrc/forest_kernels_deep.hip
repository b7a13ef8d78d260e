// Deep walk kernels (gfx950): trees of any shape and depth, scalar or vector leaves, one node per
// level and row.
//
// The top DEEP_TOP levels of a tree go as in the walk kernels (forest_kernels_walk.hip): laid out as
// a full tree, the first two levels through scalar loads, below them one node per level out of the
// wave's stage in LDS, and there the path ends on a unit (forest_model.hpp): for most rows of an
// irregular tree their leaf.  The other rows go on through the units, which their lanes gather from
// global memory, the lanes that have met their leaf masked off.  A subtree's units are contiguous,
// so a lane finds most of its path in the line or two that its first unit came with, and the path
// ends on the leaf's value itself.
//
// A workgroup of 16 waves owns NR x 64 rows, whose features it holds in LDS as float32
// ([group][feature][row]); every wave walks its own run of trees for all the rows, two trees at a time
// below their tops.
//
// Where a CU holds one workgroup, large batches run a kernel of their own for the sums (forest_deep_tiles_kernel), whose
// workgroups take tile after tile.  128 trees of depth 12, 256 features, 4,000,000 rows: 2.15 ms (a workgroup per tile 2.71;
// 14.5 with every node tested, forest_kernels_rankbank.hip).
//
// In the kernel with a workgroup per tile: keeping 64-row tiles, two workgroups on a CU and the first units in global memory,
// 2.90 ms there, 94 us against 87 for 300 trees of depth 9 over 90 features and 103,069 rows.
#include <hip/hip_runtime.h>

#include <cstdint>
#include <type_traits>

#include "forest_device.hpp"
#include "forest_kernel_common.hpp"
#include "forest_walk_common.hpp"

namespace forest_impl {
namespace {

// What a kernel leaves behind: the sums of one output column, those of several (trees sorted by
// column), those of vector leaves, or the leaf ids of every tree (FEW: of few trees, leaves_by_fours in forest_plan.hpp).
enum { DEEP_COLUMN = 0, DEEP_COLUMNS = 1, DEEP_VECTOR = 2, DEEP_LEAVES = 3, DEEP_LEAVES_THROUGH = 4, DEEP_FEW_LEAVES = 5 };

constexpr uint32_t TOP_BYTES = DEEP_TOP_WORDS * sizeof(WalkNode);     // of a tree
constexpr uint32_t NODES_BYTES = TOP_BYTES / 2;                        // its nodes, and as much for its first units
static_assert(NODES_BYTES == 64 * 16, "a lane copies 16 bytes of either");
constexpr uint32_t XBASE = DEEP_WAVES * TOP_BYTES;  // LDS: the waves' nodes, their first units, the X tile

#if defined(__HIP_DEVICE_COMPILE__)
typedef const __attribute__((address_space(1))) Vec2 *GlobalUnits;
#else
typedef const Vec2 *GlobalUnits;
#endif

// The first words of a tree's top, wave-uniform: its first unit, its column, the nodes of two levels.
struct DeepHead {
    uint32_t w[8];
};

__device__ __forceinline__ DeepHead deep_head(const char *tops, int at)
{
    const WalkTop p = (WalkTop)(tops + static_cast<int64_t>(at) * TOP_BYTES);
    DeepHead h;
#pragma unroll
    for (int i = 0; i < 8; ++i) h.w[i] = p[i];
    return h;
}

// The top of one tree, all row groups: where the path goes on, as the byte offset from the tree's first
// unit, and the unit there.
template <int NR>
__device__ __forceinline__ void deep_top(uint32_t stage, const uint32_t (&xa)[NR], const DeepHead &head, uint32_t (&at)[NR],
                                         Vec2 (&what)[NR])
{
    const uint32_t (&top)[8] = head.w;
    const float t1 = __uint_as_float(top[2]), t2 = __uint_as_float(top[4]), t3 = __uint_as_float(top[6]);
    float x1[NR], x2[NR], x3[NR];
    uint32_t idx[NR];
#pragma unroll
    for (int r = 0; r < NR; ++r) x1[r] = lds_read<float>(xa[r] + top[3]);
#pragma unroll
    for (int r = 0; r < NR; ++r) x2[r] = lds_read<float>(xa[r] + top[5]);
#pragma unroll
    for (int r = 0; r < NR; ++r) x3[r] = lds_read<float>(xa[r] + top[7]);
#pragma unroll
    for (int r = 0; r < NR; ++r) {
        const uint64_t m1 = __ballot(!(x1[r] <= t1)), m2 = __ballot(!(x2[r] <= t2)), m3 = __ballot(!(x3[r] <= t3));
        const uint64_t second = (m1 & m3) | (~m1 & m2);
        uint32_t b0, b1;
        asm("v_cndmask_b32 %0, 0, 8, %1" : "=v"(b0) : "s"(m1));
        asm("v_cndmask_b32 %0, 0, 16, %1" : "=v"(b1) : "s"(second));
        idx[r] = stage | b0 | b1;
    }
#pragma unroll
    for (int l = 2; l < DEEP_TOP; ++l) {
        Vec2 node[NR];
        float x[NR];
#pragma unroll
        for (int r = 0; r < NR; ++r) node[r] = lds_read<Vec2>(idx[r] + (8u << l));
#pragma unroll
        for (int r = 0; r < NR; ++r) x[r] = lds_read<float>(xa[r] + node[r].y);
#pragma unroll
        for (int r = 0; r < NR; ++r) idx[r] |= x[r] <= __uint_as_float(node[r].x) ? 0u : 8u << l;
    }
#pragma unroll
    for (int r = 0; r < NR; ++r) what[r] = lds_read<Vec2>(idx[r] + DEEP_WAVES * NODES_BYTES);
#pragma unroll
    for (int r = 0; r < NR; ++r) at[r] = idx[r] - stage;
}

// A workgroup's rows, from row0.
template <int NR, int MODE, int WP>
__device__ __forceinline__ void deep_rows(const DevModel m, const float *__restrict__ X, int64_t row0, int64_t n_rows, float *scores,
                                          int32_t *labels, int32_t *leaf_out)
{
    constexpr int ROWS = NR * TILE;
    constexpr bool FEW = MODE == DEEP_FEW_LEAVES, LEAVES = MODE == DEEP_LEAVES || MODE == DEEP_LEAVES_THROUGH || FEW;
    constexpr int W = LEAVES ? 1 : WP;
    constexpr int NT = 2;  // trees whose units are walked together
    static_assert(MODE == DEEP_VECTOR || WP == 1, "scalar leaves");
    extern __shared__ __align__(1024) char smem[];
    const int lane = threadIdx.x & (TILE - 1), wave = uniform(threadIdx.x >> 6);
    const int F = m.n_features, T = m.n_trees;
    const uint32_t group_stride = static_cast<uint32_t>(F) * 256;
    const uint32_t stage = static_cast<uint32_t>(wave) * NODES_BYTES;

    // This wave's trees: a contiguous run for the sums; for the leaf ids, which have the caller's order, up to four in
    // turn, so that the waves have neighbouring ids at the same time (forest_kernels_walk.hip).
    const int unit = static_cast<int>(blockIdx.y) * DEEP_WAVES + wave, units = m.n_splits * DEEP_WAVES;
    constexpr int ROUND = 4 * DEEP_WAVES;
    const auto share = [&](int k) { return FEW || T - k * ROUND >= ROUND ? 4 : (T - k * ROUND + DEEP_WAVES - 1) / DEEP_WAVES; };
    const auto first_tree = [&](int k) { return k * ROUND + wave * share(k); };
    const int t_begin = LEAVES ? first_tree(FEW ? 0 : blockIdx.y) : static_cast<int>(static_cast<int64_t>(T) * unit / units);
    const int t_end = LEAVES ? T : static_cast<int>(static_cast<int64_t>(T) * (unit + 1) / units);
    auto place = [&](int t) { return LEAVES ? ((WalkTable)m.deep.position)[t] : t; };

    const char *tops = reinterpret_cast<const char *>(m.deep.top);
    Vec4 ahead[2];
    DeepHead head = {};  // of the tree whose top comes next
    auto fetch = [&](int at) {
#pragma unroll
        for (int i = 0; i < 2; ++i)
            ahead[i] = *reinterpret_cast<const Vec4 *>(tops + static_cast<int64_t>(at) * TOP_BYTES + i * NODES_BYTES + lane * 16);
    };
    if (t_begin < t_end) {
        fetch(place(t_begin));
        head = deep_head(tops, place(t_begin));
    }
    tile_fill<NR, NR == 2 ? 8 : 4, false>(X, row0, n_rows, m.x_tile, 17, XBASE, group_stride, 256, wave, lane);
    __syncthreads();

    uint32_t xa[NR];
#pragma unroll
    for (int r = 0; r < NR; ++r) xa[r] = XBASE + static_cast<uint32_t>(r) * group_stride + lane * 4;

    double acc[W][NR];  // vector leaves
#pragma unroll
    for (int k = 0; k < W; ++k)
#pragma unroll
        for (int r = 0; r < NR; ++r) acc[k][r] = 0.0;
    ColumnSums<NR, MODE == DEEP_COLUMNS ? WALK_MAX_COLUMNS : 1> sums;
    sums.begin(MODE == DEEP_COLUMNS && t_begin < t_end ? static_cast<int>(head.w[1]) : 0);

    // The lanes' places in the units of the trees at hand: byte offset from the tree's first unit, and
    // what is there.
    uint32_t at[NT][NR];
    Vec2 what[NT][NR];
    const char *units_of[NT];  // the trees' first units (wave-uniform)
    uint32_t first_unit[NT];
    int tree_column[NT];
    const uint32_t last_feature = static_cast<uint32_t>(F) - 1;
    // What bounds a step of these is the texture path (a gather of 8 bytes takes 16 clocks and more, however few its lanes)
    // and, one after the other, the trip to LDS for the features and that to the L2 for the units.  All the features are
    // read before the first is waited for, and the next step is asked for behind the last one, so that nothing is copied
    // (4M rows of 128 x depth 12, 256 features: 2813 -> 2706 us; 103,069 rows of 300 x depth 9, 90 features: 73.3 -> 72.2).
    const auto at_a_node = [&](int j, int r) { return __builtin_isnan(__uint_as_float(what[j][r].y)); };
    const auto any_at_a_node = [&]() {
        bool any = false;
#pragma unroll
        for (int j = 0; j < NT; ++j)
#pragma unroll
            for (int r = 0; r < NR; ++r) any |= at_a_node(j, r);
        return __any(any) != 0;
    };
    auto go_on = [&]() {
        if (!any_at_a_node()) return;
        do {
            float x[NT][NR];
#pragma unroll
            for (int j = 0; j < NT; ++j)
#pragma unroll
                for (int r = 0; r < NR; ++r) {
                    // a lane at its leaf reads any feature there is: the first, or at 2-wide leaves what their bits say
                    uint32_t f = __builtin_amdgcn_ubfe(what[j][r].y, 14, 9);
                    if (LEAVES || WP == 2) f = min(f, last_feature);
                    x[j][r] = lds_read<float>(xa[r] + (f << 8));
                }
#pragma unroll
            for (int j = 0; j < NT; ++j)
#pragma unroll
                for (int r = 0; r < NR; ++r) asm volatile("" : "+v"(x[j][r]));
#pragma unroll
            for (int j = 0; j < NT; ++j)
#pragma unroll
                for (int r = 0; r < NR; ++r)
                    if (at_a_node(j, r)) {
                        const uint32_t step = (what[j][r].y & DEEP_MAX_DISTANCE) + (x[j][r] <= __uint_as_float(what[j][r].x) ? 0u : 1u);
                        at[j][r] += step << 3;
                        what[j][r] = *(GlobalUnits)((GlobalBytes)units_of[j] + at[j][r]);
                    }
        } while (any_at_a_node());
    };
    auto add_values = [&](int j) {
        if (MODE != DEEP_VECTOR) {
#pragma unroll
            for (int r = 0; r < NR; ++r) sums.acc[r] += static_cast<double>(__uint_as_float(what[j][r].x));
        } else if (WP <= 2) {
#pragma unroll
            for (int r = 0; r < NR; ++r) {
                acc[0][r] += static_cast<double>(__uint_as_float(what[j][r].x));
                if (W == 2) acc[W - 1][r] += static_cast<double>(__uint_as_float(what[j][r].y));
            }
        } else {
#pragma unroll
            for (int r = 0; r < NR; ++r) {
                const Vec4 *v = reinterpret_cast<const Vec4 *>(m.deep.value + static_cast<size_t>(what[j][r].x) * WP);
#pragma unroll
                for (int q = 0; q < WP / 4; ++q) {
                    const Vec4 p = v[q];
#pragma unroll
                    for (int i = 0; i < 4; ++i) acc[(4 * q + i) % W][r] += static_cast<double>(__uint_as_float(p[i]));
                }
            }
        }
    };
    // The top of tree t (j: its place in the pair); the next tree's top is on its way from here on.
    auto take = [&](int j, int t_after) {
        lds_write<Vec4>(stage + lane * 16, ahead[0]);
        lds_write<Vec4>(stage + DEEP_WAVES * NODES_BYTES + lane * 16, ahead[1]);
        const DeepHead here = head;
        first_unit[j] = here.w[0];
        tree_column[j] = static_cast<int>(here.w[1]);
        units_of[j] = reinterpret_cast<const char *>(m.deep.unit) + static_cast<int64_t>(here.w[0]) * 8;
        asm volatile("" : "+s"(units_of[j]));  // keeps the base whole, so that the loads take a 32-bit offset
        if (t_after < t_end) {
            const int next = place(t_after);
            fetch(next);
            head = deep_head(tops, next);
        }
        deep_top<NR>(stage, xa, here, at[j], what[j]);
    };
    // One or two trees, from their tops to their leaves; the tree after them.
    const auto walk = [&](int t, bool two, int after) {
        take(0, two ? t + 1 : after);
        if (two) {
            take(1, after);
        } else {
#pragma unroll
            for (int r = 0; r < NR; ++r) what[1][r] = Vec2{0, 0};
        }
        go_on();
    };
    if constexpr (!LEAVES) {
        for (int t = t_begin; t < t_end; t += NT) {
            const bool two = t + 1 < t_end;
            walk(t, two, t + NT);
#pragma unroll
            for (int j = 0; j < NT; ++j) {
                if (j > 0 && !two) break;
                if (MODE == DEEP_COLUMNS && tree_column[j] != sums.column) sums.change(tree_column[j]);
                add_values(j);
            }
        }
    } else {
        const int rounds = FEW ? 1 : (T + ROUND - 1) / ROUND;
        for (int k = FEW ? 0 : static_cast<int>(blockIdx.y); k < rounds; k += m.n_splits) {
            const int n = share(k), first = first_tree(k), own = min(T - first, n);
            if (FEW && own <= 0) return;
            const int next = !FEW && k + m.n_splits < rounds ? first_tree(k + m.n_splits) : T;
            uint32_t ids[NR][4] = {};
#pragma unroll
            for (int p = 0; p < 4; p += NT) {
                if (p < own) {
                    walk(first + p, p + 1 < own, p + NT < own ? first + p + NT : next);
#pragma unroll
                    for (int j = 0; j < NT; ++j) {
                        if (j > 0 && p + j >= own) break;
                        const int32_t *node = m.deep.unit_node + first_unit[j];
#pragma unroll
                        for (int r = 0; r < NR; ++r) ids[r][p + j] = static_cast<uint32_t>(node[at[j][r] >> 3]);
                    }
                }
            }
            const IdStore<MODE == DEEP_LEAVES_THROUGH> store{leaf_out + row0 * T, T};
            if (FEW || T <= 4) {  // straight from the lanes
#pragma unroll
                for (int r = 0; r < NR; ++r) {
                    const int64_t row = row0 + r * TILE + lane;
                    if (row >= n_rows || own <= 0) continue;
                    if (FEW) store(r * TILE + lane, first, 4, Vec4{ids[r][0], ids[r][1], ids[r][2], ids[r][3]});
                    else leaf_out[row * T + first] = static_cast<int32_t>(ids[r][0]);
                }
                return;
            }
            // A row group's ids meet in one half of the stages, those of row i at place i + 4 * wave of its wave's part.
#pragma unroll
            for (int r = 0; r < NR; ++r)
                lds_write<Vec4>(r * DEEP_WAVES * NODES_BYTES + stage + ((lane + 4 * wave) & (TILE - 1)) * 16, Vec4{ids[r][0], ids[r][1], ids[r][2], ids[r][3]});
            __syncthreads();
            const int from = lane & (DEEP_WAVES - 1);  // the wave whose trees this lane writes
#pragma unroll
            for (int r = 0; r < NR; ++r) {
                const int li = wave * (TILE / DEEP_WAVES) + lane / DEEP_WAVES;
                const Vec4 id = lds_read<Vec4>(r * DEEP_WAVES * NODES_BYTES + from * NODES_BYTES + ((li + 4 * from) & (TILE - 1)) * 16);
                if (row0 + r * TILE + li < n_rows) store(r * TILE + li, k * ROUND + from * n, n, id);
            }
            __syncthreads();
        }
    }
    if constexpr (MODE == DEEP_VECTOR) {
        // The waves' sums meet in LDS, in the order of the waves: [DEEP_WAVES][K][ROWS], of which the first takes the totals.
        const int K = m.n_outputs;
        double *slot = reinterpret_cast<double *>(smem);
        __syncthreads();
#pragma unroll
        for (int k = 0; k < W; ++k)
            if (k < K) {
#pragma unroll
                for (int r = 0; r < NR; ++r) slot[(wave * K + k) * ROWS + r * TILE + lane] = acc[k][r];
            }
        __syncthreads();
        for (int i = threadIdx.x; i < K * ROWS; i += DEEP_WAVES * TILE) {
            double s = 0.0;
#pragma unroll
            for (int w = 0; w < DEEP_WAVES; ++w) s += slot[w * K * ROWS + i];
            const int k = i / ROWS;
            const int64_t row = row0 + (i - k * ROWS);
            if (m.n_splits == 1) slot[i] = s;
            else if (row < n_rows) m.partial[(static_cast<int64_t>(blockIdx.y) * m.split_rows + row) * K + k] = s;
        }
        if (m.n_splits > 1) return;
        __syncthreads();
        for (int li = threadIdx.x; li < ROWS; li += DEEP_WAVES * TILE)
            if (row0 + li < n_rows) finish_values(m, slot + li, ROWS, row0 + li, scores, labels);
    } else if constexpr (!LEAVES) {
        finish_columns<NR, DEEP_WAVES>(m, smem, wave, lane, t_begin < t_end, sums, row0, n_rows, scores, labels);
    }
}

// SHARED: two workgroups on a CU (64 vector registers per lane), or one.
template <int NR, int LAST, int MODE, int WP, bool SHARED>
__global__ __launch_bounds__(DEEP_WAVES * TILE, SHARED ? 8 : 4) void forest_deep_kernel(DevModel m, const float *__restrict__ X,
                                                                                       int64_t n_rows, float *scores,
                                                                                       int32_t *labels, int32_t *leaf_out)
{
    bool after;
    const int64_t row0 = first_row(m, NR, LAST, after);
    if (after) deep_rows<LAST, MODE, WP>(m, X, row0, n_rows, scores, labels, leaf_out);
    else deep_rows<NR, MODE, WP>(m, X, row0, n_rows, scores, labels, leaf_out);
}

// The tops of NT trees whose nodes stand NODES_BYTES apart, all row groups: idx = the tree's LDS address | 8 * (leaf slot reached).
template <int NT, int NR>
__device__ __forceinline__ void deep_tops(uint32_t stage, const uint32_t (&xa)[NR], const DeepHead (&head)[NT], uint32_t (&idx)[NT][NR])
{
    float x1[NT][NR], x2[NT][NR], x3[NT][NR];
#pragma unroll
    for (int j = 0; j < NT; ++j)
#pragma unroll
        for (int r = 0; r < NR; ++r) {
            x1[j][r] = lds_read<float>(xa[r] + head[j].w[3]);
            x2[j][r] = lds_read<float>(xa[r] + head[j].w[5]);
            x3[j][r] = lds_read<float>(xa[r] + head[j].w[7]);
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
            idx[j][r] = (stage + j * NODES_BYTES) | b0 | b1;
        }
    }
#pragma unroll
    for (int l = 2; l < DEEP_TOP; ++l) {
        Vec2 node[NT][NR];
        float x[NT][NR];
#pragma unroll
        for (int j = 0; j < NT; ++j)
#pragma unroll
            for (int r = 0; r < NR; ++r) node[j][r] = lds_read<Vec2>(idx[j][r] + (8u << l));
#pragma unroll
        for (int j = 0; j < NT; ++j)
#pragma unroll
            for (int r = 0; r < NR; ++r) x[j][r] = lds_read<float>(xa[r] + node[j][r].y);
#pragma unroll
        for (int j = 0; j < NT; ++j)
#pragma unroll
            for (int r = 0; r < NR; ++r) idx[j][r] = x[j][r] <= __uint_as_float(node[j][r].x) ? idx[j][r] : idx[j][r] | 8u << l;
    }
}

// The sums of tile after tile, by workgroups that have a CU to themselves (takes_tiles, forest_plan.hpp): the rows of the next
// tile are on their way from memory to registers while this one is walked, and the tops of two trees are walked together, in
// turn with their units in the same stage.
//
// What bounds it is the CU's vector memory path, which returns loads in the order they were asked for, whichever wave did.  A tile's
// rows hold up everybody's units behind them for as long as they take from memory, so they are asked for once a tile, before
// the sums and the first tops, which need no memory (asked for before every two trees 2.75 ms, once behind the barrier of the sums
// 2.6), and in whole lines: eight rows' 128 bytes a load; with 64 bytes of 16 rows, whose lines the non-temporal policy drops between
// their halves, 2.31 ms (a tile on an otherwise idle chip 4.3 us instead of 2.0, with all CUs at it 5.4 instead of 4.7).  Then the units: 33 lines from the L2 per tree and 64 rows, 64 bytes a
// clock; 24 lanes have a path beyond the top, and what a step reads of a line is often gone before the next.  Gathered into whole
// waves through LDS the lanes ask for as many lines, in a longer chain: 1.36 ms of units instead of 0.9.  Without X it would take
// 1.83 ms, without units 1.23, without either 0.89 (LDS 62 % busy).  All the tops of four pairs of trees before their units, so that
// X waits behind more of them: 2.45 ms instead of 2.31.
template <int NR, int MODE, int WP, bool ONCE>
__global__ __launch_bounds__(DEEP_WAVES * TILE, 4) void forest_deep_tiles_kernel(DevModel model, const float *__restrict__ X, int64_t n_rows,
                                                                                float *scores, int32_t *labels, int32_t *)
{
    constexpr int ROWS = NR * TILE, W = WP, NT = 2;
    static_assert(MODE == DEEP_COLUMN ? WP == 1 : MODE == DEEP_VECTOR && WP == 2, "sums that fit the waves' stages");
    static_assert(DEEP_WAVES * W * ROWS * sizeof(double) <= XBASE, "sums that fit the waves' stages");
    const int lane = threadIdx.x & (TILE - 1), wave = uniform(threadIdx.x >> 6);
    const int F = model.n_features, T = model.n_trees;
    const uint32_t group_stride = static_cast<uint32_t>(F) * 256;
    const uint32_t stage = static_cast<uint32_t>(wave) * TOP_BYTES;  // of two trees, the nodes or the first units
    const int t_begin = T * wave / DEEP_WAVES, t_end = T * (wave + 1) / DEEP_WAVES;

    Vec4 nodes[NT], units[NT];  // of the pair that comes next
    // 16 bytes a lane of what stands `from` bytes behind the tops of trees t and t + 1
    const auto top_of = [&](int t) { return reinterpret_cast<const char *>(model.deep.top) + static_cast<int64_t>(min(t, T - 1)) * TOP_BYTES; };
    const auto fetch = [&](Vec4 (&to)[NT], int t, uint32_t from) {
#pragma unroll
        for (int j = 0; j < NT; ++j) {
            const char *top = top_of(t + j);
            uint32_t mine = lane * 16;
            asm volatile("" : "+s"(top), "+v"(mine));
            to[j] = *(GlobalVec4)((GlobalBytes)top + from + mine);
        }
    };
    constexpr int STEP = static_cast<int>(CUS) * ROWS;  // from a workgroup's tile to its next one
    const int n = static_cast<int>(n_rows);
    TileAhead<NR, ONCE> ahead;
    const auto request = [&](int row0) {
        if (row0 < n) ahead.request(X + static_cast<int64_t>(row0) * F, min(ROWS, n - row0), F, wave, lane);
    };
    int row0 = static_cast<int>(blockIdx.x) * ROWS;
    request(row0);
    fetch(nodes, t_begin, 0);
    fetch(units, t_begin, NODES_BYTES);
    ahead.store(F, XBASE, group_stride, 256, wave, lane);
    request(row0 + STEP);

    uint32_t xa[NR];
#pragma unroll
    for (int r = 0; r < NR; ++r) xa[r] = XBASE + static_cast<uint32_t>(r) * group_stride + lane * 4;
    double total[W];
    bool sums_there = false;  // of the tile before, whose rows' threads have them in `total`
    for (;;) {
        __syncthreads();
        if (sums_there && threadIdx.x < ROWS) finish_few<W>(model, total, row0 - STEP + static_cast<int>(threadIdx.x), scores, labels);

        double acc[W][NR];
#pragma unroll
        for (int k = 0; k < W; ++k)
#pragma unroll
            for (int r = 0; r < NR; ++r) acc[k][r] = 0.0;
        for (int t = t_begin; t < t_end; t += NT) {
            const bool two = t + 1 < t_end;
            uint32_t idx[NT][NR];
            DeepHead head[NT];
            uint32_t pieces = stage + lane * 16;
            asm volatile("" : "+v"(pieces));
#pragma unroll
            for (int j = 0; j < NT; ++j) {
                head[j] = deep_head(top_of(t + j), 0);
            }
#pragma unroll
            for (int j = 0; j < NT; ++j) lds_write<Vec4>(pieces + j * NODES_BYTES, nodes[j]);
            deep_tops<NT, NR>(stage, xa, head, idx);
#pragma unroll
            for (int j = 0; j < NT; ++j) lds_write<Vec4>(pieces + j * NODES_BYTES, units[j]);
            const int after = t + NT < t_end ? t + NT : t_begin;
            fetch(nodes, after, 0);
            fetch(units, after, NODES_BYTES);

            Vec2 what[NT][NR];
            uint32_t at[NT][NR];
#pragma unroll
            for (int j = 0; j < NT; ++j)
#pragma unroll
                for (int r = 0; r < NR; ++r) {
                    what[j][r] = lds_read<Vec2>(idx[j][r]);
                    at[j][r] = idx[j][r] - (stage + j * NODES_BYTES);
                }
            if (!two) {
#pragma unroll
                for (int r = 0; r < NR; ++r) what[1][r] = Vec2{0, 0};
            }
            const char *units_of[NT];
#pragma unroll
            for (int j = 0; j < NT; ++j) {
                units_of[j] = reinterpret_cast<const char *>(model.deep.unit) + static_cast<int64_t>(head[j].w[0]) * 8;
                asm volatile("" : "+s"(units_of[j]));
            }
            const auto at_a_node = [&](int j, int r) { return __builtin_isnan(__uint_as_float(what[j][r].y)); };
            const auto any_at_a_node = [&]() {
                bool any = false;
#pragma unroll
                for (int j = 0; j < NT; ++j)
#pragma unroll
                    for (int r = 0; r < NR; ++r) any |= at_a_node(j, r);
                return __any(any) != 0;
            };
            if (any_at_a_node()) {
                do {
                    float x[NT][NR];
#pragma unroll
                    for (int j = 0; j < NT; ++j)
#pragma unroll
                        for (int r = 0; r < NR; ++r) {
                            uint32_t f = __builtin_amdgcn_ubfe(what[j][r].y, 14, 9);
                            if (WP == 2) f = min(f, static_cast<uint32_t>(F) - 1);
                            x[j][r] = lds_read<float>(xa[r] + (f << 8));
                        }
#pragma unroll
                    for (int j = 0; j < NT; ++j)
#pragma unroll
                        for (int r = 0; r < NR; ++r) asm volatile("" : "+v"(x[j][r]));
#pragma unroll
                    for (int j = 0; j < NT; ++j)
#pragma unroll
                        for (int r = 0; r < NR; ++r)
                            if (at_a_node(j, r)) {
                                at[j][r] += ((what[j][r].y & DEEP_MAX_DISTANCE) + (x[j][r] <= __uint_as_float(what[j][r].x) ? 0u : 1u)) << 3;
                                what[j][r] = *(GlobalUnits)((GlobalBytes)units_of[j] + at[j][r]);
                            }
                } while (any_at_a_node());
            }
#pragma unroll
            for (int j = 0; j < NT; ++j) {
                if (j > 0 && !two) break;
#pragma unroll
                for (int r = 0; r < NR; ++r) {
                    acc[0][r] += static_cast<double>(__uint_as_float(what[j][r].x));
                    if (W == 2) acc[W - 1][r] += static_cast<double>(__uint_as_float(what[j][r].y));
                }
            }
        }
        __syncthreads();  // the tile and the stages are free
        uint32_t sums = lane * 8;  // [DEEP_WAVES][W][ROWS]
        asm volatile("" : "+v"(sums));
#pragma unroll
        for (int k = 0; k < W; ++k)
#pragma unroll
            for (int r = 0; r < NR; ++r) lds_write<double>(sums + wave * (W * ROWS * 8) + (k * ROWS + r * TILE) * 8, acc[k][r]);
        if (row0 + STEP < n) {
            ahead.store(F, XBASE, group_stride, 256, wave, lane);
            request(row0 + 2 * STEP);
        }
        __syncthreads();
        if (threadIdx.x < ROWS) {
            sums = threadIdx.x * 8;
            asm volatile("" : "+v"(sums));
#pragma unroll
            for (int k = 0; k < W; ++k) {
                total[k] = 0.0;
#pragma unroll
                for (int w = 0; w < DEEP_WAVES; ++w) total[k] += lds_read<double>(sums + (w * W + k) * ROWS * 8);
            }
        }
        row0 += STEP;
        if (row0 >= n) break;
        sums_there = true;
    }
    if (const int row = row0 - STEP + static_cast<int>(threadIdx.x); threadIdx.x < ROWS && row < n) finish_few<W>(model, total, row, scores, labels);
}

template <int MODE, int WP, bool SHARED>
KernelFn pick_groups(int groups, int last)
{
    if (groups == 1) return forest_deep_kernel<1, 1, MODE, WP, SHARED>;
    if constexpr (MODE != DEEP_FEW_LEAVES)
        if (last == 1) return forest_deep_kernel<2, 1, MODE, WP, SHARED>;
    return forest_deep_kernel<2, 2, MODE, WP, SHARED>;
}

template <bool SHARED>
KernelFn pick_mode(int groups, int last, int mode, int width)
{
    switch (mode) {
        case DEEP_FEW_LEAVES: return pick_groups<DEEP_FEW_LEAVES, 1, SHARED>(groups, last);
        case DEEP_LEAVES_THROUGH: return pick_groups<DEEP_LEAVES_THROUGH, 1, SHARED>(groups, last);
        case DEEP_LEAVES: return pick_groups<DEEP_LEAVES, 1, SHARED>(groups, last);
        case DEEP_COLUMN: return pick_groups<DEEP_COLUMN, 1, SHARED>(groups, last);
        case DEEP_COLUMNS: return pick_groups<DEEP_COLUMNS, 1, SHARED>(groups, last);
    }
    switch (width) {
        case 2: return pick_groups<DEEP_VECTOR, 2, SHARED>(groups, last);
        case 4: return forest_deep_kernel<1, 1, DEEP_VECTOR, 4, SHARED>;
        case 8: return forest_deep_kernel<1, 1, DEEP_VECTOR, 8, SHARED>;
        case 12: return forest_deep_kernel<1, 1, DEEP_VECTOR, 12, SHARED>;  // shared: 9-wide leaves, whose sums let two workgroups on a CU
        default: return forest_deep_kernel<1, 1, DEEP_VECTOR, 16, false>;   // 13 columns of 16 waves' sums take more than half a CU's LDS
    }
}

KernelFn pick(int groups, int last, int mode, int width, bool shared)
{
    return shared ? pick_mode<true>(groups, last, mode, width) : pick_mode<false>(groups, last, mode, width);
}

template <bool ONCE>
KernelFn pick_tiles(int width)
{
    if (width > 1) return forest_deep_tiles_kernel<DEEP_TILE_GROUPS, DEEP_VECTOR, 2, ONCE>;
    return forest_deep_tiles_kernel<DEEP_TILE_GROUPS, DEEP_COLUMN, 1, ONCE>;
}

KernelFn pick_tiles(int width, bool once) { return once ? pick_tiles<true>(width) : pick_tiles<false>(width); }

}  // namespace

hipError_t init_deep_kernels(size_t lds_limit)
{
    const auto init = [&](KernelFn kernel) {
        const void *fn = reinterpret_cast<const void *>(kernel);
        hipFuncAttributes attr;
        if (hipError_t e = hipFuncGetAttributes(&attr, fn); e != hipSuccess) return e;
        if (attr.sharedSizeBytes != 0) return hipErrorInvalidValue;  // the kernels address LDS from 0
        return hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, static_cast<int>(lds_limit));
    };
    for (int width : {1, 2})
        for (bool once : {false, true})
            if (hipError_t e = init(pick_tiles(width, once)); e != hipSuccess) return e;
    for (int mode : {DEEP_COLUMN, DEEP_COLUMNS, DEEP_VECTOR, DEEP_LEAVES, DEEP_LEAVES_THROUGH, DEEP_FEW_LEAVES})
        for (int width : {2, 4, 8, 12, 16})
            for (int groups : {1, 2})
                for (int last = 1; last <= groups; ++last)
                    for (bool shared : {true, false})
                        if (hipError_t e = init(pick(groups, last, mode, width, shared)); e != hipSuccess) return e;
    return hipSuccess;
}

hipError_t launch_deep_tiles(const DevModel &m, const float *X, int64_t n_rows, float *scores, int32_t *labels, hipStream_t stream)
{
    static_assert(MAX_LAUNCH_ROWS + 2 * CUS * PLAN_ROWS * DEEP_TILE_GROUPS <= 0x7fffffff, "rows count in 32 bits");
    const KernelFn fn = pick_tiles(m.leaf_width, !(m.x_tile & KEEP_X));
    const size_t lds = deep_lds_bytes(m.n_features, m.n_outputs, m.leaf_width, DEEP_TILE_GROUPS, true);
    hipLaunchKernelGGL(fn, dim3(static_cast<unsigned>(tile_workgroups(n_rows))), dim3(DEEP_WAVES * TILE), lds, stream, m, X, n_rows, scores,
                       labels, nullptr);
    return hipGetLastError();
}

hipError_t launch_deep(const DevModel &m, int groups, const TailPlan &t, const float *X, int64_t n_rows, float *scores, int32_t *labels,
                       int32_t *leaf_out, hipStream_t stream)
{
    const bool shared = deep_shares_cu(m, groups, leaf_out == nullptr);
    int mode = m.leaf_width > 1 ? DEEP_VECTOR : m.n_outputs == 1 ? DEEP_COLUMN : DEEP_COLUMNS;
    if (leaf_out) mode = leaves_by_fours(m, groups, n_rows) ? DEEP_FEW_LEAVES : ids_go_through(m.n_trees, n_rows, reinterpret_cast<uintptr_t>(leaf_out)) ? DEEP_LEAVES_THROUGH : DEEP_LEAVES;
    if (t.full + t.after > 0x7fffffffLL) return hipErrorInvalidValue;
    const dim3 grid(static_cast<unsigned>(t.full + t.after), static_cast<unsigned>(m.n_splits));
    const size_t lds = deep_lds_bytes(m.n_features, m.n_outputs, m.leaf_width, groups, leaf_out == nullptr);
    hipLaunchKernelGGL(pick(groups, t.groups, mode, deep_width(m.leaf_width), shared), grid, dim3(DEEP_WAVES * TILE), lds, stream, m, X,
                       n_rows, scores, labels, leaf_out);
    return hipGetLastError();
}

}  // namespace forest_impl
