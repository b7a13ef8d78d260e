// The model as the kernels see it, and what one call launches for it: which kernel, how many rows a workgroup
// owns and how many shares the trees are cut into.  Host only and free of HIP: the rules are checked without
// a GPU (forest_testing.h).
#pragma once

#include <cstdint>

#include "forest_model.hpp"

namespace forest_impl {

// Device tables of the register-bank program (forest_model.hpp, forest_pack.cpp).
struct BankDev {
    const uint32_t *prog;
    const uint32_t *child;
    const uint32_t *leaf;
    const BankTree *tree;
    const BankSpan *span;
    const BankBatch *batch;
    const BankPass *pass;           // [passes]
    const BankPassWave *pass_wave;  // [passes][BANK_WAVES]
    const BankTodo *todo;
    int32_t stream_base[BANK_WAVES];
    int32_t batches, max_units, enabled;
    int32_t passes;
};

// Device tables of the walk program (forest_model.hpp).
struct WalkDev {
    const WalkNode *node;
    const float *leaf;
    const int32_t *leaf_node;
    const int32_t *position;
    int32_t depth;   // 0: none
    int32_t groups;  // row groups the X tile is laid out for
    int32_t stages;
};

// Device tables of the deep walk program (forest_model.hpp).
struct DeepDev {
    const WalkNode *top;
    const WalkNode *unit;
    const int32_t *unit_node;
    const float *value;
    const int32_t *position;
    int32_t groups;  // 0: none
    int64_t units, values;  // how many there are
};

// In DevModel::x_tile: loads of X leave its lines in the L2 (keeps_lines).  An argument of its own, or a bit of the row count, cost the
// walk kernels a tenth more scalar spills; a cache line of arguments that they do not read otherwise 0.2 us a call.
constexpr int32_t KEEP_X = 1 << 30;

struct DevModel {
    const SplitEntry *prog;
    const uint32_t *prog32;
    const ChildRef *child;
    const float *leaf_value;
    const int32_t *leaf_node;
    const TreeMeta *tree;
    const double *col_trees;
    const float *base;
    int32_t n_trees, n_features, n_outputs, leaf_width;
    int32_t x_tile;  // walk kernels, set per launch: n_features and KEEP_X
    int32_t aggregate, transform, output, kind;
    int32_t max_words;
    int32_t path;            // PATH_LDS / PATH_REG / PATH_RANK
    int32_t reg_nv, reg_r;   // REG family: 32 * reg_nv feature registers, reg_r rows per lane
    // RANK family
    int32_t rank_regs;
    int32_t lds_waves;  // LDS rank family: wavefronts per workgroup
    int32_t wave_tree[RANKLDS_WAVES_WIDE + 1];  // and the trees of each wave when the launch is not split
    const FeatBucket *feat_bucket;
    const int32_t *bucket_start;
    const float *thr_sorted;
    const int32_t *feat_thr_base;
    const int32_t *feat_vfirst;
    const FastLookup *fast_feat;  // [n_features] fast lookups (forest_rank_common.hpp)
    const uint16_t *fast_tab;
    // Tree splitting for small batches: with n_splits > 1 the grid's y index selects a share of
    // the trees and the kernels store raw fp64 partial sums to partial[(split * split_rows + row)
    // * n_outputs + k] instead of finishing the row; reduce_splits() finishes.  Set per launch.
    int32_t n_splits;
    int64_t split_rows;
    double *partial;
    int64_t partial_capacity;  // doubles available at `partial`
    int64_t n_entries;         // entries of the split program, all trees (padding included)
    int64_t full_workgroups;  // walk kernels: workgroups before the smaller ones that the launch ends with (choose_tail); set per launch
    // Rank families, split launches: the rank tiles ([tile][rank register][lane] packed f16 pairs)
    // are computed once per row tile by forest_rank_tiles_kernel instead of by every workgroup.
    uint32_t *rank_tiles;
    // LDS rank family: large batches of models it fits run the register-bank kernel
    BankDev bank;
    WalkDev walk;
    DeepDev deep;
    // Picoseconds a row of a large batch takes in the walk kernels and in the dense ones (estimates, forest_plan.hpp);
    // 0: no choice between them
    float walk_ps, dense_ps;
};

// Walk kernels or dense kernels: a node on the path costs two LDS reads of the lane's own, a node of the tree half a
// vector instruction, and beside them every tree costs the walk kernels its copy to LDS (and those deeper than the top
// DEEP_TOP levels whatever its depth) and a lane's row its place in LDS, which shallow trees over few features do not
// pay back.  Picoseconds a row of a large batch takes, as sums of what grows with the features F, the output columns K,
// the trees T, their levels, the entries of the split program and the values of a vector leaf: least squares on
// the measured times of 1,500 models (full, irregular and mixed trees of depth 1 to 12, 4 to 1500 of them, 4 to 200
// features, 1 to 20 columns) at 300,000 to 2,000,000 rows; nine in ten estimates were within 25 % of the time.  The walk
// kernels have become a tenth faster since: their estimate is 0.92 to 1.29 of the time for eight in ten models, 1.10 at the
// median, and the choice costs 0.7 % over 1,200 drawn models at six batches each of 6,000 to 1,000,000 rows; 4.7 % of the
// cells lose more than 3 % and 1.7 times is the worst (12 to 16 columns over few features, which the dense kernels get).
// The walk kernels lose up to a factor of 3 where the rule does not choose them (1M rows, 10 features, us, walk /
// dense: ten 10-wide vector trees of depth 3 311 / 128; 100 trees of depth 3, five columns 166 / 86; 1000 stumps with
// an infinite threshold 1285 / 381), and win by more everywhere else.
struct WalkCost {
    double base, feature, output, tree, level, spread, idle;
    // spread: per feature, where a tile has a CU or its CU's rows to itself; idle: per tree slot of a stage or wave without one
};
struct DenseCost {
    double base, feature, reg, output, tree, level, entry, value;
};

inline double walk_row_ps(const PackedModel &m)
{
    const double F = m.n_features, K = m.n_outputs, T = m.n_trees;
    WalkCost c;
    double spread = 0.0, level = 0.0, idle = 0.0;
    if (m.walk_depth > 0) {
        c = K == 1 ? WalkCost{38.5, 0.657, 0, 0, 0.150, 0.673, 0.151} : WalkCost{57.4, 0.479, 4.49, 0.0832, 0.144, 0.813, 0.262};
        const int trees = walk_stage_trees(m.walk_depth);
        spread = m.walk_groups == 1 ? F : 0.0;
        level = T * m.walk_depth;
        idle = static_cast<double>((m.walk_stages + WALK_WAVES - 1) / WALK_WAVES * WALK_WAVES) * trees - T;
    } else {
        const int W = m.leaf_width;
        c = W == 1   ? K == 1 ? WalkCost{71.0, 0.281, 0, 1.34, 0, 1.18, 0} : WalkCost{62.6, 0.365, 4.76, 1.37, 0, 1.15, 0}
            : W == 2 ? WalkCost{0, 0.360, 30.0, 1.31, 0, 1.02, 0}
            : W <= 4 ? WalkCost{92.5, 0.394, 5.18, 2.08, 0, 1.20, 0}
            : W <= 8 ? WalkCost{106, 0.406, 2.83, 2.51, 0, 1.23, 0}
            : W == 9 ? WalkCost{0, 0.471, 15.6, 2.87, 0, 1.25, 0}
            : W <= 12 ? WalkCost{207, 0.296, 7.40, 3.68, 0, 0.572, 0}
                      : WalkCost{0, 0.338, 21.1, 5.18, 0, 0.535, 0};
        spread = F > 192 ? F : 0.0;
    }
    return c.base + c.feature * F + c.output * K + c.tree * T + c.level * level + c.spread * spread + c.idle * idle;
}

// 0: not measured as the faster of the two anywhere.
inline double dense_row_ps(const PackedModel &m, int64_t n_entries)
{
    const int W = m.leaf_width, K = m.n_outputs;
    DenseCost c;
    double scale = 1.0;
    if (m.n_features > 256) return 0.0;
    if (m.path == PATH_RANK) {
        const int regs = m.rank_regs <= 32 ? 0 : m.rank_regs <= 64 ? 1 : 2;
        static const DenseCost scalar[3] = {{11.9, 2.25, 0, 3.70, 0.239, 0, 0.0219, 0}, {0, 2.78, 0.0867, 4.37, 0.262, 0, 0.0207, 0}, {28.8, 3.67, 0.965, 2.61, 0.334, 0, 0.0211, 0}};
        static const DenseCost vec[3] = {{9.44, 2.20, 0.123, 3.79, 0, 0, 0.0231, 0.402}, {0, 2.73, 0.351, 1.23, 0.09, 0, 0.0230, 0.511}, {130, 3.57, 0.134, 0, 0.0638, 0, 0.0318, 0.631}};
        static const DenseCost wide[3] = {{0, 2.55, 0, 6.52, 0, 0, 0.0362, 0.315}, {0, 2.54, 0, 9.48, 0, 0, 0.0390, 0.285}, {0, 0, 7.62, 14.4, 1.29, 0, 0.00802, 0.327}};
        c = W == 1 ? scalar[regs] : W <= 8 ? vec[regs] : wide[regs];
    } else if (m.path == PATH_RANK_LDS && m.bank_enabled) {
        if (W > 1) return 0.0;
        c = {0, 0.748, 1.64, 51.0, 3.41, 0.0338, 0.0263, 0};
    } else if (m.path == PATH_RANK_LDS && W == 1) {
        c = {59.7, 1.20, 1.21, 11.0, 0.322, 0.262, 0.0467, 0};
    } else if (m.path == PATH_RANK_LDS) {
        // by the wavefronts a CU holds
        const size_t fit = CU_LDS_BYTES / ranklds_lds_bytes(m.rank_regs, K, W, m.lds_waves);
        if (m.lds_waves == 12) c = fit > 1 ? DenseCost{81.9, 1.28, 0.654, 4.32, 0, 0.169, 0.0468, 0.438} : DenseCost{0, 1.79, 1.79, 20.7, 2.86, 0.145, 0.0652, 0.110};
        else if (m.lds_waves == 8 && fit > 1) c = {5.27, 1.78, 1.01, 11.0, 0.616, 0.336, 0.0493, 0.383};
        else if (m.lds_waves == 2 && fit >= 4) c = {0, 0, 7.29, 0, 0, 0.483, 0.0609, 0.324};
        else return 0.0;
        if (m.lds_waves == 2 && fit < 7) scale = 7.0 / static_cast<double>(fit);  // measured with seven workgroups on a CU
    } else {
        return 0.0;
    }
    const double F = m.n_features, T = m.n_trees;
    return scale * (c.base + c.feature * F + c.reg * m.rank_regs + c.output * K + c.tree * T + c.level * m.sum_depth + c.entry * n_entries +
                    c.value * (W > 1 ? T * W : 0.0));
}

// What a PackedModel says about its kernels; the device tables are left null.
inline DevModel describe(const PackedModel &m)
{
    DevModel d{};
    d.n_trees = m.n_trees;
    d.n_features = m.n_features;
    d.n_outputs = m.n_outputs;
    d.leaf_width = m.leaf_width;
    d.aggregate = m.aggregate;
    d.transform = m.transform;
    d.output = m.output;
    d.kind = m.kind;
    d.max_words = m.max_words;
    d.path = m.path;
    d.reg_nv = m.reg_nv;
    d.reg_r = m.reg_r;
    d.rank_regs = m.rank_regs;
    d.lds_waves = m.lds_waves;
    for (int w = 0; w <= RANKLDS_WAVES_WIDE; ++w) d.wave_tree[w] = m.wave_tree[w];
    for (int w = 0; w < BANK_WAVES; ++w) d.bank.stream_base[w] = m.bank_stream_base[w];
    d.bank.batches = m.bank_batches;
    d.bank.max_units = m.bank_max_units;
    d.bank.enabled = m.bank_enabled;
    d.bank.passes = static_cast<int32_t>(m.bank_pass.size());
    d.walk.depth = m.walk_depth;
    d.walk.groups = m.walk_groups;
    d.walk.stages = m.walk_stages;
    d.deep.groups = m.deep_groups;
    d.deep.units = static_cast<int64_t>(m.deep_unit.size());
    d.deep.values = static_cast<int64_t>(m.deep_value.size());
    d.n_splits = 1;
    d.n_entries = static_cast<int64_t>(m.prog32.size() > m.prog.size() ? m.prog32.size() : m.prog.size());
    if (m.walk_depth > 0 || m.deep_groups > 0) {
        d.walk_ps = static_cast<float>(walk_row_ps(m));
        if (m.form == FOREST_FORM_AUTO) d.dense_ps = static_cast<float>(dense_row_ps(m, d.n_entries));
    }
    return d;
}

constexpr int PLAN_ROWS = 64;  // lanes per wavefront: rows go to workgroups in multiples of it

// Batches below this many workgroups split the trees over several workgroups per row tile.
constexpr int64_t SPLIT_BELOW_BLOCKS = 512;
// A split launch aims at about this many workgroups in all and gives every wave whole trees of
// at least this many program entries together.
constexpr int64_t SPLIT_TARGET_BLOCKS = 1024;
constexpr int64_t SPLIT_MIN_ENTRIES_PER_WAVE = 512;
// Walk kernels: workgroups of 16 waves that a split launch aims at, two per CU (a model whose tile leaves room for one
// per CU has half as many places; it is cut into as many shares all the same), the chip's CUs, and the copies of trees
// to LDS that a split launch leaves a wave at least.
constexpr int64_t WALK_RESIDENT = 512;
constexpr int64_t CUS = 256;
constexpr int64_t WALK_SPLIT_MIN_COPIES = 2;

// Device memory a split launch (small batch) needs besides the inputs and outputs: the tree
// shares' fp64 partial sums and, for the rank families, the rank tiles of the batch.
struct Workspace {
    double *partial = nullptr;
    int64_t partial_doubles = 0;
    uint32_t *rank_tiles = nullptr;
    int64_t rank_tile_words = 0;
};

// Bytes of the rank tiles of `tiles` row tiles, and doubles of partial sums that never limit a split launch.
inline size_t rank_tile_bytes(int rank_regs, int64_t tiles)
{
    const size_t b = sizeof(uint32_t) * 64 * static_cast<size_t>(rank_regs > 0 ? rank_regs : 0) * static_cast<size_t>(tiles);
    return (b + 255) & ~size_t{255};
}

inline int64_t split_workspace_doubles(int n_outputs)
{
    // splits x rows stays below (SPLIT_TARGET_BLOCKS + SPLIT_BELOW_BLOCKS) workgroups x 128 rows
    const int64_t want = (SPLIT_TARGET_BLOCKS + SPLIT_BELOW_BLOCKS) * 128 * n_outputs;
    const int64_t cap = int64_t{4} << 20;  // 32 MB
    return want < cap ? want : cap;
}

// Rows one workgroup of the model's dense kernel owns, and its number of wavefronts.
inline int family_rows_per_block(const DevModel &m)
{
    if (m.path == PATH_RANK || m.path == PATH_RANK_LDS) return 128;
    if (m.path == PATH_REG) return PLAN_ROWS * m.reg_r;
    return PLAN_ROWS;
}

inline int family_waves_per_block(const DevModel &m) { return m.path == PATH_RANK_LDS ? m.lds_waves : 4; }

// How many shares the trees are cut into for a batch of n_rows rows (1 = no split); `fits`
// tells whether the workspace allowed the split the batch asks for.
inline int choose_splits(const DevModel &m, const Workspace *ws, int64_t n_rows, bool needs_sums, bool &fits)
{
    fits = true;
    const int64_t rb = family_rows_per_block(m);
    const int64_t n_blocks = (n_rows + rb - 1) / rb;
    if (n_blocks >= SPLIT_BELOW_BLOCKS) return 1;
    const int64_t per_tree = m.n_trees > 0 ? (m.n_entries + m.n_trees - 1) / m.n_trees : 1;
    const int64_t trees_per_wave = (SPLIT_MIN_ENTRIES_PER_WAVE + per_tree - 1) / (per_tree > 0 ? per_tree : 1);
    int64_t s = m.n_trees / (family_waves_per_block(m) * (trees_per_wave > 0 ? trees_per_wave : 1));
    const int64_t by_grid = (SPLIT_TARGET_BLOCKS + n_blocks - 1) / n_blocks;
    if (by_grid < s) s = by_grid;
    if (s < 2) return 1;  // the model is too small to be worth cutting
    const bool ranks = m.path == PATH_RANK || m.path == PATH_RANK_LDS;
    const int64_t tile_words = ranks ? n_blocks * m.rank_regs * 64 : 0;
    if (tile_words > (ws ? ws->rank_tile_words : 0)) {
        fits = false;
        return 1;
    }
    if (needs_sums) {
        const int64_t by_ws = (ws ? ws->partial_doubles : 0) / (n_rows * m.n_outputs);
        if (by_ws < s) s = by_ws;
        if (s < 2) {
            fits = false;
            return 1;
        }
    }
    return static_cast<int>(s);
}

// The same for the models of the walk kernels, whose workgroups own 64 rows or more: as many shares
// as fill the chip's workgroups once, each of its waves left two copies of trees to LDS or more.
// (Against the dense kernels' shares with their rank tiles: 10,007 rows of 250 trees of depth 8, 64 features:
// 63.6 -> 21.5 us a call; 1,021 rows of 2000 x depth 6, 128 features: 39.3 -> 22.4.  Half as many shares: 18.5
// and 20.9 with a costly reduction, the same as now since it is cheap; at least 1 or 4 copies: no difference.)
inline int choose_walk_splits(const DevModel &m, const Workspace *ws, int64_t n_rows, bool needs_sums)
{
    const int64_t n_blocks = (n_rows + PLAN_ROWS - 1) / PLAN_ROWS;
    const int64_t copies = m.walk.depth > 0 ? m.walk.stages : m.n_trees;
    // A copy of trees of depth 3 is 16 trees, work enough for a wave if three shares or more come of it: 1000 such
    // trees, 10 features, 1,000 rows 21 -> 16 us, five columns 26 -> 19 (the dense kernels' shares: 18 and 19).  Two
    // shares do not earn their reduction: 300 trees of depth 4, 10,007 rows 12 -> 15 us.
    const int64_t min_copies = m.walk.depth == WALK_MIN_DEPTH && copies >= 3 * WALK_WAVES ? 1 : WALK_SPLIT_MIN_COPIES;
    // leaf ids are dealt four trees at a time
    const int64_t waves = needs_sums ? copies / min_copies : (m.n_trees + 3) / 4;
    int64_t s = WALK_RESIDENT / n_blocks;
    if (waves / WALK_WAVES < s) s = waves / WALK_WAVES;
    if (needs_sums && s > 1) {
        const int64_t by_ws = (ws ? ws->partial_doubles : 0) / (n_rows * m.n_outputs);
        if (by_ws < s) s = by_ws;
    }
    return s < 2 ? 1 : static_cast<int>(s);
}

// Row groups per workgroup, walk and deep walk kernels: as many as leave every CU a workgroup, or, with trees enough
// for their copies to LDS to count, half of the CUs one of two groups.  More rows per workgroup share those copies and
// keep more walks in flight, and a workgroup that has a CU to itself is nearly twice as fast as one of two, so rounds
// of two per CU are not what counts: over 240 models and 20,000 to 270,000 rows this was within 0.8 % of the best choice
// for each (sums 2 and leaf ids 5 % at 20,000 rows), where counting rounds was 25 % off at 66,000 and 40 % at
// 150,000 rows (ten trees of depth 2, 10 features, 66,000 rows: 19.2 us with one group, 14.9 with two, 11.5 with
// four).  That was with workgroups of one size; with the smaller ones at the end (choose_tail), four groups / two, us: 90,000
// rows of 500 x depth 8 70.7 / 76.4, of 700 x depth 6 59.4 / 60.4, 120,000 of 500 x depth 8 87.8 / 100; the other way 1000 x depth 6,
// 100,000 to 114,000 rows 104.5 / 93.8, 198,000 239 / 238, leaf ids of ten trees of depth 4, 90,000 rows 6.9 / 5.7.  Split launches have no
// workgroups to spare.
inline int choose_groups(const DevModel &m, int groups, int64_t n_rows, int n_splits)
{
    const auto workgroups = [&](int g) { return (n_rows + PLAN_ROWS * g - 1) / (PLAN_ROWS * g); };
    if (n_splits > 1) return 1;
    if (groups >= 4 && workgroups(4) >= CUS) return 4;
    return groups >= 2 && workgroups(2) >= (m.n_trees >= 100 ? CUS / 2 : CUS) ? 2 : 1;
}

// The workgroups that a launch ends with.  Workgroups of one size come to every CU as often but for the rest of a division
// by the CUs, and the CUs that get one of that rest finish a whole workgroup later than the others: boosted trees of depth
// 9, 103,069 rows, are 806 workgroups of 128 rows, three for every CU and a fourth for 38 of them, 81 us where 768 take 64.
// So the rows of the rest go in workgroups of fewer row groups, those that leave the CU with most of them fewest row groups,
// if these are half of a whole workgroup's at most (a workgroup of the rest copies the trees to LDS for fewer rows: 100,003 rows,
// whose rest is 135 workgroups of four groups, as they are / in 540 of one group: leaf ids of 200 x depth 6 36.1 / 42.1, sums of
// 500 x depth 8 87.5 / 95.2, of 40 x depth 6 11.5 / 12.9, of 1000 x depth 6 104.5 / 100.9; rests of 160 and 190 and behind two or
// four rounds alike).  us a call, whole / smaller
// at the end: 1M rows of 500 x depth 8, 28 features (15.3 rounds) 617 / 598; 1M of 1000 x depth 6 753 / 731; 500,000 of 2000
// x depth 6, 10 columns 822 / 805; the 103,069 rows 80.7 / 73.2; 80,896 rows (1.2 rounds) of 500 x depth 8 86.6 / 60.7, of
// ten such trees 7.31 / 6.37, leaf ids of 200 x depth 6 41.5 / 32.4; 40,000 rows of 30 irregular trees 9.2 / 8.5.
struct TailPlan {
    int64_t full;    // workgroups of the plan's row groups
    int64_t after;   // workgroups after them
    int32_t groups;  // row groups of those
};

inline TailPlan whole(int groups, int64_t n_rows)
{
    return TailPlan{(n_rows + PLAN_ROWS * groups - 1) / (PLAN_ROWS * groups), 0, groups};
}

inline TailPlan choose_tail(int groups, int64_t n_rows, int n_splits)
{
    TailPlan t = whole(groups, n_rows);
    const int64_t n = t.full, rest = n % CUS;
    if (n_splits > 1 || n < CUS || rest == 0) return t;
    int64_t best = groups;
    for (int g = groups / 2; g >= 1; g /= 2)
        if (const int64_t most = (rest * (groups / g) + CUS - 1) / CUS * g; 2 * most <= groups && most < best) {
            best = most;
            const int64_t rows = n_rows - (n - rest) * PLAN_ROWS * groups;
            t = TailPlan{n - rest, (rows + PLAN_ROWS * g - 1) / (PLAN_ROWS * g), g};
        }
    return t;
}

// Whether two workgroups fit a CU.
inline bool deep_shares_cu(const DevModel &m, int groups, bool sums)
{
    return deep_lds_bytes(m.n_features, m.n_outputs, m.leaf_width, groups, sums) <= CU_LDS_BYTES / 2;
}

// Leaf ids of few trees: a wave takes four of them and stores their ids itself (true), or the trees are dealt evenly and
// the waves exchange the ids.  An exchange puts all 16 waves through two more barriers and a share of the stores, which
// few trees do not win back in a batch of many workgroups; small batches wait for the longest wave, and wide rows for
// their tile, and there one tree a wave is the better.  us, exchange / fours, at 700,000 rows: 5 trees of depth 6, 4
// features, two columns 45 / 30; 16 of depth 6, 20 features, two columns 60 / 43; 9 of depth 3, 8 features, one column 33 / 24;
// 6 of depth 8, 20 features 34 / 29; irregular trees with 15-wide leaves of depth 8, 4 features: 10 86 / 63, 16 78 / 66.  The
// other way: 8 of depth 6, 2 features, one column 21 / 24; 24 of depth 7, 4 features 45 / 48; 7 irregular of depth 11, 110
// features, 350,000 rows 68 / 80; 8 of depth 8, 10 features, 13,000 rows 4.3 / 4.7; the same 9 of depth 8, 64 features 70 / 70.
// (12 of depth 5, 15 features, one column stay with the exchange: 35 / 28.)
inline bool leaves_by_fours(const DevModel &m, int groups, int64_t n_rows)
{
    const int64_t workgroups = (n_rows + PLAN_ROWS * groups - 1) / (PLAN_ROWS * groups);
    const int T = m.n_trees, F = m.n_features;
    if (T == 1) return true;
    if (m.walk.depth > 0) {
        if (T == 2) return true;
        if (T <= (m.walk.depth > 6 ? 6 : F < 4 ? 7 : 9)) return F <= 40 && workgroups >= CUS;
        return groups == 2 && F >= 4 && F <= 32 && T <= 16 && workgroups >= (T <= 12 ? 600 : 600 + 850 * (T - 12));
    }
    if (groups == 2) return T <= 6 && F <= 32 && workgroups >= 1500;
    if (T == 2) return F <= 64 && workgroups >= 512;
    return F <= 40 && (T <= 6 || (F >= 4 && T <= 20)) && workgroups >= 2000;
}

// Whether a launch may end in smaller workgroups.  Not leaf ids by fours, whose few trees are walked in less time than a
// workgroup takes to begin and end.  Where a CU holds one workgroup of the deep kernel (leaf ids, several columns, wider leaves; what does
// not go tile after tile), the form with both sizes walks up to 1.3 % slower, which long launches do not win back: whole / smaller at the
// end, us, 224 features, leaf ids of 300 trees of depth 9 in 1.2 rounds of the CUs 80.9 / 74.8, 10.2 484 / 481, 19.1 870 / 871, 30.2 1332 / 1344;
// of 128 trees of depth 12 21.1 rounds 560 / 557, 40.1 1026 / 1034; three columns of 300 trees 1.2 58.9 / 52.4, 21.1 629 / 623, 50.1 1435 / 1432.
constexpr int64_t TAIL_MAX_ROUNDS = 20;

inline bool ends_in_smaller(const DevModel &m, int kernel, int groups, int64_t n_rows, bool sums)
{
    if (!sums && leaves_by_fours(m, groups, n_rows)) return false;
    if (kernel == FOREST_KERNEL_WALK) return true;
    return kernel == FOREST_KERNEL_DEEP && (deep_shares_cu(m, groups, sums) || n_rows < TAIL_MAX_ROUNDS * CUS * PLAN_ROWS * groups);
}

// Sums by workgroups that take tile after tile (forest_deep_tiles_kernel), one on a CU with two row groups: where the tile leaves no room for
// a second workgroup of two groups, whose walk would hide the first one's wait for its rows, and from two tiles a CU on.  us,
// a workgroup per tile / tile after tile, 1M rows of 128 trees of depth 12, vector leaves: 40 features 430 / 499, 90
// features 475 / 513, 128 (two workgroups of one group) 590 / 515, 192 625 / 531, 224 631 / 549; of 300 trees of depth 9 529 / 706, 558 / 718,
// 768 / 720, 799 / 741, 831 / 754; 256 features: 33,000 rows 37.8 / 38.4, 66,000 60.7 / 57.6, 100,000 83.7 / 77.5, 150,000 113.7 / 97.1,
// 4M 2712 / 2150 (the last before whole lines).
//
// A batch of whole rounds and few tiles more has a last round that leaves most CUs idle.  Up to 192 features, where the other kernel has two
// workgroups of 64 rows on a CU, that kernel spreads the rest better, which counts while the rounds are few.  Tile after tile, of a workgroup
// per 64 rows = 1, 97 to 192 features, in 2.0 to 2.4 rounds / 3.0 to 3.4 / 4.1 to 4.3 / 5.1 to 5.5 / 6.0: 300 trees of depth 9 1.09 / 1.05 / 1.03 /
// 1.01 / 1.01, 1000 of them 1.08 / 1.05 / 1.04 / 1.03 / 1.02, 300 of depth 12 1.04 / 1.01 / 1.00 / 0.99 / 0.98, 128 of depth 9 1.02 / 0.98 / 0.95 / 0.93 /
// 0.92, 20 of them 1.04 / 0.98 / 0.95 / 0.91 / 0.89; rounds and a half or more 0.85 to 0.95; 7.0 rounds of 1000 trees 1.00.
//
// Waves with one tree each or none have no second tree whose top would fill the first one's waits, and the two workgroups of 64 rows have twice as
// many of them on a CU; only many tiles pay for that.  Tile after tile, of a workgroup per 64 rows = 1, 100 / 130 / 160 / 192 features: 8 trees of depth
// 13, 99,000 rows 1.16 / 1.25 / 1.16 / 1.18, 300,000 1.06 / 1.13 / 1.06 / 1.07, 1M 1.00 / 1.06 / 0.98 / 0.97; 16 of them 1.11 / 1.21 / 1.14 / 1.16, 0.99 / 1.04 /
// 0.93 / 0.96, 0.91 / 0.95 / 0.80 / 0.80; 24 of them 1.03 / 1.10 / 1.02 / 1.03, 0.93 / 0.99 / 0.91 / 0.91; 200 features, 8 trees 1.00, 0.93, 0.90.
constexpr int DEEP_TILE_GROUPS = 2;
constexpr int SINGLE_TREES_MIN_ROUNDS = 16;
constexpr int REST_MAX_ROUNDS = 7, REST_MAX_ROUNDS_FEW_TREES = 3, REST_FEW_TREES = 200;

inline bool takes_tiles(const DevModel &m, int64_t n_rows, int n_splits, bool sums)
{
    if (!sums || n_splits > 1 || m.leaf_width > 2 || (m.leaf_width == 1 && m.n_outputs > 1)) return false;
    if (n_rows < 2 * CUS * PLAN_ROWS * DEEP_TILE_GROUPS) return false;
    const int64_t tiles = (n_rows + PLAN_ROWS * DEEP_TILE_GROUPS - 1) / (PLAN_ROWS * DEEP_TILE_GROUPS), rest = tiles % CUS;
    if (m.n_trees <= DEEP_WAVES && deep_shares_cu(m, 1, true) && tiles < SINGLE_TREES_MIN_ROUNDS * CUS) return false;
    if (rest > 0 && rest <= CUS / 2 && deep_shares_cu(m, 1, true) && tiles / CUS < (m.n_trees < REST_FEW_TREES ? REST_MAX_ROUNDS_FEW_TREES : REST_MAX_ROUNDS)) return false;
    return !deep_shares_cu(m, DEEP_TILE_GROUPS, true) && deep_lds_bytes(m.n_features, m.n_outputs, m.leaf_width, DEEP_TILE_GROUPS, true) <= CU_LDS_BYTES;
}

// Pieces of 64 rows x 32 features that such a workgroup's tile comes in, one a wave.
constexpr int ahead_pieces(int n_features, int groups) { return ((n_features + 31) >> 5) * groups; }

inline int64_t tile_workgroups(int64_t n_rows)
{
    const int64_t tiles = (n_rows + PLAN_ROWS * DEEP_TILE_GROUPS - 1) / (PLAN_ROWS * DEEP_TILE_GROUPS);
    return tiles < CUS ? tiles : CUS;
}

// One lane per (row, tree): the smallest batches of the walk kernels' models (forest_kernels_split.hip).
// Up to a million tests the gathers take less than what a walk kernel's workgroups begin and end with.
// Microseconds a call, this kernel / walk kernels with their reduction, 500 trees of depth 8: 32 rows 7.5 / 9.3,
// 131 rows 8.0 / 9.6, 262 rows (a million tests) 9.4 / 9.8, 370 rows 10.8 / 9.8, 1,048 rows 23.5 / 10.0; 2000 x depth 6, 10 columns:
// 21 rows 10.4 / 10.5, 87 rows (a million) 11.9 / 10.5, 174 rows 14.8 / 10.7; 1000 x depth 3: 349 rows 6.7 / 12.8, 699 rows (two)
// 11.1 / 12.9.  Few trees, which the walk kernels take in one launch, are bounded by rows: ten of depth 4 6,000 rows
// 4.5 / 5.4, 20,000 5.2 / 5.8, 30,000 6.1 / 5.9; three of depth 6 4,000 rows 4.9 / 4.5, with five columns 5.7 / 5.8.
constexpr int64_t POINT_MAX_TESTS = 1 << 20;  // rows x trees x depth
constexpr int64_t POINT_MAX_ROWS = 8192;
// Tests of one row of trees deeper than four levels, all by one workgroup, whose CU's texture path they queue at; above
// this many the walk kernels' shares and their reduction are the faster.  us a call, this kernel / the shares, 1 row of 12,000
// tests: depth 5 10.7 / 10.6, 6 10.2 / 9.5, 7 9.8 / 9.6, 8 9.6 / 9.9; at 10,500 9.3 / 9.4 of depth 6; at 15,000 12.4 / 10.6,
// 11.9 / 9.6, 12.3 / 9.8, 11.3 / 10.0.  (Two pairs of a thread at a time: 11.7 for 2000 x depth 6.)  Several columns make the
// reduction dearer: of depth 5, whose shares are few and long, ten columns 11.5 / 11.7 at 15,000 and three 11.5 / 11.5 (12.5 /
// 11.7 for 40 rows); deeper trees gain little (ten columns, 13,000 tests, depths 6 to 8: 10.9 / 10.4, 10.1 / 10.0, 10.0 / 10.3, and 13.1 /
// 10.9 for 40 rows of depth 8) unless the columns are many (32: 11.6 / 12.1, 11.0 / 11.8, 10.8 / 12.4; 40 rows of depth 8 13.8 /
// 12.9).  Leaf ids, which need no reduction, cross at fewer tests up to depth 6 (12,000 of depth 6: 8.8 / 5.8), and trees of
// up to four levels at more (15,000 of depth 4, 20,000 of depth 3; ten columns 21,000 and 37,000); both follow the rule as
// it stands.
inline int64_t point_max_row_tests(const DevModel &m, int64_t n_rows, bool sums)
{
    return sums && m.n_outputs > 1 && (m.walk.depth == 5 || (m.n_outputs > 16 && n_rows <= 16)) ? 14000 : 12000;
}
constexpr size_t POINT_MAX_LDS = 64 * 1024;
constexpr int PT_THREADS = 1024, PT_MAX_ROWS = 16;

inline int point_rows(const DevModel &m)
{
    const int rows = PT_THREADS / (m.n_trees > 0 ? m.n_trees : 1);
    return rows < 1 ? 1 : rows > PT_MAX_ROWS ? PT_MAX_ROWS : rows;
}

inline size_t point_lds_bytes(const DevModel &m)
{
    return static_cast<size_t>(point_rows(m)) * (sizeof(double) * (m.n_outputs + 1) + sizeof(float) * (static_cast<size_t>(m.n_trees) + m.n_features)) +
           sizeof(int32_t) * (m.n_outputs + 1);
}

inline int point_threads(const DevModel &m)
{
    const int64_t pairs = static_cast<int64_t>(point_rows(m)) * m.n_trees;
    return pairs >= PT_THREADS ? PT_THREADS : static_cast<int>((pairs + PLAN_ROWS - 1) / PLAN_ROWS * PLAN_ROWS);
}

// Shares need a workspace for their sums: a call that gets none, or one too small for the shares it asks for, keeps this
// kernel (1 row of 2001 trees of depth 6: 10.3 us; one workgroup of the walk kernels takes them all in 44.3).
inline bool takes_point(const DevModel &m, const Workspace *ws, int64_t n_rows, bool sums)
{
    if (m.walk.depth == 0 || n_rows > POINT_MAX_ROWS || n_rows * m.n_trees * m.walk.depth > POINT_MAX_TESTS || point_lds_bytes(m) > POINT_MAX_LDS) return false;
    if (m.walk.depth < 5 || static_cast<int64_t>(m.n_trees) * m.walk.depth <= point_max_row_tests(m, n_rows, sums)) return true;
    Workspace ample;
    ample.partial_doubles = split_workspace_doubles(m.n_outputs);
    return choose_walk_splits(m, ws, n_rows, sums) < choose_walk_splits(m, &ample, n_rows, sums);
}

// Whether leaf ids are written past the L2, where their lines would wait to be put out by others and go to memory in no order of
// use.  A row's ids are then pieces of 16 aligned bytes; with other counts of trees, and from an address that is no multiple of
// 16, pieces share lines and a line goes to memory once for each (us, kept in the L2 / past it: 50 trees, 262,144 rows 36 / 43, 75
// trees 48 / 61, 101 59 / 62, 128 trees from an address 4 bytes off 59.7 / 64.5; 52 trees, 153,846 rows 22.5 / 20.9, 128 trees, 62,500
// rows 17.9 / 15.6, 16 trees, 4M rows 330 / 317).  Not 17 to 48 trees, of which a wave has two or three ids at a time, so many writes
// of four bytes (20 trees, 500,000 rows 49.3 / 53.9).  Up to 64 trees a workgroup writes its rows whole.  Of more it writes 256 bytes
// of a row after the other: where these do not begin 64-byte pieces, the piece between two goes to memory twice, which few ids hide
// in the cache before the memory (68 trees, 117,647 rows 21.4 / 19.4; 200 trees, 10,000 rows 8.9 / 7.9, 40,000 rows 20.4 / 18.8) and more
// do not (68 trees, 800,003 rows 120 / 145; 100 trees, 200,000 rows 43.5 / 44.0, 600,000 141 / 164; 200 trees, 100,003 rows, results
// written over 37.8 / 37.0, in new places 45.2 / 49.4, 300,000 rows 125 / 131; of a multiple of 16 trees 96 trees, 208,333 rows 39.1 /
// 39.1, 400 trees, 50,000 rows 38.7 / 37.7).  The stores count the workgroup's ids in 32 bits.
constexpr int64_t FEW_IDS = int64_t{1} << 23;

inline bool ids_go_through(int n_trees, int64_t n_rows, uintptr_t leaf_out)
{
    if (n_trees % 4 != 0 || n_trees > 1 << 20 || leaf_out % 16 != 0) return false;
    if (n_trees <= 64) return n_trees <= 16 || n_trees > 48;
    return (n_trees % 16 == 0 && leaf_out % 64 == 0) || n_rows * n_trees <= FEW_IDS;
}

// Rows of one launch at most.  HIP takes fewer than 2^32 threads per grid axis, and the walk kernels spend
// 1024 threads on 64 rows, the LDS rank kernel up to 768 on 128: a longer batch goes in ranges of this many
// rows, one launch each.
constexpr int64_t MAX_LAUNCH_ROWS = int64_t{1} << 27;

// Whether the dense kernels are the faster ones for a batch.  The estimates are of sums; leaf ids ask less of the walk
// kernels, of which only the deep one loses, where trees are fewer than a workgroup's waves (100,000 rows of twelve
// trees of depth 3, 9 columns, 4 features: 13.0 us, dense 9.2; from 30 trees on they take 0.3 to 1.1 of the dense
// time).  The margins keep the walk kernels where the estimates, or a batch of few rounds of workgroups, decide
// nothing.  A batch that the dense kernels cut into shares costs them two more launches, which their faster tests have
// to earn (1500 stumps over 4 features, 5,000 rows: 27.1 us, dense 19.9); with vector leaves they do not.
// The walk kernels' estimates are those of workgroups of one size and a trip to LDS per wave's sum and are too high by now: 66,000
// rows of 483 and 911 trees of depth 3 take 34.6 and 57.6 us so and would take 22.4 and 38.3 by walk, 500,000 rows of 395 trees of
// depth 4 in ten columns 192 and 146; of 60 models of depth up to 5, 48 are within 5 % of the better form.
constexpr int64_t DENSE_MIN_ROWS = 4096;

inline bool prefers_dense(const DevModel &m, int64_t n_rows, bool sums)
{
    if (m.dense_ps <= 0.0f || n_rows < DENSE_MIN_ROWS) return false;
    const double dense = m.dense_ps, walk = m.walk_ps;
    const int64_t round = SPLIT_BELOW_BLOCKS * 128;
    if (!sums) return n_rows >= round && m.deep.groups > 0 && m.n_trees < DEEP_WAVES && dense < 0.75 * walk;
    if (n_rows < round)
        return m.path == PATH_RANK && m.leaf_width == 1 && dense < 0.9 * walk && (walk - dense) * static_cast<double>(n_rows) > 3e6;
    if (n_rows < 2 * round) return dense < (m.leaf_width > 1 ? 0.75 : 0.9) * walk;
    return dense < 0.97 * walk;
}

struct LaunchPlan {
    int32_t kernel = FOREST_KERNEL_LDS;
    int32_t groups = 1;  // walk kernels: row groups of 64 rows per workgroup
    int32_t splits = 1;  // shares the trees are cut into
    bool fits = true;    // false: the dense kernels' split launch does not fit the workspace
    bool tiles = false;  // deep kernel: workgroups that take tile after tile
};

// `sums`: scores or labels are asked for, not leaf ids.  A batch the dense kernels' workspace does not hold is
// marked so whichever kernel runs it: what forest_predict_static takes does not depend on the kernel.
inline LaunchPlan plan_launch(const DevModel &m, const Workspace *ws, int64_t n_rows, bool sums)
{
    LaunchPlan p;
    p.splits = choose_splits(m, ws, n_rows, sums, p.fits);
    const bool dense = p.fits && prefers_dense(m, n_rows, sums);
    if (takes_point(m, ws, n_rows, sums)) {
        p.kernel = FOREST_KERNEL_POINT;
        p.splits = 1;
    } else if (m.walk.depth > 0 && !dense) {
        p.kernel = FOREST_KERNEL_WALK;
        p.splits = choose_walk_splits(m, ws, n_rows, sums);
        p.groups = choose_groups(m, m.walk.groups, n_rows, p.splits);
    } else if (m.deep.groups > 0 && !dense) {
        // trees deeper than 8, vector leaves, infinite thresholds: what a row does not meet is not tested
        // (128 trees of depth 12: 2.9 ms against 14.5 with the register-bank kernel)
        p.kernel = FOREST_KERNEL_DEEP;
        p.splits = choose_walk_splits(m, ws, n_rows, sums);
        p.tiles = takes_tiles(m, n_rows, p.splits, sums);
        p.groups = p.tiles ? DEEP_TILE_GROUPS : choose_groups(m, m.deep.groups, n_rows, p.splits);
    } else if (m.path == PATH_RANK) {
        p.kernel = FOREST_KERNEL_RANK;
    } else if (m.path == PATH_RANK_LDS) {
        // large batches of the models it fits: rank registers banked over the waves' vector registers
        p.kernel = p.splits == 1 && m.bank.enabled ? FOREST_KERNEL_RANK_BANK : FOREST_KERNEL_RANK_LDS;
    } else if (m.path == PATH_REG) {
        p.kernel = FOREST_KERNEL_REG;
    }
    return p;
}

// Whether a tile of X is read with loads that leave its lines in the L2, or non-temporally: X is read once and should not push
// the trees out.  Where rows are no whole lines a line lies in two blocks of 32 features or two rows and is asked for again, and a
// second fetch holds up what waits behind it; but the lines that stay cost the trees their place.  So they stay where both about fit an
// XCD's L2 (the trees three times where a CU walks them for one row group at a time), where the trees are few whatever X does to them
// (33 x depth 7, 285 features 184 / 216 us, 480,000 rows), or where several shares of the trees read the tile.  Over 3,012 calls of 29 models with 30 KB to 4 MB of tables, 17 to 530 features and 5,000 to 1M rows, fresh X and X that the
// memory-side cache holds, the lines kept always take 1.7 % more than the better of both and 17 % at worst, never 1.6 and 22, by this rule
// 0.3.  Kept / non-temporal, 1M rows: 128 trees of depth 12, 3-wide leaves (4.2 MB), 200 features 1224 / 1095 us; 600 irregular
// trees of depth 10 (4.1 MB), 90 features 1319 / 1268; 500 x depth 8 (1.5 MB), 300 features 1877 / 1722, 127 features 0.98; 500 x
// depth 7 (0.8 MB), 260 features 1.05, 400 features 1.14; 200 x depth 6 (150 KB), 400 features 0.99; 300
// irregular trees of depth 9 (1.4 MB), three columns, 200 features 1.06; the same, one column, 90 features, 103,069 rows 0.99, X
// in the memory-side cache 67.5 / 70.6; 40 x depth 6, 100 features 0.91; in two shares and more 300 x depth 6, five columns, 200
// features, 10,007 rows 0.93.  Where it errs: 500 features, 1000 x depth 3 1.05; leaf ids of more trees than features, 300,000 rows of
// 200 x depth 6 over 127 features 1.09, 100,003 rows 1.00, 0.93 where X is in the cache.
constexpr int64_t KEEP_L2_BYTES = 4608 << 10, KEEP_FEW_TREES_BYTES = 128 << 10;
constexpr int KEEP_MIN_FEATURES = 17, XCD_CUS = 32;

inline bool keeps_lines(const DevModel &m, const LaunchPlan &p, bool sums, uintptr_t X)
{
    const bool walk = p.kernel == FOREST_KERNEL_WALK;
    if ((!walk && p.kernel != FOREST_KERNEL_DEEP) || m.n_features < KEEP_MIN_FEATURES) return false;
    if (m.n_features % 32 == 0 && X % 128 == 0) return false;
    if (p.splits > 1) return true;
    const int64_t T = m.n_trees, node = sizeof(WalkNode), id = sizeof(int32_t), value = sizeof(float);
    const int64_t tables = walk ? (T * (node + value)) << m.walk.depth
                                : T * static_cast<int64_t>(DEEP_STAGE_BYTES) + m.deep.units * (node + (sums ? 0 : id)) + (sums ? m.deep.values * value : 0);
    if (tables <= KEEP_FEW_TREES_BYTES) return true;
    const size_t lds = walk ? walk_lds_bytes(m.walk.depth, m.n_features, m.n_outputs, m.walk.groups)
                            : deep_lds_bytes(m.n_features, m.n_outputs, m.leaf_width, p.groups, sums);
    const int64_t rows = static_cast<int64_t>(XCD_CUS) * (2 * lds <= CU_LDS_BYTES ? 2 : 1) * PLAN_ROWS * p.groups;  // of an XCD's workgroups
    return tables * (rows == XCD_CUS * PLAN_ROWS ? 3 : 1) + rows * m.n_features * value <= KEEP_L2_BYTES;
}

// The workgroups of one range of rows, walk kernels; of those that take tile after tile, the tiles.
inline TailPlan range_workgroups(const DevModel &m, const LaunchPlan &p, int64_t n_rows, bool sums)
{
    return !p.tiles && ends_in_smaller(m, p.kernel, p.groups, n_rows, sums) ? choose_tail(p.groups, n_rows, p.splits) : whole(p.groups, n_rows);
}

// The shape of the launches of a plan.
inline forest_launch_t launch_shape(const DevModel &m, const LaunchPlan &p, int64_t n_rows, bool sums)
{
    forest_launch_t s{};
    s.kernel = p.kernel;
    s.shares = p.splits;
    switch (p.kernel) {
        case FOREST_KERNEL_POINT:
            s.rows_per_workgroup = point_rows(m);
            s.threads = point_threads(m);
            break;
        case FOREST_KERNEL_WALK:
            s.rows_per_workgroup = PLAN_ROWS * p.groups;
            s.threads = PLAN_ROWS * WALK_WAVES;
            s.lds_bytes = static_cast<int32_t>(walk_lds_bytes(m.walk.depth, m.n_features, m.n_outputs, m.walk.groups));
            s.leaves_by_fours = !sums && leaves_by_fours(m, p.groups, n_rows);
            break;
        case FOREST_KERNEL_DEEP:
            s.rows_per_workgroup = PLAN_ROWS * p.groups;
            s.threads = PLAN_ROWS * DEEP_WAVES;
            s.lds_bytes = static_cast<int32_t>(deep_lds_bytes(m.n_features, m.n_outputs, m.leaf_width, p.groups, sums));
            s.leaves_by_fours = !sums && leaves_by_fours(m, p.groups, n_rows);
            break;
        case FOREST_KERNEL_RANK_BANK:
            s.rows_per_workgroup = BANK_ROWS;
            s.threads = PLAN_ROWS * BANK_WAVES;
            break;
        default:
            s.rows_per_workgroup = family_rows_per_block(m);
            s.threads = PLAN_ROWS * family_waves_per_block(m);
    }
    s.launches = static_cast<int32_t>((n_rows + MAX_LAUNCH_ROWS - 1) / MAX_LAUNCH_ROWS);
    const int64_t rows = n_rows < MAX_LAUNCH_ROWS ? n_rows : MAX_LAUNCH_ROWS;
    s.workgroups = (rows + s.rows_per_workgroup - 1) / s.rows_per_workgroup;
    s.last_rows_per_workgroup = s.rows_per_workgroup;
    if (p.kernel == FOREST_KERNEL_WALK || p.kernel == FOREST_KERNEL_DEEP) {
        const TailPlan t = range_workgroups(m, p, rows, sums);
        s.workgroups = t.full + t.after;
        s.last_rows_per_workgroup = PLAN_ROWS * t.groups;
        s.tile_after_tile = p.tiles;
        s.loading_waves = p.tiles ? ahead_pieces(m.n_features, DEEP_TILE_GROUPS) : s.threads / PLAN_ROWS;
    }
    return s;
}

}  // namespace forest_impl
