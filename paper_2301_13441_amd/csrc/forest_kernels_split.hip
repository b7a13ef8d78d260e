// Kernels that only small batches use: threshold ranks per row tile, the sum of the tree shares'
// partial sums, and the walk with a lane per (row, tree) for the smallest.
//
// A batch of a few thousand rows has too few 128-row tiles to fill 256 compute units, so the
// trees are cut into shares as well (grid y of the family kernels).  Two things are then done
// once per batch instead of once per workgroup: the threshold ranks of the rank families are
// computed here, one thread per (row, feature), and left in global memory for every share's
// workgroup to load; and the shares' fp64 partial sums are added up here and the rows finished.
#include <hip/hip_runtime.h>

#include <cstdint>

#include "forest_device.hpp"
#include "forest_kernel_common.hpp"
#include "forest_rank_common.hpp"

namespace forest_impl {
namespace {

// grid (row tiles, features): 128 threads, one per row of the tile.
__global__ __launch_bounds__(RROWS) void forest_rank_tiles_kernel(DevModel m, const float *__restrict__ X,
                                                                  int64_t n_rows)
{
    const int F = m.n_features;
    const int f = blockIdx.y;
    const int r = threadIdx.x;
    const int64_t row = static_cast<int64_t>(blockIdx.x) * RROWS + r;
    const float x = row < n_rows ? X[row * F + f] : 0.0f;
    uint16_t *tile16 = reinterpret_cast<uint16_t *>(m.rank_tiles + static_cast<size_t>(blockIdx.x) * m.rank_regs * TILE);
    store_rank(tile16, m, f, r, rank_of(m, f, x));
}

// What a column's sum goes through.  Loaded for a thread's first column before the sums are waited for: behind them the
// load is a trip to memory of its own.
struct ColumnTerms {
    float base;
    double trees;
};

// What the kernels below are launched with.  Their calls are the shortest there are, and what the host spends on a launch grows
// with its arguments: 2.4 us with 32 bytes, 2.8 up to 96, 3.3 with 128 and 3.6 with 512; a kernel that asks for its
// workgroup's size is given 256 bytes more, so that is an argument too.
struct Finish {
    const float *base;
    const double *col_trees;
    int16_t n_outputs, threads;
    int8_t mean, transform;
};
static_assert(FOREST_MAX_OUTPUTS <= 0x7fff, "columns in 16 bits");

Finish finish_of(const DevModel &m, int threads)
{
    return Finish{m.base, m.col_trees, static_cast<int16_t>(m.n_outputs), static_cast<int16_t>(threads), m.aggregate == FOREST_AGG_MEAN, static_cast<int8_t>(m.transform)};
}

__device__ __forceinline__ ColumnTerms column_terms(const Finish &m, int k) { return ColumnTerms{m.base[k], m.col_trees[k]}; }

// finish_values for `rows` rows from row0 with all threads of the workgroup: thread by (row, column), and by row
// where the columns meet (label, softmax).  raw[li * row_step + k * column_step] are the summed leaf values
// of row row0 + li, overwritten; by_row: `rows` doubles of LDS.  Every thread of the workgroup calls it,
// behind a barrier after the sums.  A reduction has few rows per workgroup: with a thread per row the
// exponentials of a softmax over 10 columns come one after the other.  (1,021 rows, 10 columns, 31 shares:
// 9.6 us with a thread per row, 16 threads per sum and 8 rows per workgroup, 4.8 so; 10,007 rows, 5 columns,
// 3 shares: 7.8 and 4.4.  In the walk kernels, whose other waves have their own trees to walk, finishing
// rows this way was 2 to 4 % slower than a thread per row.)
__device__ __forceinline__ void finish_rows(const Finish &m, const ColumnTerms &mine, double *raw, int row_step, int column_step,
                                            int rows, double *by_row, int64_t row0, int64_t n_rows, float *scores, int32_t *labels)
{
    const int K = m.n_outputs, threads = m.threads, pairs = rows * K;
    const bool softmax = scores && m.transform == FOREST_TRANSFORM_SOFTMAX;
    for (int p = threadIdx.x; p < pairs; p += threads) {
        const int li = p / K, k = p - li * K;
        double *at = raw + li * row_step + k * column_step;
        double s = *at;
        const ColumnTerms terms = p == static_cast<int>(threadIdx.x) ? mine : column_terms(m, k);
        // a column no tree feeds: the mean over no trees adds nothing to the base score
        if (m.mean && terms.trees > 0.0) s = s / terms.trees;
        s = static_cast<double>(terms.base) + s;
        if (softmax || labels) *at = s;
        if (scores && !softmax && row0 + li < n_rows)
            scores[row0 * K + p] = static_cast<float>(m.transform == FOREST_TRANSFORM_SIGMOID ? 1.0 / (1.0 + exp(-s)) : s);
    }
    if (!softmax && !labels) return;  // uniform
    __syncthreads();
    for (int li = threadIdx.x; li < rows; li += threads) {
        const double *at = raw + li * row_step;
        double best = at[0];
        int lab = 0;
        for (int k = 1; k < K; ++k)
            if (const double s = at[k * column_step]; s > best) {
                best = s;
                lab = k;
            }
        by_row[li] = best;
        if (K == 1) lab = (m.transform == FOREST_TRANSFORM_SIGMOID) ? (best > 0.0) : (best > 0.5);
        if (labels && row0 + li < n_rows) labels[row0 + li] = lab;
    }
    if (!softmax) return;
    __syncthreads();
    for (int p = threadIdx.x; p < pairs; p += threads) {
        const int li = p / K, k = p - li * K;
        double *at = raw + li * row_step + k * column_step;
        *at = exp(*at - by_row[li]);
    }
    __syncthreads();
    for (int li = threadIdx.x; li < rows; li += threads) {
        double z = 0.0;
        for (int k = 0; k < K; ++k) z += raw[li * row_step + k * column_step];
        by_row[li] = z;
    }
    __syncthreads();
    for (int p = threadIdx.x; p < pairs; p += threads) {
        const int li = p / K, k = p - li * K;
        if (row0 + li < n_rows) scores[row0 * K + p] = static_cast<float>(raw[li * row_step + k * column_step] / by_row[li]);
    }
}

constexpr int RS_THREADS = 256;
constexpr int RS_MAX_ROWS = 64;  // rows per workgroup of the reduction

// `lanes` threads share the sum of a (row, column): thread g adds the shares g, g + lanes, ... in ascending
// order, one thread adds the results of the lanes in theirs, and the workgroup finishes its rows exactly
// as an unsplit launch does.  The order of the additions is fixed, so results are reproducible.  The sums
// of a share lie in row order, so neighbouring threads read neighbouring sums.  What bounds it is the trips to memory:
// four shares' sums are loaded together, and a column's base score and tree count with them.  (1,021 rows, 10 columns,
// 31 shares: 15.6 -> 15.1 us a call; 10,007 rows, 5 columns, 3 shares: 17.2 -> 16.8.)
struct ReduceArgs {
    Finish finish;
    const double *partial;  // [n_splits][n_rows][n_outputs]
    float *scores;
    int32_t *labels;
    int64_t n_rows;
    int32_t n_splits;
    int16_t rows, lanes;
};
static_assert(sizeof(ReduceArgs) <= 96, "arguments of a short launch");

__global__ __launch_bounds__(RS_THREADS) void forest_reduce_splits_kernel(ReduceArgs a)
{
    __shared__ double part[RS_THREADS], by_row[RS_MAX_ROWS];
    const Finish &m = a.finish;
    const int rows = a.rows, lanes = a.lanes;
    const int64_t n_rows = a.n_rows;
    const int K = m.n_outputs, pairs = rows * K;  // lanes * pairs <= RS_THREADS
    const int64_t row0 = static_cast<int64_t>(blockIdx.x) * rows;
    const int g = static_cast<int>(threadIdx.x) / pairs, p = static_cast<int>(threadIdx.x) - g * pairs;
    const ColumnTerms terms = column_terms(m, p % K);
    if (g < lanes) {
        double s = 0.0;
        if (row0 * K + p < n_rows * K)
            for (int sp = g; sp < a.n_splits; sp += 4 * lanes) {
                double v[4];  // on their way together
#pragma unroll
                for (int i = 0; i < 4; ++i) v[i] = sp + i * lanes < a.n_splits ? a.partial[((sp + i * lanes) * n_rows + row0) * K + p] : 0.0;
#pragma unroll
                for (int i = 0; i < 4; ++i) s += v[i];
            }
        part[threadIdx.x] = s;
    }
    __syncthreads();
    if (g == 0)
        for (int i = 1; i < lanes; ++i) part[p] += part[i * pairs + p];
    __syncthreads();
    finish_rows(m, terms, part, K, 1, rows, by_row, row0, n_rows, a.scores, a.labels);
}

// The smallest batches of the walk kernels' models: a lane is a (row, tree) pair and walks the tree through
// global memory, so that a few rows still fill wavefronts and a call is one launch.  A workgroup owns
// `rows` rows, whose features it holds in LDS; the leaf values meet there, [row][tree], and a wave adds
// those of a (row, column), whose trees are neighbours in processing order, or, where there are more sums
// than waves, a part of a wave does.  What bounds it is the chain of
// dependent loads, one per level, and for more pairs the gathers: a cycle of the texture path per lane; and the launch (1 row of
// 500 x depth 8 with the whole model's description for an argument: 5.8 us a call, 5.3 so).
struct PointArgs {
    Finish finish;
    const WalkNode *node;
    const float *leaf;  // values, or, read as integers, the ids that the leaf ids are
    const float *X;
    float *out;  // scores, or leaf ids
    int32_t *labels;
    int32_t n_trees, n_features, n_rows;
    int16_t rows;  // of a workgroup
    int8_t depth, shift;  // x_offset >> shift is the feature
};
static_assert(sizeof(PointArgs) <= 96, "arguments of a short launch");

template <bool LEAVES>
__global__ __launch_bounds__(PT_THREADS) void forest_point_kernel(PointArgs a)
{
    extern __shared__ __align__(16) char smem[];
    const Finish &m = a.finish;
    const float *__restrict__ X = a.X;
    const int64_t n_rows = a.n_rows;
    const int rows = a.rows;
    const int F = a.n_features, T = a.n_trees, K = m.n_outputs, D = a.depth;
    double *sum = reinterpret_cast<double *>(smem);                       // [rows][K]
    double *by_row = sum + rows * K;                                      // [rows]
    float *value = reinterpret_cast<float *>(by_row + rows);              // [rows][T]
    int32_t *first = reinterpret_cast<int32_t *>(value + rows * T);       // [K + 1] the columns' first trees
    float *xs = LEAVES ? reinterpret_cast<float *>(smem) : reinterpret_cast<float *>(first + K + 1);  // [rows][F]
    const int64_t row0 = static_cast<int64_t>(blockIdx.x) * rows;
    const int here = n_rows - row0 < rows ? static_cast<int>(n_rows - row0) : rows;
    const int threads = m.threads;
    ColumnTerms terms{};
    if (!LEAVES) terms = column_terms(m, static_cast<int>(threadIdx.x) % K);
    for (int i = threadIdx.x; i < here * F; i += threads) xs[i] = X[row0 * F + i];
    if (!LEAVES && threadIdx.x < TILE) {
        // The columns' trees follow each other; counts are small integers.  A scan by the first wave: one after the other
        // the counts are as many trips to memory; as many steps as the columns need (one column, 1 row of 59 x depth 2: 3.94
        // us with all six, 3.77 with none).
        static_assert(FOREST_MAX_OUTPUTS <= TILE, "a lane per column");
        const int lane = threadIdx.x;
        int n = lane < K ? static_cast<int>(m.col_trees[lane]) : 0;
        for (int d = 1; d < K; d <<= 1) {
            const int below = __shfl_up(n, d, TILE);
            if (lane >= d) n += below;
        }
        if (lane < K) first[lane + 1] = n;
        if (lane == 0) first[0] = 0;
    }
    __syncthreads();
    const int shift = a.shift;
    for (int p = threadIdx.x; p < here * T; p += threads) {
        const int r = p / T, t = p - r * T;
        const WalkNode *__restrict__ node = a.node + (static_cast<int64_t>(t) << D);
        const float *x = xs + r * F;
        uint32_t at = 0;
        for (int l = 0; l < D; ++l) {
            const WalkNode n = node[(1u << l) + at];
            at |= (x[n.x_offset >> shift] <= n.threshold ? 0u : 1u) << l;
        }
        const int64_t leaf = (static_cast<int64_t>(t) << D) + at;
        if (LEAVES) reinterpret_cast<int32_t *>(a.out)[(row0 + r) * T + static_cast<int32_t>(node[0].x_offset)] = reinterpret_cast<const int32_t *>(a.leaf)[leaf];
        else value[p] = a.leaf[leaf];
    }
    if (LEAVES) return;
    __syncthreads();
    // As many lanes per sum as there are threads for, a wave at most.  (Ten trees of five columns, 1,000 rows: 80 sums
    // for three waves, 15.5 us a call with a wave per sum, 4.5 so.)
    int lanes = TILE;
    while (lanes > 1 && rows * K * lanes > threads) lanes >>= 1;
    const int lane = threadIdx.x & (lanes - 1);
    for (int p = threadIdx.x / lanes; p < rows * K; p += threads / lanes) {
        const int r = p / K, k = p - r * K;
        double s = 0.0;
        if (r < here)
            for (int t = first[k] + lane; t < first[k + 1]; t += lanes) s += static_cast<double>(value[r * T + t]);
        for (int d = lanes >> 1; d >= 1; d >>= 1) s += __shfl_xor(s, d, TILE);
        if (lane == 0) sum[p] = s;
    }
    __syncthreads();
    finish_rows(m, terms, sum, K, 1, rows, by_row, row0, n_rows, a.out, a.labels);
}

}  // namespace

hipError_t launch_point(const DevModel &m, const float *X, int64_t n_rows, float *scores, int32_t *labels, int32_t *leaf_out,
                        hipStream_t stream)
{
    const int rows = point_rows(m);
    const int threads = point_threads(m);
    const dim3 grid(static_cast<unsigned>((n_rows + rows - 1) / rows));
    static_assert(POINT_MAX_ROWS <= 0x7fffffff && PT_MAX_ROWS <= 0x7fff && PT_THREADS <= 0x7fff, "in 32 and 16 bits");
    // x_offset = feature * 256 * groups, groups 1, 2 or 4
    const PointArgs a{finish_of(m, threads), m.walk.node, leaf_out ? reinterpret_cast<const float *>(m.walk.leaf_node) : m.walk.leaf, X,
                      leaf_out ? reinterpret_cast<float *>(leaf_out) : scores, labels, m.n_trees, m.n_features, static_cast<int32_t>(n_rows),
                      static_cast<int16_t>(rows), static_cast<int8_t>(m.walk.depth), static_cast<int8_t>(8 + (m.walk.groups >> 1))};
    if (leaf_out) hipLaunchKernelGGL(forest_point_kernel<true>, grid, dim3(threads), point_lds_bytes(m), stream, a);
    else hipLaunchKernelGGL(forest_point_kernel<false>, grid, dim3(threads), point_lds_bytes(m), stream, a);
    return hipGetLastError();
}

hipError_t launch_rank_tiles(const DevModel &m, const float *X, int64_t n_rows, hipStream_t stream)
{
    if (m.rank_regs <= 0) return hipSuccess;  // no feature has a threshold
    const int64_t n_tiles = (n_rows + RROWS - 1) / RROWS;
    hipLaunchKernelGGL(forest_rank_tiles_kernel,
                       dim3(static_cast<unsigned>(n_tiles), static_cast<unsigned>(m.n_features)), dim3(RROWS), 0,
                       stream, m, X, n_rows);
    return hipGetLastError();
}

hipError_t launch_reduce_splits(const DevModel &m, int64_t n_rows, float *scores, int32_t *labels,
                                hipStream_t stream)
{
    // a thread per sum and four shares, and as many rows as that leaves threads for
    int lanes = 1;
    while (lanes * 4 < m.n_splits && lanes < 16 && 2 * lanes * m.n_outputs <= RS_THREADS) lanes *= 2;
    int rows = RS_THREADS / (lanes * m.n_outputs);
    if (rows > RS_MAX_ROWS) rows = RS_MAX_ROWS;
    const int64_t n_blocks = (n_rows + rows - 1) / rows;
    const ReduceArgs a{finish_of(m, RS_THREADS), m.partial, scores, labels, n_rows, m.n_splits, static_cast<int16_t>(rows), static_cast<int16_t>(lanes)};
    hipLaunchKernelGGL(forest_reduce_splits_kernel, dim3(static_cast<unsigned>(n_blocks)), dim3(RS_THREADS), 0, stream, a);
    return hipGetLastError();
}

}  // namespace forest_impl
