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

#if defined(__HIP_DEVICE_COMPILE__)
typedef const __attribute__((address_space(4))) uint32_t *WalkTop;
typedef const __attribute__((address_space(4))) int32_t *WalkTable;
typedef const __attribute__((address_space(1))) char *GlobalBytes;
typedef const __attribute__((address_space(1))) float *GlobalFloats;
typedef const __attribute__((address_space(1))) int32_t *GlobalInts;
#else
typedef const uint32_t *WalkTop;  // host pass: the kernel body is only parsed
typedef const int32_t *WalkTable;
typedef const char *GlobalBytes;
typedef const float *GlobalFloats;
typedef const int32_t *GlobalInts;
#endif

struct __attribute__((aligned(4))) Float4 {
    float v[4];
};
typedef float FloatRun4 __attribute__((ext_vector_type(4), aligned(4)));
struct __attribute__((aligned(4))) Int4 {
    int32_t v[4];
};

// The X tile of a workgroup: rows [row0, row0 + 64 NR) as float32, row group g, feature f and row r of the
// group at xbase + g * group_stride + f * stride + 4 r.  It is filled in pieces of 16 rows x 16 features,
// four neighbouring features of a row per lane: 64 bytes of a row of X, and LDS writes that fall into
// 16 banks.  A wave takes a contiguous run of pieces, so that both halves of a 128-byte line are
// requested by one wave one after the other, with the non-temporal policy: X is read once and should
// not push the trees out of the L2.
struct TileShape {
    const float *X;
    int64_t n_rows;
    int F, blocks;  // blocks of 16 features
    uint32_t xbase, group_stride, stride;
};

// The first of a run of pieces: 16 rows from 16 * rows, 16 features from 16 * block.
struct TilePiece {
    int rows, block;
    __device__ __forceinline__ void next(int blocks)
    {
        if (++block == blocks) {
            block = 0;
            ++rows;
        }
    }
};

// The first P pieces of a run of n, those there are, to registers ...
template <int P>
__device__ __forceinline__ void tile_load(const TileShape &s, int64_t row0, TilePiece at, int n, int lane, Float4 (&v)[P])
{
    const int r = lane & 15, c = (lane >> 4) * 4;
#pragma unroll
    for (int u = 0; u < P; ++u, at.next(s.blocks)) {
        if (u < n) {  // wave-uniform, as everything but the lane's own columns
            const int f0 = at.block * 16;
            const int64_t row = row0 + at.rows * 16 + r;
            const float *p = s.X + (row < s.n_rows ? row : row0) * s.F + f0 + c;
            if (f0 + 16 <= s.F) {
                const FloatRun4 q = __builtin_nontemporal_load(reinterpret_cast<const FloatRun4 *>(p));
#pragma unroll
                for (int i = 0; i < 4; ++i) v[u].v[i] = q[i];
            } else {
#pragma unroll
                for (int i = 0; i < 4; ++i) v[u].v[i] = f0 + c + i < s.F ? p[i] : 0.0f;
            }
        }
    }
}

// ... and from there to the tile.  NAN_IS_INF: a NaN is stored as +Inf.
template <int P, bool NAN_IS_INF>
__device__ __forceinline__ TilePiece tile_store(const TileShape &s, TilePiece at, int n, int lane, const Float4 (&v)[P])
{
    const int r = lane & 15, c = (lane >> 4) * 4;
#pragma unroll
    for (int u = 0; u < P; ++u, at.next(s.blocks)) {
        if (u < n) {
            const int f0 = at.block * 16;
            const uint32_t to = s.xbase + static_cast<uint32_t>(at.rows >> 2) * s.group_stride + static_cast<uint32_t>(f0 + c) * s.stride +
                                static_cast<uint32_t>((at.rows & 3) * 16 + r) * 4;
#pragma unroll
            for (int i = 0; i < 4; ++i)
                if (f0 + 16 <= s.F || f0 + c + i < s.F)
                    lds_write<float>(to + i * s.stride, NAN_IS_INF ? fminf(v[u].v[i], __builtin_inff()) : v[u].v[i]);
        }
    }
    return at;
}

// The tile of NR row groups, P pieces in flight per lane.
template <int NR, int P, bool NAN_IS_INF>
__device__ __forceinline__ void tile_fill(const float *X, int64_t row0, int64_t n_rows, int F, uint32_t xbase, uint32_t group_stride,
                                          uint32_t stride, int wave, int lane)
{
    const int blocks = (F + 15) >> 4, pieces = blocks * (NR * 4);
    const TileShape s{X, n_rows, F, blocks, xbase, group_stride, stride};
    const int begin = pieces * wave / WALK_WAVES, end = pieces * (wave + 1) / WALK_WAVES;
    TilePiece at{begin / blocks, 0};
    at.block = begin - at.rows * blocks;
    for (int t = begin; t < end; t += P) {
        Float4 v[P];
        tile_load<P>(s, row0, at, end - t, lane, v);
        at = tile_store<P, NAN_IS_INF>(s, at, end - t, lane, v);
    }
}

}  // namespace forest_impl
