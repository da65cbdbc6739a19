// tile_dev.hpp -- what the kernels that work on TILE_X x TILE_Y x TILE_Z boxes
// share (k_tile, k_adj_tile): lane maps and scalar helpers.
#pragma once
#include "fdtd_dev.hpp"

constexpr int TX = TILE_X, TY = TILE_Y, TZ = TILE_Z;
static_assert(TX * TY == 256 && TZ == 4 && 2 * FDTD_R * TY * TZ == 256 && TY == 2 * FDTD_R, "lane maps of the halos");

__device__ __forceinline__ bool slab_point(int c, int n, int lo, int hi) {
    return c >= 0 && c < n && in_slab(c, n, lo, hi);
}
__device__ __forceinline__ float lane_value(float v, int lane) {
    return __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, v), lane));
}
__device__ __forceinline__ int uniform(int v) { return __builtin_amdgcn_readfirstlane(v); }
// the same scalar, its later tests computed anew: a test kept from one phase to the next costs two scalar
// registers each, and the kernels have none to spare
__device__ __forceinline__ int again(int v) {
    v = uniform(v);
    asm("" : "+s"(v));
    return v;
}
// bits o of the planes z0 + o, 0 <= o < N, inside [lo, hi)
template <int N> __device__ __forceinline__ uint32_t plane_bits(int z0, int lo, int hi) {
    const int a = min(max(lo - z0, 0), N), b = min(max(hi - z0, 0), N);
    return ((1u << b) - 1u) & ~((1u << a) - 1u);
}
// first derivative from LDS (or registers): taps at c[-4 stride] .. c[4 stride]
__device__ __forceinline__ float d1_lds(const float *c, int stride, const float *w) {
    float lo[4], hi[4];
#pragma unroll
    for (int l = 1; l <= 4; ++l) {
        lo[l - 1] = c[-l * stride];
        hi[l - 1] = c[l * stride];
    }
    return d1_axis(w, lo, hi);
}
