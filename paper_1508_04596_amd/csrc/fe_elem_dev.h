// Device helpers shared by the element kernels (internal).
#pragma once

#include "fe_batch.h"
#include "fe_internal.h"

namespace fe {

constexpr double QG = 0.57735026918962576451;  // Gauss abscissa 1/sqrt(3)

// Material interpolation (Eqs. conducint, alphaint) and derivatives.
__device__ __forceinline__ double alpha_of(const Geo &g, double y) { return g.amax * (1.0 - y) / (1.0 + g.qa * y); }
__device__ __forceinline__ double K_of(const Geo &g, double y)
{
    return (y * (g.Ck * (1.0 + g.qf) - 1.0) + 1.0) / (g.Ck * (1.0 + g.qf * y));
}
__device__ __forceinline__ double dalpha_of(const Geo &g, double y)
{
    double d = 1.0 + g.qa * y;
    return -g.amax * (1.0 + g.qa) / (d * d);
}
__device__ __forceinline__ double dK_of(const Geo &g, double y)
{
    double d = 1.0 + g.qf * y;
    return (1.0 + g.qf) * (g.Ck - 1.0) / (g.Ck * d * d);
}

// Workgroups are dispatched round-robin over the 8 XCDs (each with its own L2).
// Map workgroup b to a tile so that every XCD works through a contiguous range
// of tiles: neighbouring tiles, which re-read each other's face nodes, then
// share an L2.  A bijection on [0, n): the last n mod 8 tiles map to themselves.
__device__ __forceinline__ int xcd_tile(int b, int n)
{
    const int q = n >> 3;
    if (b >= (q << 3)) return b;
    return (b & 7) * q + (b >> 3);
}

__device__ __forceinline__ int64_t gnode(const Geo &g, int I, int J, int K)
{
    return (int64_t)I + (int64_t)(g.nx + 1) * ((int64_t)J + (int64_t)(g.ny + 1) * K);
}

// Is node coordinate I (local lx) shared with the neighbouring tile in that direction?
__device__ __forceinline__ bool shared_dir(int l, int I, int n, int T_)
{
    return (l == 0 && I > 0) || (l == T_ && I < n);
}

}  // namespace fe
