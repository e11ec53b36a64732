// PDE (Helmholtz) density filter on the element grid (Sec. "Optimisation
// problem": the design field is regularised by a PDE-based density filter).
//
//   -r^2 lap(psi) + psi = gamma,  zero normal derivative on the box boundary,
//
// psi trilinear on the nodes, gamma constant per element, r = R / (2 sqrt 3).
// Filtered element value = mean of psi over the element's nodes:
//   F gamma = A K^-1 T gamma,  F^T g = T^T K^-1 A^T g,  K = r^2 K_lap + M.
// The element matrix depends only on the Hamming distance of the two corners, so
// K couples a node with its 27 neighbours by four constants times the number of
// elements that hold both, and K psi = b is solved by Jacobi-preconditioned
// conjugate gradients with every scalar kept on the device.
//
// Two launches per iteration, or one on small grids (k_cg below; CG_ONE).  Of two, the
// first forms the direction p = z + beta p where K p needs it: a workgroup stages p of a
// plane of its tile and the rim in LDS, whose sums over the nine neighbours of a node
// serve three planes.  The second updates the residual, and x every other time.  The
// partial sums of a pass are added by every workgroup of the next, in the same order, in
// place of a launch of its own.
// Bound: up to about 10^6 nodes the latency of a pass (5.5 us: partial sums, then
// one plane after the other), above it memory (10 vectors per iteration; 160x160x320
// elements at about 3.9 TB/s).  Forward and transpose at 64x64x128, 24 iterations
// each: 2083 -> 969 us.  Before, K p gathered 64 values per node (20.7 us a pass) in
// five launches per iteration; 18 gathers per node from global memory instead of the
// staged plane took 15.3 us, staged 10.7.
#include <cstring>

#include "fe_elem_dev.h"
#include "fe_topopt.h"

namespace fe {
namespace {

__device__ __forceinline__ int64_t fnode(const FGeo &g, int I, int J, int K)
{
    return (int64_t)I + (int64_t)(g.nx + 1) * ((int64_t)J + (int64_t)(g.ny + 1) * K);
}

__device__ __forceinline__ void node_ijk(const FGeo &g, int64_t n, int &I, int &J, int &K)
{
    I = (int)(n % (g.nx + 1));
    const int64_t r = n / (g.nx + 1);
    J = (int)(r % (g.ny + 1));
    K = (int)(r / (g.ny + 1));
}

// block partial sums: out[j * RED_BLOCKS + blockIdx.x], j < NV
template <int NV>
__device__ __forceinline__ void block_partials(const double *v, double *out)
{
    __shared__ double red[NV][RED_THREADS / 64];
#pragma unroll
    for (int j = 0; j < NV; ++j) {
        double s = v[j];
        for (int o = 32; o > 0; o >>= 1) s += __shfl_down(s, o, 64);
        if ((threadIdx.x & 63) == 0) red[j][threadIdx.x >> 6] = s;
    }
    __syncthreads();
    if (threadIdx.x < NV) {
        double s = 0.0;
        for (int w = 0; w < RED_THREADS / 64; ++w) s += red[threadIdx.x][w];
        out[threadIdx.x * RED_BLOCKS + blockIdx.x] = s;
    }
}

// Element (i, j, k) in the caller's arrays.  THIN: x and z are exchanged here.
template <bool THIN>
__device__ __forceinline__ int64_t elem(const FGeo &g, int i, int j, int k)
{
    return THIN ? k + (int64_t)g.nz * (j + (int64_t)g.ny * i) : i + (int64_t)g.nx * (j + (int64_t)g.ny * k);
}

// node value = scale * sum of the element values around the node (T: h^3/8; A^T: 1/8)
template <bool THIN>
__global__ __launch_bounds__(256) void k_elem_to_node(FGeo g, const double *__restrict__ e,
                                                      double scale, double *__restrict__ out)
{
    const int64_t nn = (int64_t)(g.nx + 1) * (g.ny + 1) * (g.nz + 1);
    const int64_t n = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (n >= nn) return;
    int I, J, K;
    node_ijk(g, n, I, J, K);
    double acc = 0.0;
    for (int ez = K - 1; ez <= K; ++ez) {
        if (ez < 0 || ez >= g.nz) continue;
        for (int ey = J - 1; ey <= J; ++ey) {
            if (ey < 0 || ey >= g.ny) continue;
            for (int ex = I - 1; ex <= I; ++ex) {
                if (ex < 0 || ex >= g.nx) continue;
                acc += e[elem<THIN>(g, ex, ey, ez)];
            }
        }
    }
    out[n] = scale * acc;
}

// element value = scale * sum of its 8 node values (A: 1/8; T^T: h^3/8)
template <bool THIN>
__global__ __launch_bounds__(256) void k_node_to_elem(FGeo g, const double *__restrict__ nv,
                                                      double scale, double *__restrict__ out)
{
    const int64_t ne = (int64_t)g.nx * g.ny * g.nz;
    const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= ne) return;
    const int i = (int)(e % g.nx), j = (int)((e / g.nx) % g.ny), k = (int)(e / ((int64_t)g.nx * g.ny));
    double acc = 0.0;
#pragma unroll
    for (int b = 0; b < 8; ++b) acc += nv[fnode(g, i + (b & 1), j + ((b >> 1) & 1), k + (b >> 2))];
    out[THIN ? elem<THIN>(g, i, j, k) : e] = scale * acc;
}

// Work of the CG passes: tiles of wx x wy nodes (at most 256, one per thread) times
// cz planes, spread over at most RED_BLOCKS workgroups (one partial sum each).
struct CgTiling {
    int wx, wy, cz;      // nodes of a tile
    int nx, ny, tiles;   // tiles along x and y, all tiles
};
constexpr int TILE_W = 40;                            // most nodes of a tile along x
constexpr int TILE_HALO = (2 + 2) * (RED_THREADS / 2 + 2);  // largest tile with its rim (2 x 128)

// This thread's node column of a tile.
struct Column {
    bool in;
    int I0, J0, K0, K1;             // first node of the tile, planes
    int I, J;
    int64_t n, plane;               // node in its plane, nodes of a plane
    double wxm, wxp, wym, wyp;      // 1 if there is a neighbour on that side, else 0
    double cx, cy;                  // elements along x and y (1 or 2)
};

// First tile of workgroup b: consecutive tiles, so that neighbours share an XCD's L2.
__device__ __forceinline__ int tile_begin(const CgTiling &t, int b)
{
    return (int)((int64_t)t.tiles * b / (int)gridDim.x);
}

__device__ __forceinline__ Column column(const FGeo &g, const CgTiling &t, int tile)
{
    Column c;
    const int bx = tile % t.nx, r = tile / t.nx, by = r % t.ny, bz = r / t.ny;
    const int ly = (int)threadIdx.x / t.wx, lx = (int)threadIdx.x - ly * t.wx;
    c.I0 = bx * t.wx;
    c.J0 = by * t.wy;
    c.I = c.I0 + lx;
    c.J = c.J0 + ly;
    c.in = ly < t.wy && c.I <= g.nx && c.J <= g.ny;
    c.K0 = bz * t.cz;
    c.K1 = min(c.K0 + t.cz, g.nz + 1);
    c.plane = (int64_t)(g.nx + 1) * (g.ny + 1);
    c.n = c.in ? c.I + (int64_t)(g.nx + 1) * c.J : 0;
    c.wxm = c.I > 0;
    c.wxp = c.I < g.nx;
    c.wym = c.J > 0;
    c.wyp = c.J < g.ny;
    c.cx = c.wxm + c.wxp;
    c.cy = c.wym + c.wyp;
    return c;
}

// Sum of nparts block partials, the same in every workgroup.
__device__ __forceinline__ double total(const double *__restrict__ partial, int nparts)
{
    __shared__ double red[RED_THREADS / 64];
    double s = 0.0;
    for (int q = threadIdx.x; q < nparts; q += RED_THREADS) s += partial[q];
    for (int o = 32; o > 0; o >>= 1) s += __shfl_down(s, o, 64);
    __syncthreads();
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = s;
    __syncthreads();
    double v = 0.0;
    for (int w = 0; w < RED_THREADS / 64; ++w) v += red[w];
    return v;
}

// The first workgroup's: the sum of <r, r>'s partials for the host, in pinned memory.
__device__ __forceinline__ void tell_rr0(const double *__restrict__ prr, int nparts, double *rr0)
{
    if (blockIdx.x != 0) return;
    const double rr = total(prr, nparts);
    if (threadIdx.x == 0) __hip_atomic_store(rr0, rr, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}

// Sums of a staged plane (u: its tile with the rim) over a node itself, its edge
// neighbours and its corner neighbours, each weighted by the elements along x and y in
// common.
struct Sums {
    double a0, a1, a2, p;
};
__device__ __forceinline__ Sums plane_sums(const double *u, const Column &c, const CgTiling &t)
{
    const int sx = t.wx + 2;
    const int at = ((int)threadIdx.x / t.wx + 1) * sx + (int)threadIdx.x % t.wx + 1;
    const double *P = u + (c.in ? at : sx + 1);
    Sums s;
    s.p = P[0];
    s.a0 = c.cx * c.cy * s.p;
    s.a1 = c.cy * (P[-1] + P[1]) + c.cx * (P[-sx] + P[sx]);
    s.a2 = (P[-sx - 1] + P[-sx + 1]) + (P[sx - 1] + P[sx + 1]);
    return s;
}
// (K u) of a node with cz elements along z from its three planes' sums
__device__ __forceinline__ double stencil(const FGeo &g, double cz, const Sums &lo, const Sums &me,
                                          const Sums &hi)
{
    return cz * (g.E[0] * me.a0 + g.E[1] * me.a1 + g.E[2] * me.a2) + g.E[1] * (lo.a0 + hi.a0) +
           g.E[2] * (lo.a1 + hi.a1) + g.E[3] * (lo.a2 + hi.a2);
}

// CG start from x = 0: z = D^-1 b (D = E0 times the node's elements); partials of
// <r, z> and <r, r>.
__global__ __launch_bounds__(RED_THREADS) void k_cg_init(FGeo g, CgTiling t, double iE0,
                                                         const double *__restrict__ b,
                                                         double *__restrict__ x,
                                                         double *__restrict__ z, double *prz)
{
    double v[2] = {0.0, 0.0};
    const int lb = xcd_tile((int)blockIdx.x, (int)gridDim.x);
    const int t1 = tile_begin(t, lb + 1);
    for (int tile = tile_begin(t, lb); tile < t1; ++tile) {
        const Column c = column(g, t, tile);
        if (!c.in) continue;
        for (int K = c.K0; K < c.K1; ++K) {
            const int64_t n = c.n + c.plane * K;
            const double cz = (K > 0) + (K < g.nz);
            const double rn = b[n], zn = rn * (iE0 / (c.cx * c.cy * cz));
            x[n] = 0.0;
            z[n] = zn;
            v[0] += rn * zn;
            v[1] += rn * rn;
        }
    }
    block_partials<2>(v, prz);
}

// p = z + beta p_old (z in the first iteration), y = K p, partials of <p, y>.
// rr0: pinned memory for <r, r> of the start (FIRST).
// beta = rz / rz_old: rz from the last pass's nparts partials, kept in sc[cur] for the
// passes that follow; rz_old = sc[1 - cur].
template <bool FIRST>
__global__ __launch_bounds__(RED_THREADS) void k_cg_apply(FGeo g, CgTiling t, int nparts,
                                                          const double *__restrict__ prz,
                                                          double *sc, int cur,
                                                          const double *__restrict__ z,
                                                          const double *__restrict__ pold,
                                                          double *__restrict__ p,
                                                          double *__restrict__ y, double *ppy,
                                                          double *rr0)
{
    __shared__ double w[2][TILE_HALO];  // p of a plane of the tile and its rim, ring of two
    const int sx = t.wx + 2, halo = sx * (t.wy + 2);
    constexpr int NL = (TILE_HALO + RED_THREADS - 1) / RED_THREADS;
    double v = 0.0, beta = 0.0;
    bool first = true;
    const int lb = xcd_tile((int)blockIdx.x, (int)gridDim.x);
    const int t1 = tile_begin(t, lb + 1);
    for (int tile = tile_begin(t, lb); tile < t1; ++tile) {
        const Column c = column(g, t, tile);
        // this thread's values of the rimmed plane (0 outside the grid)
        int64_t off[NL];
        bool ok[NL];
#pragma unroll
        for (int q = 0; q < NL; ++q) {
            const int e = (int)threadIdx.x + q * RED_THREADS, hy = e / sx, hx = e - hy * sx;
            const int I = c.I0 + hx - 1, J = c.J0 + hy - 1;
            ok[q] = e < halo && I >= 0 && I <= g.nx && J >= 0 && J <= g.ny;
            off[q] = ok[q] ? I + (int64_t)(g.nx + 1) * J : 0;
        }
        double zr[NL], pr[NL];
        auto load = [&](int K) {
            const int64_t b = c.plane * K;
#pragma unroll
            for (int q = 0; q < NL; ++q)
                if (q * RED_THREADS < halo) {
                    zr[q] = z[b + off[q]];
                    pr[q] = FIRST ? 0.0 : pold[b + off[q]];
                }
        };
        auto stage = [&](int b) {
#pragma unroll
            for (int q = 0; q < NL; ++q) {
                const int e = (int)threadIdx.x + q * RED_THREADS;
                if (e < halo) w[b][e] = ok[q] ? (FIRST ? zr[q] : fma(beta, pr[q], zr[q])) : 0.0;
            }
        };
        const Sums none = {0.0, 0.0, 0.0, 0.0};
        const int Ka = max(c.K0 - 1, 0), Kb = min(c.K1, g.nz);  // planes to stage
        load(Ka);
        if (first) {
            const double rz = total(prz, nparts), old = FIRST ? 1.0 : sc[1 - cur];
            if (blockIdx.x == 0 && threadIdx.x == 0) sc[cur] = rz;
            if (FIRST) {
                tell_rr0(prz + RED_BLOCKS, nparts, rr0);
                if (!(rz > 0.0)) return;  // the host ends the solve (first_look)
            }
            beta = old > 0.0 ? rz / old : 0.0;
            first = false;
        } else {
            __syncthreads();  // the last tile's planes have been read
        }
        Sums lo = none, me = none;
        for (int K = Ka; K <= Kb + 1; ++K) {
            // plane K joins; plane K - 1 is complete
            Sums hi = none;
            if (K <= Kb) {
                stage(K & 1);
                if (K < Kb) load(K + 1);
                __syncthreads();
                hi = plane_sums(w[K & 1], c, t);
            }
            const int Ko = K - 1;
            if (c.in && Ko >= c.K0 && Ko < c.K1) {
                const double cz = (Ko > 0) + (Ko < g.nz);
                const double yn = stencil(g, cz, lo, me, hi);
                const int64_t n = c.n + c.plane * Ko;
                p[n] = me.p;
                y[n] = yn;
                v += me.p * yn;
            }
            lo = me;
            me = hi;
        }
    }
    block_partials<1>(&v, ppy);
}

// alpha = rz / <p, y>; r -= alpha y, kept as z = D^-1 r; partials of <r, z> and
// <r, r>.  x is updated every other iteration (X), with both directions at hand:
// x += alpha_old p_old + alpha p, alpha_old as the iteration before left it in
// sc[2] (both = 0: x += alpha p).  A zero right-hand side leaves x = 0.
template <bool X>
__global__ __launch_bounds__(RED_THREADS) void k_cg_step(FGeo g, CgTiling t, int nparts, double iE0,
                                                         const double *__restrict__ ppy, double *sc,
                                                         int cur, int both,
                                                         const double *__restrict__ pold,
                                                         const double *__restrict__ p,
                                                         const double *__restrict__ y,
                                                         double *__restrict__ x,
                                                         double *__restrict__ z, double *prz)
{
    const double py = total(ppy, nparts), rz = sc[cur];
    const double alpha = rz == 0.0 && py == 0.0 ? 0.0 : rz / py;
    const double before = X && both ? sc[2] : 0.0;
    if (!X && blockIdx.x == 0 && threadIdx.x == 0) sc[2] = alpha;
    if (!X && !(rz > 0.0)) return;  // z = 0 or NaN: prz stays as it is
    double v[2] = {0.0, 0.0};
    const int lb = xcd_tile((int)blockIdx.x, (int)gridDim.x);
    const int t1 = tile_begin(t, lb + 1);
    for (int tile = tile_begin(t, lb); tile < t1; ++tile) {
        const Column c = column(g, t, tile);
        if (!c.in) continue;
        const double cxy = c.cx * c.cy;
#pragma unroll 2
        for (int K = c.K0; K < c.K1; ++K) {
            const int64_t n = c.n + c.plane * K;
            const double cnt = (K > 0 && K < g.nz) ? 2.0 * cxy : cxy;
            if (X) {
                double xn = fma(alpha, p[n], x[n]);
                if (both) xn = fma(before, pold[n], xn);
                x[n] = xn;
            }
            const double zn = z[n] - alpha * y[n] * (iE0 / cnt);
            z[n] = zn;
            const double rn = zn * (g.E[0] * cnt);
            v[0] += rn * zn;
            v[1] += rn * rn;
        }
    }
    block_partials<2>(v, prz);
}

// Sums of the nparts block partials of two quantities, the same in every workgroup.
__device__ __forceinline__ void totals(const double *__restrict__ partial, int nparts, double &a,
                                       double &b)
{
    __shared__ double red[2][RED_THREADS / 64];
    double s[2] = {0.0, 0.0};
    for (int q = threadIdx.x; q < nparts; q += RED_THREADS) {
        s[0] += partial[q];
        s[1] += partial[RED_BLOCKS + q];
    }
#pragma unroll
    for (int j = 0; j < 2; ++j) {
        for (int o = 32; o > 0; o >>= 1) s[j] += __shfl_down(s[j], o, 64);
        if ((threadIdx.x & 63) == 0) red[j][threadIdx.x >> 6] = s[j];
    }
    __syncthreads();
    a = b = 0.0;
    for (int w = 0; w < RED_THREADS / 64; ++w) {
        a += red[0][w];
        b += red[1][w];
    }
}

// Vectors of an iteration: u = D^-1 r (D = E0 times the node's elements), w = K u and
// s = K p are read with the tile's rim and written to their second buffers, p and x are
// updated in place.
struct CgVec {
    const double *u, *w, *s;
    double *un, *wn, *sn, *p, *x;
};

// One iteration in one launch (Chronopoulos and Gear's form of conjugate gradients, for
// small grids): from the last pass's partials of rz = <r, u> and uw = <u, w>,
//   beta = rz / rz_old,  alpha = rz / (uw - beta rz / alpha_old),
//   p = u + beta p,  s = w + beta s,  x += alpha p,  u -= alpha D^-1 s,  w = K u,
// and the partials of the new rz, uw and <r, r> (out).  rz and alpha are kept in
// sc[2 cur], sc[2 cur + 1] for the next.  CG_INIT: u = D^-1 b (v.u = b), x = 0.
// CG_FIRST: the first iteration, s = p = 0 are not read; rr0: pinned memory for <r, r> of
// the start.  x is updated every other
// iteration, with both directions at hand: xmode 0 no, 1 x += alpha p, 2 x +=
// alpha_old p_old + alpha p.  A zero right-hand side leaves x = 0.
enum CgPass { CG_INIT, CG_FIRST, CG_NEXT };
template <CgPass PASS>
__global__ __launch_bounds__(RED_THREADS) void k_cg(FGeo g, CgTiling t, int nparts, double iE0,
                                                    const double *__restrict__ partial, double *sc,
                                                    int cur, int xmode, CgVec vec,
                                                    double *out, double *rr0)
{
    __shared__ double P2[2][TILE_HALO];  // u of a plane of the tile and its rim, ring of two
    constexpr bool INIT = PASS == CG_INIT, fresh = PASS == CG_FIRST;
    const double E0 = g.E[0];
    const int sx = t.wx + 2, halo = sx * (t.wy + 2);
    constexpr int NL = (TILE_HALO + RED_THREADS - 1) / RED_THREADS;
    const double *__restrict__ u = vec.u;
    const double *__restrict__ w = vec.w;
    const double *__restrict__ s = vec.s;
    double v[3] = {0.0, 0.0, 0.0};
    double alpha = 0.0, beta = 0.0, before = 0.0;
    bool first = true;
    const int lb = xcd_tile((int)blockIdx.x, (int)gridDim.x);
    const int t1 = tile_begin(t, lb + 1);
    for (int tile = tile_begin(t, lb); tile < t1; ++tile) {
        const Column c = column(g, t, tile);
        // this thread's values of the rimmed plane: in the grid, in the tile itself
        // (those it also updates), elements along x and y
        int64_t off[NL];
        bool ok[NL], mine[NL];
        double cxy[NL], id[NL];
#pragma unroll
        for (int q = 0; q < NL; ++q) {
            const int e = (int)threadIdx.x + q * RED_THREADS, hy = e / sx, hx = e - hy * sx;
            const int I = c.I0 + hx - 1, J = c.J0 + hy - 1;
            ok[q] = e < halo && I >= 0 && I <= g.nx && J >= 0 && J <= g.ny;
            mine[q] = ok[q] && hx >= 1 && hx <= t.wx && hy >= 1 && hy <= t.wy;
            off[q] = ok[q] ? I + (int64_t)(g.nx + 1) * J : 0;
            cxy[q] = ((I > 0) + (I < g.nx)) * ((J > 0) + (J < g.ny));
            id[q] = ok[q] ? iE0 / cxy[q] : 0.0;
        }
        double ur[NL], wr[NL], sr[NL], pr[NL], xr[NL];
        auto load = [&](int K) {
            const int64_t b = c.plane * K;
            const bool own = K >= c.K0 && K < c.K1;
#pragma unroll
            for (int q = 0; q < NL; ++q)
                if (q * RED_THREADS < halo) {
                    ur[q] = u[b + off[q]];
                    if (INIT) continue;
                    wr[q] = w[b + off[q]];
                    sr[q] = fresh ? 0.0 : s[b + off[q]];
                    pr[q] = own && mine[q] && !fresh ? vec.p[b + off[q]] : 0.0;
                    xr[q] = own && mine[q] && xmode ? vec.x[b + off[q]] : 0.0;
                }
        };
        auto stage = [&](int K) {
            const int64_t b = c.plane * K;
            const bool own = K >= c.K0 && K < c.K1;
            const bool inner = K > 0 && K < g.nz;  // two elements along z
#pragma unroll
            for (int q = 0; q < NL; ++q) {
                const int e = (int)threadIdx.x + q * RED_THREADS;
                if (e >= halo) continue;
                const double di = inner ? 0.5 * id[q] : id[q];
                const double sn = INIT ? 0.0 : fma(beta, sr[q], wr[q]);
                const double un = ok[q] ? (INIT ? ur[q] * di : ur[q] - alpha * sn * di) : 0.0;
                P2[K & 1][e] = un;
                if (!(own && mine[q])) continue;
                const int64_t n = b + off[q];
                vec.un[n] = un;
                if (INIT) {
                    vec.x[n] = 0.0;
                } else {
                    const double pn = fma(beta, pr[q], ur[q]);
                    vec.sn[n] = sn;
                    vec.p[n] = pn;
                    if (xmode) vec.x[n] = fma(alpha, pn, xmode == 2 ? fma(before, pr[q], xr[q]) : xr[q]);
                }
                const double rn = un * (E0 * cxy[q] * (inner ? 2.0 : 1.0));
                v[0] += rn * un;
                v[2] += rn * rn;
            }
        };
        const Sums none = {0.0, 0.0, 0.0, 0.0};
        const int Ka = max(c.K0 - 1, 0), Kb = min(c.K1, g.nz);  // planes to stage
        load(Ka);
        if (!first) {
            __syncthreads();  // the last tile's planes have been read
        } else if (!INIT) {
            double rz, uw;
            totals(partial, nparts, rz, uw);
            if (fresh) tell_rr0(partial + 2 * RED_BLOCKS, nparts, rr0);
            const double old = fresh ? 0.0 : sc[2 - 2 * cur];
            before = fresh ? 0.0 : sc[3 - 2 * cur];
            beta = old > 0.0 ? rz / old : 0.0;
            const double d = beta == 0.0 ? uw : uw - beta * rz / before;
            alpha = rz == 0.0 && uw == 0.0 ? 0.0 : rz / d;
            if (blockIdx.x == 0 && threadIdx.x == 0) {
                sc[2 * cur] = rz;
                sc[2 * cur + 1] = alpha;
            }
        }
        first = false;
        Sums lo = none, me = none;
        for (int K = Ka; K <= Kb + 1; ++K) {
            // plane K joins; plane K - 1 is complete
            Sums hi = none;
            if (K <= Kb) {
                stage(K);
                if (K < Kb) load(K + 1);
                __syncthreads();
                hi = plane_sums(P2[K & 1], c, t);
            }
            const int Ko = K - 1;
            if (c.in && Ko >= c.K0 && Ko < c.K1) {
                const double cz = (Ko > 0) + (Ko < g.nz);
                const double wn = stencil(g, cz, lo, me, hi);
                vec.wn[c.n + c.plane * Ko] = wn;
                v[1] += me.p * wn;
            }
            lo = me;
            me = hi;
        }
    }
    block_partials<3>(v, out);
}

inline unsigned nblk(int64_t n) { return (unsigned)((n + 255) / 256); }

}  // namespace

// ---- host side --------------------------------------------------------------------

// Largest grid (nodes) whose iteration is one launch: up to there a pass's latency
// bounds, above it the rims of the three vectors it stages cost more than the launch (us
// per solve, two launches / one: 16^3 350 268, 32x32x64 355 290, 48x48x96 387 344, 64^3
// 396 375, 64x64x96 425 414, 64x64x128 484 503, 96^3 628 943).  Only up to there are its
// second buffers allocated.
constexpr int64_t CG_ONE = 300000;

hipError_t filter_alloc(Filter *f, const fe_grid &grid, double radius)
{
    const double h = grid.h, r = radius / (2.0 * 1.7320508075688772935);
    const double kap[4] = {1.0 / 3.0, 0.0, -1.0 / 12.0, -1.0 / 12.0};
    const double mu[4] = {8.0, 4.0, 2.0, 1.0};
    // The passes give a thread to every node of an x-y tile and walk along z, so a column
    // of few nodes across leaves most threads idle: its x and z are exchanged (the element
    // matrix does not tell the axes apart, and only the element arrays keep the caller's
    // order).  us per solve, along z / exchanged: 1x1x9000 961 274, 2x2x40000 1289 443,
    // 4x4x2000 320 278; 6x6x2000, wide enough, 324 354, and 6x6x60, whose tiles have one
    // plane, 247 281.
    f->thin = (int64_t)(grid.nx + 1) * (grid.ny + 1) <= 32 && grid.nz > 512;
    f->g.nx = f->thin ? grid.nz : grid.nx;
    f->g.ny = grid.ny;
    f->g.nz = f->thin ? grid.nx : grid.nz;
    for (int d = 0; d < 4; ++d) f->g.E[d] = r * r * h * kap[d] + h * h * h / 216.0 * mu[d];
    f->nn = (int64_t)(grid.nx + 1) * (grid.ny + 1) * (grid.nz + 1);
    f->ne = (int64_t)grid.nx * grid.ny * grid.nz;
    f->load = h * h * h / 8.0;
    const size_t nb = sizeof(double) * f->nn;
    hipError_t e = hipMalloc(&f->b, nb);
    if (e == hipSuccess) e = hipMalloc(&f->x, nb);
    if (e == hipSuccess) e = hipMalloc(&f->r, nb);
    if (e == hipSuccess) e = hipMalloc(&f->p, nb);
    if (e == hipSuccess) e = hipMalloc(&f->y, nb);
    for (double **q : {&f->r2, &f->y2, &f->s2})
        if (e == hipSuccess && f->nn <= CG_ONE) e = hipMalloc(q, nb);
    if (e == hipSuccess) e = hipMalloc(&f->partial, sizeof(double) * 6 * RED_BLOCKS);
    if (e == hipSuccess) e = hipMalloc(&f->sc, sizeof(double) * 8);
    if (e == hipSuccess) e = hipHostMalloc(&f->hsc, sizeof(double) * 8);
    if (e == hipSuccess) e = hipHostGetDevicePointer((void **)&f->dhsc, f->hsc, 0);
    return e;
}

void filter_free(Filter *f)
{
    for (double *q : {f->b, f->x, f->r, f->p, f->y, f->r2, f->y2, f->s2, f->partial, f->sc})
        if (q) (void)hipFree(q);
    if (f->hsc) (void)hipHostFree(f->hsc);
}

// Tiles as wide as divides the grid best, up to TILE_W.  Planes per tile: each tile
// stages two planes more than it has, but fewer tiles than 1.5 per CU leave the chip
// idle and one plane per tile doubles what a tile stages (us per solve at 1 / 2 / 4 /
// 6 / 8 planes, 24 iterations: 32x32x64 340 294 372 379 393; 64x64x128 591 539 481
// 469 514; 96^3 706 656 669 568 631; 160x160x320 5503 4900 4694 4655 4585).
// One launch per iteration (small grids): as few planes as keep all tiles resident, two
// per CU (40x40x80 with 648 tiles of one plane: 453, with 324 of two: 333).
static CgTiling cg_tiling(const FGeo &g, bool one)
{
    CgTiling t;
    t.nx = (g.nx + TILE_W) / TILE_W;
    t.wx = (g.nx + t.nx) / t.nx;
    t.wy = std::min(RED_THREADS / t.wx, g.ny + 1);
    t.ny = (g.ny + t.wy) / t.wy;
    const int64_t planes = (int64_t)t.nx * t.ny * (g.nz + 1);
    const int64_t cz = one ? (planes + 511) / 512 : std::max<int64_t>(2, planes / 400);
    t.cz = (int)std::min<int64_t>(std::min<int64_t>(cz, 8), g.nz + 1);
    t.tiles = t.nx * t.ny * ((g.nz + t.cz) / t.cz);
    return t;
}

// What hsc[5] holds until the first iteration's kernel writes <r, r> of the start there.
constexpr double RR0_AWAITED = -1.0;

// The look at <r, r> of the start, taken with the first iteration under way: a zero or
// non-finite right-hand side ends here with x = 0, not after eight iterations (us per solve, eight /
// here: 16^3 122 37, 64x64x128 194 42, 160x160x320 1475 178).  So does one whose target
// rtol^2 rr0 is below the range of a double: <r, r>, of the same size, would pass as
// converged when its terms underflow.  FE_PENDING: go on.
// The host reads the word itself: an event between the passes took 6 us more per solve
// (16^3: 276 against 270).  The wait ends with the stream's work or its error at the
// latest.
static int first_look(Filter *f, double rtol, hipStream_t st)
{
    double rr0;
    for (int n = 1;; ++n) {
        __atomic_load(f->hsc + 5, &rr0, __ATOMIC_ACQUIRE);
        if (rr0 != RR0_AWAITED) break;
        __builtin_ia32_pause();
        if (n % 4096 == 0) {
            const hipError_t e = hipStreamQuery(st);
            if (e == hipErrorNotReady) continue;
            FE_CHECK_HIP(e);
            __atomic_load(f->hsc + 5, &rr0, __ATOMIC_ACQUIRE);
            break;
        }
    }
    f->last_its = 0;
    if (rr0 == 0.0) return FE_OK;
    const bool bad = !(rr0 > 0.0) || !std::isfinite(rr0);
    if (!bad && rtol * rtol * rr0 > 0.0) return FE_PENDING;
    FE_CHECK_HIP(hipStreamSynchronize(st));  // (an error leaves no pass running)
    return bad ? FE_ENAN : FE_NOT_CONVERGED;
}

// After iteration it: FE_PENDING to go on (prr: the partials of <r, r>).
static int converged(Filter *f, const double *prr, int nb, int it, double rtol, hipStream_t st)
{
    FE_CHECK_HIP(launch_reduce(prr, 1, f->sc + 4, nullptr, false, st, nb));
    FE_CHECK_HIP(hipMemcpyAsync(f->hsc + 4, f->sc + 4, sizeof(double), hipMemcpyDeviceToHost, st));
    FE_CHECK_HIP(hipStreamSynchronize(st));
    const double rr = f->hsc[4], rr0 = f->hsc[5];
    f->last_its = it;
    if (!std::isfinite(rr)) return FE_ENAN;
    return rr <= rtol * rtol * rr0 ? FE_OK : FE_PENDING;
}

static int solve_one(Filter *f, hipStream_t st, double rtol, int max_its)
{
    const FGeo &g = f->g;
    const CgTiling t = cg_tiling(g, true);
    const int nb = std::min(t.tiles, RED_BLOCKS);
    const dim3 gb(nb), gt(RED_THREADS);
    // partials of rz, uw and rr, two sets in turn; sc: rz and alpha of the last two
    // iterations, then rr
    double *part[2] = {f->partial, f->partial + 3 * RED_BLOCKS};
    const double iE0 = 1.0 / g.E[0];
    CgVec v = {f->b, nullptr, nullptr, f->r, f->y, nullptr, f->p, f->x};
    hipLaunchKernelGGL(k_cg<CG_INIT>, gb, gt, 0, st, g, t, nb, iE0, (const double *)nullptr, f->sc, 0,
                       0, v, part[0], f->dhsc + 5);
    FE_CHECK_HIP(hipGetLastError());
    int rc;
    f->hsc[5] = RR0_AWAITED;
    v = {f->r, f->y, f->s2, f->r2, f->y2, f->b, f->p, f->x};
    for (int it = 1; it <= max_its; ++it) {
        const int cur = it & 1;
        hipLaunchKernelGGL(it == 1 ? k_cg<CG_FIRST> : k_cg<CG_NEXT>, gb, gt, 0, st, g, t, nb, iE0,
                           (const double *)part[1 - cur], f->sc, cur, it % 2 == 0 ? 2 : it == max_its ? 1 : 0, v, part[cur],
                           f->dhsc + 5);
        FE_CHECK_HIP(hipGetLastError());
        v = {v.un, v.wn, v.sn, const_cast<double *>(v.u), const_cast<double *>(v.w),
             const_cast<double *>(v.s), f->p, f->x};
        if (it == 1 && (rc = first_look(f, rtol, st)) != FE_PENDING) return rc;
        if (it % 8 == 0 || it == max_its) {
            rc = converged(f, part[cur] + 2 * RED_BLOCKS, nb, it, rtol, st);
            if (rc != FE_PENDING) return rc;
        }
    }
    return FE_NOT_CONVERGED;
}

static int solve_two(Filter *f, hipStream_t st, double rtol, int max_its)
{
    const FGeo &g = f->g;
    const CgTiling t = cg_tiling(g, false);
    const int nb = std::min(t.tiles, RED_BLOCKS);
    const dim3 gb(nb), gt(RED_THREADS);
    double *ppy = f->partial, *prz = f->partial + RED_BLOCKS, *prr = prz + RED_BLOCKS;
    const double iE0 = 1.0 / g.E[0];
    hipLaunchKernelGGL(k_cg_init, gb, gt, 0, st, g, t, iE0, (const double *)f->b, f->x, f->r, prz);
    FE_CHECK_HIP(hipGetLastError());
    // sc[0], sc[1]: rz of the last two iterations; sc[2]: alpha of the one before
    int rc;
    f->hsc[5] = RR0_AWAITED;
    double *pn = f->p, *po = f->b;
    int cur = 0;
    for (int it = 1; it <= max_its; ++it) {
        if (it == 1)
            hipLaunchKernelGGL(k_cg_apply<true>, gb, gt, 0, st, g, t, nb, (const double *)prz, f->sc,
                               cur, (const double *)f->r, (const double *)po, pn, f->y, ppy,
                               f->dhsc + 5);
        else
            hipLaunchKernelGGL(k_cg_apply<false>, gb, gt, 0, st, g, t, nb, (const double *)prz,
                               f->sc, cur, (const double *)f->r, (const double *)po, pn, f->y, ppy,
                               f->dhsc + 5);
        if (it % 2 == 0 || it == max_its)
            hipLaunchKernelGGL(k_cg_step<true>, gb, gt, 0, st, g, t, nb, iE0, (const double *)ppy,
                               f->sc, cur, it % 2 == 0, (const double *)po, (const double *)pn,
                               (const double *)f->y, f->x, f->r, prz);
        else
            hipLaunchKernelGGL(k_cg_step<false>, gb, gt, 0, st, g, t, nb, iE0, (const double *)ppy,
                               f->sc, cur, 0, (const double *)po, (const double *)pn,
                               (const double *)f->y, f->x, f->r, prz);
        FE_CHECK_HIP(hipGetLastError());
        cur = 1 - cur;
        std::swap(pn, po);
        if (it == 1 && (rc = first_look(f, rtol, st)) != FE_PENDING) return rc;
        if (it % 8 == 0 || it == max_its) {
            rc = converged(f, prr, nb, it, rtol, st);
            if (rc != FE_PENDING) return rc;
        }
    }
    return FE_NOT_CONVERGED;
}

// psi = K^-1 b (b, psi: the filter's own node buffers b and x; b is overwritten);
// returns FE_OK, FE_NOT_CONVERGED or an error
int filter_solve(Filter *f, hipStream_t st, double rtol, int max_its)
{
    return f->s2 ? solve_one(f, st, rtol, max_its) : solve_two(f, st, rtol, max_its);
}

hipError_t filter_load(Filter *f, const double *gamma, double scale, hipStream_t st)
{
    hipLaunchKernelGGL(f->thin ? k_elem_to_node<true> : k_elem_to_node<false>, dim3(nblk(f->nn)),
                       dim3(256), 0, st, f->g, gamma, scale, f->b);
    return hipGetLastError();
}

hipError_t filter_unload(Filter *f, double scale, double *out, hipStream_t st)
{
    hipLaunchKernelGGL(f->thin ? k_node_to_elem<true> : k_node_to_elem<false>, dim3(nblk(f->ne)),
                       dim3(256), 0, st, f->g, (const double *)f->x, scale, out);
    return hipGetLastError();
}

}  // namespace fe
