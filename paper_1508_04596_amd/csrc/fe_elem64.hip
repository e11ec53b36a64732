// FP64 operator passes on gfx950: residual, J v and J^T w, four lanes per element.
//
// Lane q = 0..3 of an element stands for the x-y Gauss point (qx, qy) =
// (q & 1, q >> 1) and for the x-y corner of the same number, and there for both
// Gauss points along z and both corners of the z edge.  A workgroup marches
// through its tile's layers of 8x8 elements (16 per wave); a wave's four lane
// groups of 16 are the four q of its 16 elements, so that the interpolation in x
// and y and its transpose are constant 4x4 matrices across lane groups, each one
// v_mfma_f64_4x4x4 (operand: row q, column element; result the same).
//
// Why four lanes.  One lane per element needs 410 registers in FP64, hence one wave
// per SIMD, with nothing to issue while it waits, and 750 moves to and from the
// accumulation registers per element: 51.9 us for J v at 64^3 and 1.495 ms at
// 160x160x320.  A quarter of the state fits 256 registers, two waves share a SIMD
// and cover each other's waits: 38.5 us and 0.94 ms (residual 0.86 -> 0.70 ms,
// J^T w 1.54 -> 1.00 ms), about 82 % of the issue slots of the layer loop in use.
// What bounds it is FP64 issue: the matrix unit does not run beside the vector
// unit (32 fma take 154 cycles of a SIMD, 8 of these products 138, both together
// 286), so a product costs four fma and is used only where the lanes' exchange
// would cost more.  A layer of 16 elements takes about 345 FP64 operations and 92
// products: 21 slots per field of the state, whose node planes are interpolated
// once and serve the layers on both sides, 32 per field of the direction, whose
// planes would not fit the registers (it is interpolated at each point anew),
// 39 per row on the test side, 107 per Gauss point.  Measured and not taken:
// reading all four corners from LDS instead of the products (8 operations per
// field and plane, but LDS bandwidth then bounds: 1.23 ms at 160x160x320); both
// directions' planes kept (spills); FP32 in the same form (its exchange is a
// modifier of the operation and one lane per element fits two waves: 0.64 against
// 0.67 ms at 160x160x320 but 31 against 28 us at 64^3, so FP32 keeps one lane).
//
// Gradients are kept times h.  With alpha' = alpha h, K' = K / h, Pr' = Pr / h,
// B' = B h, s' = s h, tau' = tau / h and strong residuals times h, every formula
// keeps its form, tau'^-2 = |u_e|^2 / 16 + 16 Pr'^2 + alpha'^2 and
// tauT'^-2 = |u_e|^2 / 16 + 16 K'^2 lose h, and the rows carry the factor h^2 / 8.
//
// Nodes whose elements all lie in the tile are written directly, nodes on faces
// shared with neighbouring tiles go to per-tile slots, which the shared-node pass
// (fe_elem.hip) adds in a fixed order.  No atomics: results are bitwise
// reproducible.
#include "fe_elem_dev.h"

namespace fe {
namespace {

constexpr double WLO = 0.5 * (1.0 - QG), WHI = 0.5 * (1.0 + QG);  // linear weights at a Gauss point

// 1 / sqrt(a), a > 0: the hardware estimate and one correction step, within one
// unit in the last place (the error of 1 / sqrt(a) in two rounded operations).
// |u_e|^2 overflows from |u| = 2e153 on: 1 / sqrt(inf) = 0, where the step's 1 - inf * 0
// would be NaN (the maximum takes the number).
__device__ __forceinline__ double rsqrt_n(double a)
{
    const double r = __builtin_amdgcn_rsq(a);  // relative error < 2^-22
    const double e = fmax(fma(-(a * r), r, 1.0), -1.0);
    return fma(r * e, fma(0.375, e, 0.5), r);
}

// Lane roles and the steps across the lanes of an element.
struct Quad {
    int n, q;  // element of the wave, lane of the element
    // this lane's matrix entries (row i = lane & 3, column k = q) with
    // w(a, b) = WHI if a = b else WLO and s = -1 / +1: NN[i][k] = w(ix,kx) w(iy,ky),
    // its own transpose; DX[i][k] = s_kx w(iy,ky) and DY[i][k] = s_ky w(ix,kx) from
    // corners to Gauss points; DX^T and DY^T
    double nn, dx, dy, dxt, dyt;
    __device__ __forceinline__ explicit Quad(int lane)
    {
        n = lane & 15;
        q = lane >> 4;
        const int i = lane & 3, k = q;
        const double wx = ((i ^ k) & 1) ? WLO : WHI, wy = ((i ^ k) & 2) ? WLO : WHI;
        nn = wx * wy;
        dx = (k & 1) ? wy : -wy;
        dy = (k & 2) ? wx : -wx;
        dxt = (i & 1) ? wy : -wy;
        dyt = (i & 2) ? wx : -wx;
    }
    __device__ __forceinline__ static double mm(double a, double b, double c)
    {
        return __builtin_amdgcn_mfma_f64_4x4x4f64(a, b, c, 0, 0, 0);
    }
    // value, h d/dx, h d/dy at this lane's Gauss point of the lanes' corner values
    __device__ __forceinline__ void interp(double v, double &n_, double &x, double &y) const
    {
        n_ = mm(nn, v, 0.0);
        x = mm(dx, v, 0.0);
        y = mm(dy, v, 0.0);
    }
    __device__ __forceinline__ double interp_n(double v) const { return mm(nn, v, 0.0); }
    // a sixteenth of the sum over the element's lanes
    __device__ __forceinline__ double sum16(double v) const { return mm(0.0625, v, 0.0); }
    // corner rows of the Gauss-point terms c, x, y (factors of N, h dN/dx, h dN/dy)
    __device__ __forceinline__ double rows(double c, double x, double y) const
    {
        return mm(dyt, y, mm(dxt, x, mm(nn, c, 0.0)));
    }
};

// A node plane's fields at this lane's x-y Gauss point: value, h d/dx, h d/dy.
struct Plane {
    double n[NF], x[NF], y[NF];
};

// Element scalars of one operator evaluation, scaled by h as above.
struct ElemMat {
    double alpha, Kc, s, tau, tauT, dtau, dtauT;
};

// Physical constants of the Gauss-point arithmetic.
struct PhysC {
    double Pr, Beg[3];
    __device__ __forceinline__ explicit PhysC(const Geo &g)
    {
        Pr = g.Pr / g.h;
#pragma unroll
        for (int i = 0; i < 3; ++i) Beg[i] = g.B * g.eg[i] * g.h;
    }
};

// Gauss-point terms: C[f] = {c, Cx, Cy, Cz}, the factors of N_a and of the three
// components of h grad N_a in row f of the element.  V: {value, h d/dx, h d/dy,
// h d/dz} of u, v, w, p, T.
__device__ __forceinline__ void point_residual(const PhysC &c, const ElemMat &m,
                                               const double V[NF][4], double C[NF][4])
{
    const double u[3] = {V[0][0], V[1][0], V[2][0]};
    double rM[3];
#pragma unroll
    for (int i = 0; i < 3; ++i) {
        double gal = fma(m.alpha, u[i], c.Beg[i] * V[4][0]);
#pragma unroll
        for (int d = 0; d < 3; ++d) gal = fma(u[d], V[i][1 + d], gal);
        C[i][0] = gal;
        rM[i] = gal + V[3][1 + i];
    }
    double rT = -m.s;
#pragma unroll
    for (int d = 0; d < 3; ++d) rT = fma(u[d], V[4][1 + d], rT);
#pragma unroll
    for (int i = 0; i < 3; ++i) {
        const double tr = m.tau * rM[i];
        C[3][1 + i] = tr;
#pragma unroll
        for (int d = 0; d < 3; ++d) C[i][1 + d] = fma(c.Pr, V[i][1 + d] + V[d][1 + i], u[d] * tr);
        C[i][1 + i] -= V[3][0];
    }
    C[3][0] = V[0][1] + V[1][2] + V[2][3];
    const double trT = m.tauT * rT;
    C[4][0] = rT;
#pragma unroll
    for (int d = 0; d < 3; ++d) C[4][1 + d] = fma(m.Kc, V[4][1 + d], u[d] * trT);
}

// As above for the directional derivative along the direction with field values
// D (exact linearisation: dtau and dtauT are the variations of tau and tauT).
__device__ __forceinline__ void point_jv(const PhysC &c, const ElemMat &m, const double V[NF][4],
                                         const double D[NF][4], double C[NF][4])
{
    const double u[3] = {V[0][0], V[1][0], V[2][0]}, du[3] = {D[0][0], D[1][0], D[2][0]};
    double A[3], Bm[3];
#pragma unroll
    for (int i = 0; i < 3; ++i) {
        double rM = fma(m.alpha, u[i], fma(c.Beg[i], V[4][0], V[3][1 + i]));
        double dg = fma(m.alpha, du[i], c.Beg[i] * D[4][0]);
#pragma unroll
        for (int d = 0; d < 3; ++d) {
            rM = fma(u[d], V[i][1 + d], rM);
            dg = fma(du[d], V[i][1 + d], fma(u[d], D[i][1 + d], dg));
        }
        C[i][0] = dg;
        A[i] = fma(m.dtau, rM, m.tau * (dg + D[3][1 + i]));
        Bm[i] = m.tau * rM;
    }
    double rT = -m.s, drT = 0.0;
#pragma unroll
    for (int d = 0; d < 3; ++d) {
        rT = fma(u[d], V[4][1 + d], rT);
        drT = fma(du[d], V[4][1 + d], fma(u[d], D[4][1 + d], drT));
    }
#pragma unroll
    for (int i = 0; i < 3; ++i) {
#pragma unroll
        for (int d = 0; d < 3; ++d)
            C[i][1 + d] = fma(c.Pr, D[i][1 + d] + D[d][1 + i], fma(u[d], A[i], du[d] * Bm[i]));
        C[i][1 + i] -= D[3][0];
        C[3][1 + i] = A[i];
    }
    C[3][0] = D[0][1] + D[1][2] + D[2][3];
    const double AT = fma(m.dtauT, rT, m.tauT * drT), BT = m.tauT * rT;
    C[4][0] = drT;
#pragma unroll
    for (int d = 0; d < 3; ++d)
        C[4][1 + d] = fma(m.Kc, D[4][1 + d], fma(u[d], AT, du[d] * BT));
}

// As above for the transposed product in one reverse pass: L holds the adjoint
// test fields (Lambda on the velocity rows, Pi on the pressure row, Theta on the
// temperature row).  The multipliers of the varied strong residuals are
// tau (u . grad Lambda + grad Pi) and tauT u . grad Theta; A and AT sum what the
// variations of tau and tauT with the element velocity multiply.
__device__ __forceinline__ void point_jtv(const PhysC &c, const ElemMat &m, const double V[NF][4],
                                          const double L[NF][4], double C[NF][4], double &A, double &AT)
{
    const double u[3] = {V[0][0], V[1][0], V[2][0]};
    double rM[3], LM[3];
#pragma unroll
    for (int i = 0; i < 3; ++i) {
        double r = fma(m.alpha, u[i], fma(c.Beg[i], V[4][0], V[3][1 + i]));
        double q = L[3][1 + i];
#pragma unroll
        for (int d = 0; d < 3; ++d) {
            r = fma(u[d], V[i][1 + d], r);
            q = fma(u[d], L[i][1 + d], q);
        }
        rM[i] = r;
        A = fma(q, r, A);
        C[3][1 + i] = m.tau * q;
        LM[i] = fma(m.tau, q, L[i][0]);
    }
    double rT = -m.s, uTh = 0.0;
#pragma unroll
    for (int d = 0; d < 3; ++d) {
        rT = fma(u[d], V[4][1 + d], rT);
        uTh = fma(u[d], L[4][1 + d], uTh);
    }
    AT = fma(uTh, rT, AT);
    const double ThM = fma(m.tauT, uTh, L[4][0]), trT = m.tauT * rT;
#pragma unroll
    for (int j = 0; j < 3; ++j) {
        double cj = fma(m.alpha, LM[j], fma(trT, L[4][1 + j], ThM * V[4][1 + j]));
        double t = 0.0;
#pragma unroll
        for (int i = 0; i < 3; ++i) {
            cj = fma(LM[i], V[i][1 + j], cj);
            t = fma(L[i][1 + j], rM[i], t);
        }
        C[j][0] = fma(m.tau, t, cj);
#pragma unroll
        for (int d = 0; d < 3; ++d) C[j][1 + d] = fma(LM[j], u[d], c.Pr * (L[j][1 + d] + L[d][1 + j]));
        C[j][1 + j] += L[3][0];
    }
    C[3][0] = -(L[0][1] + L[1][2] + L[2][3]);
    C[4][0] = fma(c.Beg[0], LM[0], fma(c.Beg[1], LM[1], c.Beg[2] * LM[2]));
#pragma unroll
    for (int d = 0; d < 3; ++d) C[4][1 + d] = fma(m.Kc, L[4][1 + d], ThM * u[d]);
}

// Rows of a layer's lower and upper node plane at this lane's corner.  Each Gauss
// point is transposed as it comes (four products per row), which frees its twenty
// terms; its rows join both planes with the z weights WHI / WLO (point z = 0:
// lower) and -1 / +1 (Cz).  hi carries to the layer above as its lo.
struct TestAcc {
    double lo[NF], hi[NF] = {0.0, 0.0, 0.0, 0.0, 0.0};
    __device__ __forceinline__ void point(const Quad &qd, int z, const double C[NF][4])
    {
#pragma unroll
        for (int f = 0; f < NF; ++f) {
            const double p = qd.rows(C[f][0], C[f][1], C[f][2]), q = qd.interp_n(C[f][3]);
            lo[f] = fma(z ? WLO : WHI, p, z ? lo[f] : hi[f]) - q;
            hi[f] = z ? fma(WHI, p, hi[f]) + q : fma(WLO, p, q);
        }
    }
};

constexpr int PEL = TX * TY;  // elements of a layer (64: 16 per wave)
// Parked rows of one corner: rows of 8 elements at pitch 9 with a row of zeros
// before and after and a column of zeros between, so that a node on the tile's
// rim adds zeros instead of testing which elements it has; the arrays of two
// corners start 32 banks apart.
constexpr int PROW = BX * NF;
constexpr int PQ = 464;
constexpr int NIT = (PVAL + NTHR - 1) / NTHR;
static_assert(TX == 8 && PEL == 16 * (NTHR / 64), "a wave's 16 elements are two rows of a layer");
static_assert((TY + 2) * PROW + NF <= PQ, "parked rows and their rim fit");

template <int NV>
struct LayerLds {
    double x[2][NV][PVAL];      // node planes (x, direction), ring of two
    double p[2][4 * PQ];        // element rows of a node plane, ring of two
    double mat[2][3][2 * PEL];  // alpha', K', s' of two layers' elements, ring of two
};

// One workgroup marches through its tile's layers of 8x8 elements.  Thread t
// stages and finishes the values t and t + 256 of a node plane (node-major, so
// loads and stores are contiguous); a wave evaluates two rows of elements.  One
// set of element rows per node plane is parked in LDS, where the (up to) four
// element columns around a node are added in a fixed order.
// One barrier per layer: planes, parked rows and material alternate between two
// buffers, and a buffer is written again only after the barrier that follows its
// last reader.  Tv: the direction's storage type, widened as it is staged.
template <int OP, typename Tv>
__device__ __forceinline__ void elem_tile(const Geo &g, const double *__restrict__ x,
                                          const Tv *__restrict__ v,
                                          const double *__restrict__ gamma,
                                          const double *__restrict__ src,
                                          const uint8_t *__restrict__ nmask,
                                          double *__restrict__ out, double *__restrict__ slots,
                                          int blk, int nblk)
{
    constexpr bool DIR = OP != OP_RES;
    constexpr int NV = DIR ? 2 : 1;
    __shared__ LayerLds<NV> S;
    const int tile = xcd_tile(blk, nblk);
    const int btx = tile % g.ntx, rt = tile / g.ntx, bty = rt % g.nty, btz = rt / g.nty;
    const int tx0 = btx * TX, ty0 = bty * TY, k0 = btz * g.etz;
    const int nl = min(g.etz, g.nz - k0);  // layers
    const int tid = (int)threadIdx.x;
    const double wrow = 0.125 * g.h * g.h;

    // this thread's two values of a node plane
    const int64_t ps = (int64_t)(g.nx + 1) * (g.ny + 1);
    const int64_t n00 = gnode(g, tx0, ty0, k0);
    unsigned noff[NIT], voff[NIT];  // node and value offset in the plane (0: outside the grid)
    int pa[NIT];
    unsigned hist[NIT];  // whether the value is prescribed, one bit per staged plane
    bool in[NIT], sh[NIT];
#pragma unroll
    for (int it = 0; it < NIT; ++it) {
        const int idx = tid + it * NTHR;
        const int nb = idx / NF, f = idx - nb * NF, lx = nb % BX, ly = nb / BX;
        const int I = tx0 + lx, J = ty0 + ly;
        in[it] = idx < PVAL && I <= g.nx && J <= g.ny;
        sh[it] = shared_dir(lx, I, g.nx, TX) || shared_dir(ly, J, g.ny, TY);
        noff[it] = in[it] ? (unsigned)lx + (unsigned)(g.nx + 1) * (unsigned)ly : 0u;
        voff[it] = NF * noff[it] + f;
        hist[it] = 0;
        pa[it] = in[it] ? ly * PROW + lx * NF + f : 0;
    }
    struct Regs {
        double x[NIT], v[NIT];
        unsigned m[NIT];
    };
    auto load_plane = [&](int p, Regs &r) {
        const int64_t nb = n00 + p * ps;
        const double *xp = x + NF * nb;
        const Tv *vp = DIR ? v + NF * nb : nullptr;
        const uint8_t *mp = nmask + nb;
#pragma unroll
        for (int it = 0; it < NIT; ++it) {
            r.x[it] = xp[voff[it]];
            r.v[it] = DIR ? (double)vp[voff[it]] : 0.0;
            r.m[it] = mp[noff[it]];
        }
    };
    auto store_plane = [&](int b, const Regs &r) {
#pragma unroll
        for (int it = 0; it < NIT; ++it) {
            const int idx = tid + it * NTHR;
            const unsigned fixed = (r.m[it] >> (voff[it] - NF * noff[it])) & 1u;
            hist[it] = (hist[it] << 1) | fixed;
            if (idx < PVAL) {
                S.x[b][0][idx] = in[it] ? r.x[it] : 0.0;
                if (DIR) S.x[b][NV - 1][idx] = (in[it] && !fixed) ? r.v[it] : 0.0;
            }
        }
    };
    // material (Eqs. conducint, alphaint) of the elements of layers 2 c and 2 c + 1,
    // one per thread of the first half
    struct MatRegs {
        bool in;
        double y, s;
    };
    auto load_mat = [&](int c) {
        const int i = tx0 + tid % TX, j = ty0 + (tid / TX) % TY, k = k0 + 2 * c + tid / PEL;
        MatRegs r;
        r.in = tid < 2 * PEL && i < g.nx && j < g.ny && k < k0 + nl;
        const int64_t e = r.in ? (int64_t)i + (int64_t)g.nx * ((int64_t)j + (int64_t)g.ny * k) : 0;
        r.y = gamma[e];
        r.s = src[e];
        return r;
    };
    auto store_mat = [&](int c, const MatRegs &r) {
        if (tid < 2 * PEL) {
            S.mat[c & 1][0][tid] = r.in ? alpha_of(g, r.y) * g.h : 0.0;
            S.mat[c & 1][1][tid] = r.in ? K_of(g, r.y) / g.h : 1.0;
            S.mat[c & 1][2][tid] = r.in ? r.s * g.h : 0.0;
        }
    };
    // add the parked rows of plane p and write its values; back: planes staged since
    auto finish_plane = [&](int p, int back) {
        const double *P = S.p[p & 1];
        const int64_t nb = n00 + p * ps;
        const bool shz = (p == 0 && k0 > 0) || (p == nl && k0 + nl < g.nz);
        double *op = out + NF * nb, *sp = slots + tile * eslot_tile(g.etz) + p * PVAL;
#pragma unroll
        for (int it = 0; it < NIT; ++it) {
            // elements (-1, -1), (0, -1), (-1, 0), (0, 0) around the node; the
            // parked row of element (ex, ey) is at (ey + 1, ex + 1) of its corner's array
            const double *Pn = P + pa[it];
            double val = wrow * ((Pn[3 * PQ] + Pn[2 * PQ + NF]) +
                                 (Pn[1 * PQ + PROW] + Pn[0 * PQ + PROW + NF]));
            if (!in[it]) continue;
            if (sh[it] || shz) {
                sp[tid + it * NTHR] = val;
            } else {
                if ((hist[it] >> back) & 1)
                    val = OP == OP_RES ? 0.0 : (double)(v + NF * nb)[voff[it]];
                op[voff[it]] = val;
            }
        }
    };

    Regs r0, r1;
    load_plane(0, r0);
    load_plane(1, r1);
    const MatRegs m0 = load_mat(0);
    for (int e = tid; e < 2 * 4 * PQ; e += NTHR) (&S.p[0][0])[e] = 0.0;
    store_mat(0, m0);
    store_plane(0, r0);
    store_plane(1, r1);
    __syncthreads();

    // this lane's element column, Gauss point and corner
    const Quad qd(tid & 63);
    const int el = 16 * (tid >> 6) + qd.n, li = el % TX, lj = el / TX;
    const bool valid = tx0 + li < g.nx && ty0 + lj < g.ny;
    const int cn = NF * (li + (qd.q & 1) + BX * (lj + (qd.q >> 1)));  // this lane's corner
    const int park = qd.q * PQ + (lj + 1) * PROW + (li + 1) * NF;
    const PhysC ph(g);
    const double pr2 = 16.0 * (g.Pr / g.h) * (g.Pr / g.h);

    // Lower plane of the state, the direction's values of the lower plane at this
    // lane's corner and |u|^2 and u . du there; J^T w: u there
    Plane xl;
    double wl[NF], ul[3] = {0.0, 0.0, 0.0}, U2l, dl;
    auto plane = [&](int b, Plane &o) {
        const double *p = &S.x[b][0][cn];
#pragma unroll
        for (int f = 0; f < NF; ++f) qd.interp(p[f], o.n[f], o.x[f], o.y[f]);
    };
    auto corner = [&](int b, double w[NF], double &U2, double &du) {
        U2 = du = 0.0;
#pragma unroll
        for (int f = 0; f < NF; ++f) w[f] = DIR ? S.x[b][NV - 1][cn + f] : 0.0;
#pragma unroll
        for (int i = 0; i < 3; ++i) {
            const double u = S.x[b][0][cn + i];
            U2 = fma(u, u, U2);
            if (OP == OP_JV) du = fma(u, w[i], du);
        }
    };
    plane(0, xl);
    corner(0, wl, U2l, dl);
    if (OP == OP_JTV) {
#pragma unroll
        for (int i = 0; i < 3; ++i) ul[i] = S.x[0][0][cn + i];
    }
    TestAcc acc;
    __syncthreads();

#pragma unroll 1
    for (int l = 0; l < nl; ++l) {
        const bool more = l + 2 <= nl;
        Regs r = {};
        const bool mat = (l & 1) == 0 && l + 2 < nl;  // material of the next two layers
        MatRegs mr = {};
        const int b = (l + 1) & 1;
        double wh[NF], U2h, dh;
        corner(b, wh, U2h, dh);
        ElemMat m;
        const int mb = (l >> 1) & 1, me = PEL * (l & 1) + el;
        m.alpha = S.mat[mb][0][me];
        m.Kc = S.mat[mb][1][me];
        m.s = S.mat[mb][2][me];
        const double U2 = qd.sum16(U2l + U2h);
        m.tau = rsqrt_n(fma(m.alpha, m.alpha, U2 + pr2));
        m.tauT = rsqrt_n(fma(16.0 * m.Kc, m.Kc, U2));
        m.dtau = m.dtauT = 0.0;
        if (OP == OP_JV) {
            const double du = qd.sum16(dl + dh);
            m.dtau = -(m.tau * m.tau * m.tau) * du;
            m.dtauT = -(m.tauT * m.tauT * m.tauT) * du;
        }
        Plane xh;
        plane(b, xh);
        __builtin_amdgcn_sched_barrier(0);
        double wz3[NF];  // h d/dz of the direction
        if (DIR) {
#pragma unroll
            for (int f = 0; f < NF; ++f) wz3[f] = qd.interp_n(wh[f] - wl[f]);
        }
        double A = 0.0, AT = 0.0;
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int z = 0; z < 2; ++z) {
            const double wz = z ? WHI : WLO;
            double V[NF][4], D[NF][4], C[NF][4];
#pragma unroll
            for (int f = 0; f < NF; ++f) {
                V[f][3] = xh.n[f] - xl.n[f];
                V[f][0] = fma(wz, V[f][3], xl.n[f]);
                V[f][1] = fma(wz, xh.x[f] - xl.x[f], xl.x[f]);
                V[f][2] = fma(wz, xh.y[f] - xl.y[f], xl.y[f]);
                if (DIR) {
                    qd.interp(fma(wz, wh[f] - wl[f], wl[f]), D[f][0], D[f][1], D[f][2]);
                    D[f][3] = wz3[f];
                }
            }
            if (OP == OP_RES)
                point_residual(ph, m, V, C);
            else if (OP == OP_JV)
                point_jv(ph, m, V, D, C);
            else
                point_jtv(ph, m, V, D, C, A, AT);
            acc.point(qd, z, C);
            __builtin_amdgcn_sched_barrier(0);
            if (z == 0) {
                // the second point forms its differences anew: kept from the first,
                // they would take 30 registers more than there are
#pragma unroll
                for (int f = 0; f < NF; ++f) {
                    asm volatile("" : "+v"(xl.n[f]), "+v"(xl.x[f]), "+v"(xl.y[f]));
                    asm volatile("" : "+v"(xh.n[f]), "+v"(xh.x[f]), "+v"(xh.y[f]));
                }
                asm volatile("" ::: "memory");
                if (more) load_plane(l + 2, r);
                if (mat) mr = load_mat((l >> 1) + 1);
            }
        }
        double coef = 0.0;
        if (OP == OP_JTV)  // variations of tau and tauT with the element velocity
            coef = -(m.tau * m.tau * m.tau * qd.sum16(A) + m.tauT * m.tauT * m.tauT * qd.sum16(AT));
#pragma unroll
        for (int f = 0; f < NF; ++f) {
            double lo = acc.lo[f];
            if (OP == OP_JTV && f < 3) {
                lo = fma(coef, ul[f], lo);
                acc.hi[f] = fma(coef, S.x[b][0][cn + f], acc.hi[f]);
            }
            S.p[l & 1][park + f] = valid ? lo : 0.0;
        }
        xl = xh;
        U2l = U2h;
        dl = dh;
        if (OP == OP_JTV) {
#pragma unroll
            for (int i = 0; i < 3; ++i) ul[i] = S.x[b][0][cn + i];
        }
        if (DIR) {
#pragma unroll
            for (int f = 0; f < NF; ++f) wl[f] = wh[f];
        }
        if (more) store_plane(l & 1, r);
        if (mat) store_mat((l >> 1) + 1, mr);
        __syncthreads();
        finish_plane(l, more ? 2 : 1);
    }
#pragma unroll
    for (int f = 0; f < NF; ++f) S.p[nl & 1][park + f] = valid ? acc.hi[f] : 0.0;
    __syncthreads();
    finish_plane(nl, 0);
}

template <int OP, typename Tv>
__global__ __launch_bounds__(NTHR, 2) void k_elem64(Geo g, const double *__restrict__ x,
                                                    const Tv *__restrict__ v,
                                                    const double *__restrict__ gamma,
                                                    const double *__restrict__ src,
                                                    const uint8_t *__restrict__ nmask,
                                                    double *__restrict__ out,
                                                    double *__restrict__ slots)
{
    elem_tile<OP, Tv>(g, x, v, gamma, src, nmask, out, slots, (int)blockIdx.x, (int)gridDim.x);
}

// ---- batched launches: the same body over a table of problems ---------------------

__global__ __launch_bounds__(NTHR, 2) void kb_elem64_jv(const BElem<double, double> *__restrict__ tab,
                                                        const int *__restrict__ off, int n)
{
    const int e = batch_entry(off, n);
    const BElem<double, double> &a = tab[e];
    const int b0 = off[e];
    elem_tile<OP_JV, double>(a.g, a.x, a.v, a.gamma, a.s, a.nmask, a.out, a.slots,
                             (int)blockIdx.x - b0, off[e + 1] - b0);
}

__global__ __launch_bounds__(NTHR, 2) void kb_elem64_smooth(const BElemSmooth<double> *__restrict__ tab,
                                                            const int *__restrict__ off, int n)
{
    const int e = batch_entry(off, n);
    const BElemSmooth<double> &a = tab[e];
    const int b0 = off[e];
    elem_tile<OP_JV, double>(a.g, a.xs, (const double *)a.x, a.gamma, a.s, a.nmask, a.t, a.slots,
                             (int)blockIdx.x - b0, off[e + 1] - b0);
}

template <int OP, typename Tv>
void launch(const Geo &g, const double *x, const Tv *v, const double *gamma, const double *s,
            const uint8_t *nmask, double *out, double *slots, hipStream_t st)
{
    hipLaunchKernelGGL((k_elem64<OP, Tv>), dim3((unsigned)n_etiles(g)), dim3(NTHR), 0, st, g, x, v,
                       gamma, s, nmask, out, slots);
}

}  // namespace

template <typename Tv>
hipError_t launch_elem64_pass(ElemOp op, const Geo &g, const double *x, const Tv *v,
                              const double *gamma, const double *s, const uint8_t *nmask,
                              double *out, double *slots, hipStream_t st)
{
    switch (op) {
    case OP_RES:
        // (no direction: the shared-node pass is asked for the state's type)
        if constexpr (sizeof(Tv) == sizeof(double)) {
            launch<OP_RES, Tv>(g, x, v, gamma, s, nmask, out, slots, st);
            break;
        }
        return hipErrorInvalidValue;
    case OP_JV: launch<OP_JV, Tv>(g, x, v, gamma, s, nmask, out, slots, st); break;
    case OP_JTV: launch<OP_JTV, Tv>(g, x, v, gamma, s, nmask, out, slots, st); break;
    }
    return hipGetLastError();
}
template hipError_t launch_elem64_pass<double>(ElemOp, const Geo &, const double *, const double *,
                                               const double *, const double *, const uint8_t *,
                                               double *, double *, hipStream_t);
template hipError_t launch_elem64_pass<float>(ElemOp, const Geo &, const double *, const float *,
                                              const double *, const double *, const uint8_t *,
                                              double *, double *, hipStream_t);

template <>
hipError_t blaunch_elem_jv<double, double>(const BLaunch &L, hipStream_t st)
{
    if (L.blocks <= 0) return hipSuccess;
    hipLaunchKernelGGL(kb_elem64_jv, dim3((unsigned)L.blocks), dim3(NTHR), 0, st,
                       (const BElem<double, double> *)L.tab, L.off, L.n);
    return hipGetLastError();
}

template <>
hipError_t blaunch_elem_smooth_pass<double>(const BLaunch &L, hipStream_t st)
{
    if (L.blocks <= 0) return hipSuccess;
    hipLaunchKernelGGL(kb_elem64_smooth, dim3((unsigned)L.blocks), dim3(NTHR), 0, st,
                       (const BElemSmooth<double> *)L.tab, L.off, L.n);
    return hipGetLastError();
}

}  // namespace fe
