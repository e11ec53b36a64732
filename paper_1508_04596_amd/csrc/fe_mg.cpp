// Matrix-free geometric multigrid preconditioner (host side).
//
// The paper preconditions flexible GMRES with geometric multigrid (Sec.
// "Solving the linear systems").  Here every level is a rediscretisation of the
// same stabilised operator on a grid with half the elements per direction:
// the design and source are averaged over the eight child elements, the
// linearisation state is injected from the coincident fine nodes, and the
// element kernels of the fine level evaluate J v on every level.  Smoothing is
// damped nodal block-Jacobi; small levels apply their operator as an assembled
// 27-point block stencil (from element Jacobians, once per Newton step), since
// the element pass costs the same latency however few tiles a grid has.  The
// coarsest level is solved directly: its Jacobian is assembled from 135
// probing products (one per (node colour mod 3^3, field)), condensed to the
// DOFs that are not prescribed (prescribed rows are identity rows and
// prescribed columns are zero, so they drop out exactly), factorised by band
// LU on the host, and inverted explicitly on the GPU from the factors, so that
// each V-cycle's coarse solve is one matrix-vector product on the device.
// V-cycles run in FP64, or in FP32 when the Krylov operator is FP32.
#include <algorithm>
#include <cmath>
#include <cstdio>
#include <cstring>
#include <vector>

#include "fe_band_lu.h"
#include "fe_internal.h"
#include "fe_mg.h"

namespace fe {

hipError_t mg_coarsen_elem(const fe_grid &c, const fe_grid &f, const double *fv, double *cv,
                          hipStream_t st);
hipError_t mg_inject_state(const fe_grid &c, const fe_grid &f, const double *fv, double *cv,
                           hipStream_t st);
hipError_t mg_inject_mask(const fe_grid &c, const fe_grid &f, const uint8_t *fv, uint8_t *cv,
                          hipStream_t st);
template <typename T>
hipError_t mg_restrict_smooth(const fe_grid &c, const fe_grid &f, const T *b, const T *t,
                              const uint8_t *cmask, T *bc, const T *Dc, T *xc, T omega,
                              bool transpose, hipStream_t st);
template <typename T>
hipError_t mg_prolong_add(const fe_grid &f, const fe_grid &c, const T *xc, const uint8_t *fmask,
                          T *x, hipStream_t st);
template <typename T>
hipError_t mg_smooth(const T *D, const T *b, const T *t, T *x, int64_t nn, T omega, bool transpose,
                     bool accumulate, hipStream_t st);
template <typename T>
hipError_t mg_stencil_apply(int nx, int ny, int nz, const T *S, const T *v, T *out, bool transpose,
                            hipStream_t st);
hipError_t mg_stencil_diag(int64_t nn, const double *S, double *D, hipStream_t st);
hipError_t mg_coarse_inverse(int n, int kl, int ku, const double *Lc, const double *Uc,
                             const double *Ud, const int *piv, double *X, hipStream_t st);
template <typename T>
hipError_t mg_restrict_coarse(const fe_grid &c, const fe_grid &f, int n, const double *X,
                              const int *fidx, const T *b, const T *t, double *P, bool transpose,
                              hipStream_t st);
template <typename T>
hipError_t mg_coarse_sum(int nfull, int n, const int *pos, const double *P, T *x, hipStream_t st);
template <typename T>
hipError_t mg_sweep_first(int nx, int ny, int nz, const T *S, const T *D, const T *b,
                          const double *v, T *bout, T *xout, T omega, bool transpose, hipStream_t st);
template <typename T>
hipError_t mg_sweep_prolong(const fe_grid &f, const fe_grid &c, const T *S, const T *D, const T *b,
                            const T *x, const T *xc, const uint8_t *fmask, T *xout, T omega,
                            bool transpose, hipStream_t st);
bool mg_sweep_coarse_pays(int nfull, int n);
template <typename T>
hipError_t mg_sweep_coarse(const fe_grid &f, const fe_grid &c, const T *S, const T *D, const T *b,
                           const T *x, int nfull, int n, const int *pos, const double *P,
                           const uint8_t *fmask, T *xout, T omega, bool transpose, hipStream_t st);
template <typename T>
hipError_t mg_stencil_smooth(int nx, int ny, int nz, const T *S, const T *D, const T *b, const T *xin,
                             T *xout, T omega, bool transpose, hipStream_t st);
hipError_t mg_smooth0_cast(const float *D, const double *v, float *b32, float *x, int64_t nn,
                           float omega, bool transpose, hipStream_t st);
template <typename T>
hipError_t mg_copy(const T *a, T *b, int64_t n, hipStream_t st);

constexpr int64_t MG_MAX_COARSE_DOF = 2400;   // largest directly factored level
constexpr int64_t MG_TARGET_COARSE_DOF = 1500; // stop coarsening below this size

static void free_level(fe_problem *p, MgLevel &L, bool owned)
{
    if (owned) {
        dfree(p, L.nmask);
        dfree(p, L.gamma);
        dfree(p, L.s);
        dfree(p, L.x);
        dfree(p, L.x32);
        dfree(p, L.D);
        dfree(p, L.D32);
        dfree(p, L.slots);
        dfree(p, L.slots25);
    }
    dfree(p, L.S);
    dfree(p, L.S32);
    dfree(p, L.xa);
    dfree(p, L.xa32);
    dfree(p, L.b);
    dfree(p, L.xs);
    dfree(p, L.t);
    dfree(p, L.b32);
    dfree(p, L.xs32);
    dfree(p, L.t32);
}

void mg_free(Mg *mg)
{
    if (!mg) return;
    fe_problem *p = mg->owner;
    for (size_t l = 0; l < mg->lev.size(); ++l) free_level(p, mg->lev[l], l > 0);
    dfree(p, mg->probe);
    dfree(p, mg->probe_out);
    dfree(p, mg->dfac);
    dfree(p, mg->dpiv);
    dfree(p, mg->dmap);
    dfree(p, mg->Xinv);
    dfree(p, mg->cpart);
    hfree(p, mg->hbuf);
    hfree(p, mg->hfac);
    hfree(p, mg->hpiv);
    hfree(p, mg->hmask);
    hfree(p, mg->hmap);
    if (mg->probe_ready) (void)hipEventDestroy(mg->probe_ready);
    delete mg;
}

int64_t mg_asm_nodes(int opt) { return opt < 0 ? MG_ASM_NODES_DEFAULT : (int64_t)opt; }

// Next coarser grid: elements of twice the edge, ceil(n / 2) per direction.  An
// odd fine count leaves the last coarse layer half outside the fine grid; its
// nodes past the end take their values from the fine boundary nodes.
static fe_grid coarser(fe_grid g)
{
    g.nx = (g.nx + 1) / 2;
    g.ny = (g.ny + 1) / 2;
    g.nz = (g.nz + 1) / 2;
    g.h *= 2.0;
    return g;
}

// Levels while the coarse grids stay nested (every count even) or, with pad,
// also through odd counts; 0 when that gives no usable hierarchy.
static int count_levels(fe_grid g, bool pad)
{
    int n = 1;
    while (true) {
        const int64_t ndof = (int64_t)NF * (g.nx + 1) * (g.ny + 1) * (g.nz + 1);
        if (ndof <= MG_TARGET_COARSE_DOF) break;
        if (g.nx < 4 || g.ny < 4 || g.nz < 4) break;
        if (!pad && (g.nx % 2 || g.ny % 2 || g.nz % 2)) break;
        g = coarser(g);
        ++n;
    }
    const int64_t ndof = (int64_t)NF * (g.nx + 1) * (g.ny + 1) * (g.nz + 1);
    if (n < 2 || ndof > MG_MAX_COARSE_DOF) return 0;
    return n;
}

// Nested levels where they give a hierarchy; otherwise (odd counts before the
// coarse problem is small enough) padded ones.
int mg_num_levels(const fe_grid &g)
{
    const int n = count_levels(g, false);
    return n ? n : count_levels(g, true);
}

static int64_t r256(int64_t b) { return (b + 255) / 256 * 256; }

// Half bandwidth of the coarsest matrix in lexicographic node order, NF DOF per node.
static int64_t coarse_band(const fe_grid &c)
{
    return NF * (1 + (c.nx + 1) + (int64_t)(c.nx + 1) * (c.ny + 1)) + NF - 1;
}

// Device bytes mg_create allocates for grid g (each allocation rounded up to 256 B).
int64_t mg_footprint_bytes(const fe_grid &g0, bool mixed, int64_t asm_nodes)
{
    const int nl = mg_num_levels(g0);
    if (nl < 2) return 0;
    fe_grid g = g0;
    int64_t b = 0, ndof_c = 0, ne_c = 0, ne_je = 0;
    for (int l = 0; l < nl; ++l) {
        if (l > 0) g = coarser(g);
        const int64_t nn = (int64_t)(g.nx + 1) * (g.ny + 1) * (g.nz + 1), ndof = NF * nn;
        const int64_t ne = (int64_t)g.nx * g.ny * g.nz;
        const int64_t nt = (int64_t)((g.nx + TX - 1) / TX) * ((g.ny + TY - 1) / TY) * ((g.nz + TZ - 1) / TZ);
        if (l > 0) {
            b += r256(nn) + 2 * r256(8 * ne) + r256(8 * ndof) + r256(8 * 25 * nn);
            b += r256(n_slots(g) * 8) + r256(nt * BOXN * 25 * 8);
            b += 2 * r256(8 * ndof);
            if (mixed) b += r256(4 * ndof) + r256(4 * 25 * nn) + 2 * r256(4 * ndof);
        } else if (mixed) {
            b += r256(4 * ndof);
        }
        b += r256(8 * ndof);
        if (mixed) b += r256(4 * ndof);
        if (l < nl - 1 && nn <= asm_nodes) {
            b += r256(8 * 675 * nn) + r256(8 * ndof);
            if (mixed) b += r256(4 * 675 * nn) + r256(4 * ndof);
            ne_je = std::max(ne_je, ne);
        }
        ndof_c = ndof;
        ne_c = ne;
    }
    b += r256(8 * 1600 * std::max(ne_c, ne_je)) + r256(8 * 135 * ndof_c);
    const int64_t bw = coarse_band(g);
    b += r256(8 * ndof_c * (3 * bw + 1)) + r256(4 * ndof_c) + r256(8 * ndof_c) + r256(8 * ndof_c * ndof_c);
    b += r256(8 * ((ndof_c + 63) / 64) * ndof_c);
    return b;
}

// Allocate the hierarchy for problem p (levels >= 1 own their data).
int mg_create(fe_problem *p, bool mixed, int64_t asm_nodes, Mg **out)
{
    *out = nullptr;
    const int nl = mg_num_levels(p->grid);
    if (nl < 2) {
        set_error("multigrid: the grid cannot be coarsened to a directly solvable level "
                  "(element counts must halve evenly down to <= 2400 coarse DOF)");
        return FE_EINVAL;
    }
    Mg *mg = new Mg();
    mg->owner = p;
    mg->mixed = mixed;
    mg->asm_nodes = asm_nodes;
    mg->lev.resize(nl);
    hipError_t e = hipSuccess;
    fe_grid g = p->grid;
    for (int l = 0; l < nl; ++l) {
        MgLevel &L = mg->lev[l];
        if (l > 0) g = coarser(g);
        L.grid = g;
        L.geo = make_geo(g, p->phys);
        L.nn = n_nodes(L.geo);
        L.ne = n_elem(L.geo);
        L.ndof = NF * L.nn;
        const size_t nb = sizeof(double) * L.ndof;
        if (l > 0) {
            if (e == hipSuccess) e = dalloc(p, &L.nmask, L.nn);
            if (e == hipSuccess) e = dalloc(p, &L.gamma, sizeof(double) * L.ne);
            if (e == hipSuccess) e = dalloc(p, &L.s, sizeof(double) * L.ne);
            if (e == hipSuccess) e = dalloc(p, &L.x, nb);
            if (e == hipSuccess) e = dalloc(p, &L.D, sizeof(double) * 25 * L.nn);
            if (e == hipSuccess) e = dalloc(p, &L.slots, (size_t)n_slots(g) * sizeof(double));
            if (e == hipSuccess) e = dalloc(p, &L.slots25, (size_t)n_tiles(L.geo) * BOXN * 25 * sizeof(double));
            if (e == hipSuccess && mixed) e = dalloc(p, &L.x32, sizeof(float) * L.ndof);
            if (e == hipSuccess && mixed) e = dalloc(p, &L.D32, sizeof(float) * 25 * L.nn);
            if (e == hipSuccess) e = dalloc(p, &L.b, nb);
            if (e == hipSuccess) e = dalloc(p, &L.xs, nb);
            if (e == hipSuccess && mixed) e = dalloc(p, &L.b32, sizeof(float) * L.ndof);
            if (e == hipSuccess && mixed) e = dalloc(p, &L.xs32, sizeof(float) * L.ndof);
        } else if (mixed) {
            if (e == hipSuccess) e = dalloc(p, &L.b32, sizeof(float) * L.ndof);  // cast of the Krylov vector
        }
        if (e == hipSuccess) e = dalloc(p, &L.t, nb);
        if (e == hipSuccess && mixed) e = dalloc(p, &L.t32, sizeof(float) * L.ndof);
        L.assembled = l < nl - 1 && L.nn <= asm_nodes;
        if (L.assembled) {
            if (e == hipSuccess) e = dalloc(p, &L.S, sizeof(double) * 675 * L.nn);
            if (e == hipSuccess && mixed) e = dalloc(p, &L.S32, sizeof(float) * 675 * L.nn);
            if (e == hipSuccess) e = dalloc(p, &L.xa, nb);
            if (e == hipSuccess && mixed) e = dalloc(p, &L.xa32, sizeof(float) * L.ndof);
        }
    }
    const MgLevel &C = mg->lev.back();
    mg->nc = C.ndof;
    int64_t ne_je = C.ne;
    for (const MgLevel &L : mg->lev)
        if (L.assembled) ne_je = std::max(ne_je, L.ne);
    if (e == hipSuccess) e = dalloc(p, &mg->probe, sizeof(double) * 1600 * ne_je);  // element Jacobians
    if (e == hipSuccess) e = dalloc(p, &mg->probe_out, sizeof(double) * 135 * C.ndof);
    if (e == hipSuccess) e = halloc(p, &mg->hbuf, sizeof(double) * 135 * C.ndof);
    // sized for the full matrix: condensing never widens the band
    const int bw = (int)coarse_band(C.grid);
    mg->bw = bw;
    const size_t nfac = (size_t)C.ndof * (3 * bw + 1);
    if (e == hipSuccess) e = halloc(p, &mg->hfac, sizeof(double) * nfac);
    if (e == hipSuccess) e = halloc(p, &mg->hpiv, sizeof(int) * C.ndof);
    if (e == hipSuccess) e = halloc(p, &mg->hmask, C.nn);
    if (e == hipSuccess) e = halloc(p, &mg->hmap, sizeof(int) * 2 * C.ndof);
    if (e == hipSuccess) e = dalloc(p, &mg->dfac, sizeof(double) * nfac);
    if (e == hipSuccess) e = dalloc(p, &mg->dpiv, sizeof(int) * C.ndof);
    if (e == hipSuccess) e = dalloc(p, &mg->dmap, sizeof(int) * 2 * C.ndof);
    if (e == hipSuccess) e = dalloc(p, &mg->Xinv, sizeof(double) * C.ndof * C.ndof);
    if (e == hipSuccess) e = dalloc(p, &mg->cpart, sizeof(double) * ((C.ndof + 63) / 64) * C.ndof);
    if (e == hipSuccess) e = hipEventCreateWithFlags(&mg->probe_ready, hipEventDisableTiming);
    if (e != hipSuccess) {
        mg_free(mg);
        return hip_fail(e, "hipMalloc (multigrid)");
    }
    mg->A.assign((size_t)C.ndof * lu_row(bw, bw), 0.0);
    mg->panel.assign((size_t)LU_NB * (LU_NB + bw), 0.0);
    *out = mg;
    return FE_OK;
}

// Coarse design and source, once per solve (the design is fixed during it).
int mg_set_design(Mg *mg, fe_problem *p, const double *gamma, const double *s, hipStream_t st)
{
    mg->lev[0].gamma = const_cast<double *>(gamma);
    mg->lev[0].s = const_cast<double *>(s);
    mg->lev[0].nmask = p->nmask;
    mg->lev[0].slots = p->slots;
    for (auto &L : mg->lev) L.geo = make_geo(L.grid, p->phys);  // parameters may have changed
    for (size_t l = 1; l < mg->lev.size(); ++l) {
        MgLevel &C = mg->lev[l], &F = mg->lev[l - 1];
        FE_CHECK_HIP(mg_coarsen_elem(C.grid, F.grid, F.gamma, C.gamma, st));
        FE_CHECK_HIP(mg_coarsen_elem(C.grid, F.grid, F.s, C.s, st));
        FE_CHECK_HIP(mg_inject_mask(C.grid, F.grid, F.nmask, C.nmask, st));
    }
    mg->coarse_ready = false;  // the coarsest matrix depends on the design
    return FE_OK;
}

// Index maps of the coarsest level's free DOFs from its node mask (free DOFs
// keep their lexicographic order), and the half bandwidths of the condensed
// matrix: the largest index distance between two free DOFs of nodes at most one
// node apart in each direction.
static void condense_coarse(Mg *mg, const fe_grid &grid)
{
    const int64_t n = mg->nc;
    int *fidx = mg->hmap, *pos = mg->hmap + n;
    int64_t m = 0;
    for (int64_t i = 0; i < n; ++i) {
        if ((mg->hmask[i / NF] >> (i % NF)) & 1) {
            pos[i] = -1;
        } else {
            pos[i] = (int)m;
            fidx[m++] = (int)i;
        }
    }
    mg->nf = m;
    const int nx = grid.nx, ny = grid.ny, nz = grid.nz;
    // first and last free DOF of a node (first > last: none)
    auto first = [&](int64_t N) {
        int64_t r = n;
        for (int g = 0; g < NF; ++g)
            if (pos[NF * N + g] >= 0) r = std::min<int64_t>(r, pos[NF * N + g]);
        return r;
    };
    auto last = [&](int64_t N) {
        int64_t r = -1;
        for (int g = 0; g < NF; ++g) r = std::max<int64_t>(r, pos[NF * N + g]);
        return r;
    };
    int64_t half = 0;  // (nodes are neighbours both ways: kl = ku)
    for (int K = 0; K <= nz; ++K)
        for (int J = 0; J <= ny; ++J)
            for (int I = 0; I <= nx; ++I) {
                const int64_t N = I + (int64_t)(nx + 1) * (J + (int64_t)(ny + 1) * K);
                const int64_t r = last(N);
                if (r < 0) continue;
                for (int dz = -1; dz <= 0; ++dz)  // (later nodes have later DOFs)
                    for (int dy = -1; dy <= 1; ++dy)
                        for (int dx = -1; dx <= 1; ++dx) {
                            const int i = I + dx, j = J + dy, k = K + dz;
                            if (i < 0 || j < 0 || k < 0 || i > nx || j > ny) continue;
                            const int64_t M = i + (int64_t)(nx + 1) * (j + (int64_t)(ny + 1) * k);
                            half = std::max(half, r - first(M));
                        }
            }
    // at least one sub- and super-diagonal (zero ones where the matrix has none)
    mg->kl = mg->ku = (int)std::min<int64_t>(std::max<int64_t>(half, 1), mg->bw);
}

// The coarsest matrix restricted to its free DOFs (m of them), as a band matrix, from
// the 135 colour-by-field probing products: entry (pos[N g], pos[M f]) is row
// N g of product (colour(M), f), M within one node of N, both DOFs free.  The products
// have just come from the device: they are read front to back (240 us at 1125 DOFs entry
// by entry, 130 this way).
static void assemble_free_from_probes(const fe_grid &grid, const double *probe, const int *pos,
                                      int64_t m, int kl, int ku, double *Aw)
{
    const int nx = grid.nx, ny = grid.ny, nz = grid.nz;
    std::fill(Aw, Aw + m * lu_row(kl, ku), 0.0);
    const BandMatrix A(Aw, kl, ku);
    // the neighbour (or itself) of index i whose index mod 3 is c, or -1
    auto near = [](int i, int c, int n) {
        const int j = i + (c - i % 3 + 4) % 3 - 1;
        return j <= n ? j : -1;
    };
    for (int q = 0; q < 135; ++q) {
        const int col = q / NF, f = q % NF, ci = col % 3, cj = col / 3 % 3, ck = col / 9;
        for (int K = 0; K <= nz; ++K)
            for (int J = 0; J <= ny; ++J) {
                const int k = near(K, ck, nz), j = near(J, cj, ny);
                const int64_t N0 = (int64_t)(nx + 1) * (J + (int64_t)(ny + 1) * K);
                const int64_t M0 = (int64_t)(nx + 1) * (j + (int64_t)(ny + 1) * k);
                if (k >= 0 && j >= 0)
                    for (int I = 0; I <= nx; ++I) {
                        const int i = near(I, ci, nx);
                        const int c = i < 0 ? -1 : pos[NF * (M0 + i) + f];
                        if (c < 0) continue;
                        const int *r = pos + NF * (N0 + I);
                        for (int g = 0; g < NF; ++g)
                            if (r[g] >= 0) A.row(r[g])[c] = probe[NF * (N0 + I) + g];
                    }
            }
        probe += NF * (int64_t)(nx + 1) * (ny + 1) * (nz + 1);
    }
}

// Band LU of the condensed coarsest matrix in mg->A; the factors go to the pinned
// buffers in the layout the device inverse reads.
static int band_lu(Mg *mg)
{
    const int64_t n = mg->nf, w = mg->kl + mg->ku;
    double *Lc = mg->hfac, *Uc = Lc + n * mg->kl, *Ud = Uc + n * w;
    static const bool wide = __builtin_cpu_supports("avx512f");
    if (band_lu_factor(n, mg->kl, mg->ku, mg->A.data(), Lc, Uc, Ud, mg->hpiv, mg->panel.data(), wide))
        return FE_OK;
    set_error("multigrid: singular or non-finite coarsest-level matrix");
    return FE_ENAN;
}

// Per Newton step, in two calls around the caller's own fine-level set-up:
// mg_setup_begin injects the linearisation state into every level and starts
// the coarsest level's probing products and their copy to the host;
// mg_setup_finish builds the block diagonals (and FP32 copies in mixed mode)
// and assembled stencils of the other levels, then factorises the coarsest
// level on the host (overlapping that GPU work) and inverts it on the device.
int mg_setup_begin(Mg *mg, fe_problem *p, const double *x, hipStream_t st)
{
    (void)p;
    mg->lev[0].x = const_cast<double *>(x);
    const int nl = (int)mg->lev.size();
    for (int l = 1; l < nl; ++l) {
        MgLevel &C = mg->lev[l], &F = mg->lev[l - 1];
        FE_CHECK_HIP(mg_inject_state(C.grid, F.grid, F.x, C.x, st));
    }
    // with a kept factorisation the coarsest level is not probed again
    mg->skip_coarse = mg->reuse_coarse && mg->coarse_ready;
    if (mg->skip_coarse) return FE_OK;
    // the 135 probing products J p_(colour,field) in FP64 from the coarsest
    // level's element Jacobians (two launches), copied to the host
    MgLevel &C = mg->lev.back();
    FE_CHECK_HIP(launch_probe_products(C.geo, C.x, C.gamma, C.s, C.nmask, mg->probe,
                                       mg->probe_out, st));
    FE_CHECK_HIP(hipMemcpyAsync(mg->hbuf, mg->probe_out, sizeof(double) * 135 * C.ndof,
                                hipMemcpyDeviceToHost, st));
    FE_CHECK_HIP(hipMemcpyAsync(mg->hmask, C.nmask, C.nn, hipMemcpyDeviceToHost, st));
    FE_CHECK_HIP(hipEventRecord(mg->probe_ready, st));
    return FE_OK;
}

int mg_setup_finish(Mg *mg, fe_problem *p, const double *D0, const float *D032, const float *x032,
                    hipStream_t st)
{
    (void)p;
    MgLevel &L0 = mg->lev[0];
    L0.D = const_cast<double *>(D0);
    L0.D32 = const_cast<float *>(D032);
    L0.x32 = const_cast<float *>(x032);
    const int nl = (int)mg->lev.size();
    MgLevel &C = mg->lev.back();
    // a mixed-precision Newton step (FP32 state given) smooths with FP32 blocks
    // only, formed and inverted in FP32; otherwise (FP64 solves, the adjoint)
    // the blocks are FP64, with an FP32 copy in a mixed hierarchy
    const bool blocks32 = x032 != nullptr;
    for (int l = 1; l < nl - 1; ++l) {
        MgLevel &L = mg->lev[l];
        if (mg->mixed) FE_CHECK_HIP((launch_cast<double, float>(L.x, L.x32, L.ndof, st)));
        if (L.assembled) continue;
        if (blocks32) {
            FE_CHECK_HIP((launch_blockdiag<float>(L.geo, L.x32, L.gamma, L.s, L.nmask, L.D32,
                                                  reinterpret_cast<float *>(L.slots25), st)));
            FE_CHECK_HIP(launch_invert_blocks32(L.D32, L.nn, st));
        } else {
            FE_CHECK_HIP((launch_blockdiag<double>(L.geo, L.x, L.gamma, L.s, L.nmask, L.D,
                                                   L.slots25, st)));
            FE_CHECK_HIP(launch_invert_blocks(L.D, mg->mixed ? L.D32 : nullptr, L.nn, st));
        }
    }
    // assembled levels: element Jacobians, then the 27-point block stencil, whose
    // centre blocks are the smoother's diagonal blocks (below the finest level,
    // whose blocks the caller provides)
    for (int l = 0; l < nl - 1; ++l) {
        MgLevel &L = mg->lev[l];
        if (!L.assembled) continue;
        FE_CHECK_HIP(launch_stencil_assemble(L.geo, L.x, L.gamma, L.s, L.nmask, mg->probe, L.S, st));
        if (mg->mixed) FE_CHECK_HIP((launch_cast<double, float>(L.S, L.S32, 675 * L.nn, st)));
        if (l > 0) {
            FE_CHECK_HIP(mg_stencil_diag(L.nn, L.S, L.D, st));
            FE_CHECK_HIP(launch_invert_blocks(L.D, mg->mixed ? L.D32 : nullptr, L.nn, st));
        }
    }
    if (mg->skip_coarse) return FE_OK;  // the kept factorisation serves this step
    // (the event also orders the previous set-up's copy out of hfac before the
    // factorisation below rewrites it)
    FE_CHECK_HIP(hipEventSynchronize(mg->probe_ready));
    condense_coarse(mg, C.grid);
    assemble_free_from_probes(C.grid, mg->hbuf, mg->hmap + mg->nc, mg->nf, mg->kl, mg->ku,
                              mg->A.data());
    int rc = band_lu(mg);
    if (rc) return rc;
    // the factors and index maps to the device, then the inverse column by column
    const int64_t n = mg->nf, w = mg->kl + mg->ku;
    if (n > 0) {
        FE_CHECK_HIP(hipMemcpyAsync(mg->dfac, mg->hfac, sizeof(double) * n * (mg->kl + w + 1),
                                    hipMemcpyHostToDevice, st));
        FE_CHECK_HIP(hipMemcpyAsync(mg->dpiv, mg->hpiv, sizeof(int) * n, hipMemcpyHostToDevice, st));
    }
    FE_CHECK_HIP(hipMemcpyAsync(mg->dmap, mg->hmap, sizeof(int) * 2 * mg->nc, hipMemcpyHostToDevice, st));
    const double *Lc = mg->dfac, *Uc = Lc + n * mg->kl, *Ud = Uc + n * w;
    if (n > 0) FE_CHECK_HIP(mg_coarse_inverse((int)n, mg->kl, mg->ku, Lc, Uc, Ud, mg->dpiv, mg->Xinv, st));
    mg->coarse_ready = true;
    return FE_OK;
}

// Dense row-major J from the 135 colour-by-field probing products: entry
// (N g, M f) is row N g of product (colour(M), f), M within one node of N.
void assemble_from_probes(const fe_grid &grid, const double *probe, double *A)
{
    const int nx = grid.nx, ny = grid.ny, nz = grid.nz;
    const int64_t n = NF * (int64_t)(nx + 1) * (ny + 1) * (nz + 1);
    std::fill(A, A + n * n, 0.0);
    for (int K = 0; K <= nz; ++K)
        for (int J = 0; J <= ny; ++J)
            for (int I = 0; I <= nx; ++I) {
                const int64_t N = I + (int64_t)(nx + 1) * (J + (int64_t)(ny + 1) * K);
                for (int dz = -1; dz <= 1; ++dz)
                    for (int dy = -1; dy <= 1; ++dy)
                        for (int dx = -1; dx <= 1; ++dx) {
                            const int i = I + dx, j = J + dy, k = K + dz;
                            if (i < 0 || j < 0 || k < 0 || i > nx || j > ny || k > nz) continue;
                            const int64_t M = i + (int64_t)(nx + 1) * (j + (int64_t)(ny + 1) * k);
                            const int col = (i % 3) + 3 * (j % 3) + 9 * (k % 3);
                            for (int g = 0; g < NF; ++g)
                                for (int f = 0; f < NF; ++f)
                                    A[(NF * N + g) * n + NF * M + f] =
                                        probe[(int64_t)(NF * col + f) * n + NF * N + g];
                        }
            }
}

template <typename T>
static T *vecT(MgLevel &L, int which);
template <>
double *vecT<double>(MgLevel &L, int which) { return which == 0 ? L.b : which == 1 ? L.xs : L.t; }
template <>
float *vecT<float>(MgLevel &L, int which) { return which == 0 ? L.b32 : which == 1 ? L.xs32 : L.t32; }
template <typename T>
static const T *stateT(const MgLevel &L);
template <>
const double *stateT<double>(const MgLevel &L) { return L.x; }
template <>
const float *stateT<float>(const MgLevel &L) { return L.x32; }
template <typename T>
static const T *blocksT(const MgLevel &L);
template <>
const double *blocksT<double>(const MgLevel &L) { return L.D; }
template <>
const float *blocksT<float>(const MgLevel &L) { return L.D32; }

template <typename T>
static const T *stencilT(const MgLevel &L);
template <>
const double *stencilT<double>(const MgLevel &L) { return L.S; }
template <>
const float *stencilT<float>(const MgLevel &L) { return L.S32; }

template <typename T>
static hipError_t op(const MgLevel &L, const T *v, T *out, bool tr, hipStream_t st)
{
    if (L.assembled)
        return mg_stencil_apply<T>(L.grid.nx, L.grid.ny, L.grid.nz, stencilT<T>(L), v, out, tr, st);
    return launch_elem<T, T>(tr ? OP_JTV : OP_JV, L.geo, stateT<T>(L), v, L.gamma, L.s, L.nmask, out,
                             (T *)L.slots, st);
}

template <typename T>
static T *altT(MgLevel &L);
template <>
double *altT<double>(MgLevel &L) { return L.xa; }
template <>
float *altT<float>(MgLevel &L) { return L.xa32; }

// x = omega D^{-1} b with b = (float) v (mixed-precision cycles; FP64 has nothing to cast)
static hipError_t smooth0_cast(MgLevel &L, const double *v, float *b, float *x, float om, bool tr,
                               hipStream_t st)
{
    return mg_smooth0_cast(L.D32, v, b, x, L.nn, om, tr, st);
}
static hipError_t smooth0_cast(MgLevel &, const double *, double *, double *, double, bool,
                               hipStream_t)
{
    return hipErrorInvalidValue;
}

// V-cycle from level l (not the coarsest) on b; x receives the result.
// first_done: the first pre-smoothing sweep from x = 0 (x = omega D^{-1} b) has
// already been applied to x, by the restriction kernel of the level above (or, at
// the finest level of a mixed-precision cycle, together with the cast of the Krylov
// vector).  v (finest level of a mixed-precision cycle): b is still to be cast from v.
// A damped block-Jacobi sweep x += omega D^{-1} (b - A x) (transposed when tr)
// is fused with the element pass on matrix-free levels, and is one kernel on
// assembled ones, which writes the new iterate to the level's second buffer:
// the iterate alternates between x and that buffer, and ends in x.  On assembled
// levels the second sweep also forms the first one's x, and the first sweep after
// the coarse-grid correction adds that correction.
template <typename T>
static int vcycle(Mg *mg, int l, const T *b, T *x, bool tr, hipStream_t st, bool first_done = false,
                  const double *v = nullptr)
{
    MgLevel &L = mg->lev[l];
    const int nl = (int)mg->lev.size();
    const T om = (T)mg->omega;
    const T *D = blocksT<T>(L), *S = stencilT<T>(L);
    T *t = vecT<T>(L, 2);
    T *cur = x;
    auto other = [&]() { return cur == x ? altT<T>(L) : x; };
    auto sweep = [&]() -> hipError_t {
        if (L.assembled) {
            T *nxt = other();
            const hipError_t e = mg_stencil_smooth<T>(L.grid.nx, L.grid.ny, L.grid.nz, S, D, b, cur,
                                                      nxt, om, tr, st);
            cur = nxt;
            return e;
        }
        return launch_elem_smooth<T>(tr, L.geo, stateT<T>(L), cur, L.gamma, L.s, L.nmask, t,
                                     (T *)L.slots, D, b, om, st);
    };
    int pre = 1;
    if (!first_done) {
        if (L.assembled && mg->nu1 > 1) {
            T *nxt = other();
            FE_CHECK_HIP(mg_sweep_first<T>(L.grid.nx, L.grid.ny, L.grid.nz, S, D, b, v,
                                           v ? const_cast<T *>(b) : nullptr, nxt, om, tr, st));
            cur = nxt;
            pre = 2;
        } else if (v) {
            FE_CHECK_HIP(smooth0_cast(L, v, const_cast<T *>(b), x, om, tr, st));
        } else {
            FE_CHECK_HIP(mg_smooth<T>(D, b, nullptr, x, L.nn, om, tr, false, st));
        }
    }
    for (int it = pre; it < mg->nu1; ++it) FE_CHECK_HIP(sweep());
    MgLevel &C = mg->lev[l + 1];
    FE_CHECK_HIP(op<T>(L, cur, t, tr, st));
    T *bc = vecT<T>(C, 0), *xc = vecT<T>(C, 1);
    int post = 0;
    if (l + 1 < nl - 1) {
        // the coarse level's first sweep is fused into the restriction
        FE_CHECK_HIP(mg_restrict_smooth<T>(C.grid, L.grid, b, t, C.nmask, bc, blocksT<T>(C), xc, om,
                                           tr, st));
        int rc = vcycle<T>(mg, l + 1, bc, xc, tr, st, true);
        if (rc) return rc;
    } else {
        // directly solved coarsest level: x_c = A^{-1} R (b - t)
        const int nc = (int)mg->nc, nf = (int)mg->nf;
        const int *pos = mg->dmap + mg->nc;
        if (nf > 0)
            FE_CHECK_HIP(mg_restrict_coarse<T>(C.grid, L.grid, nf, mg->Xinv, mg->dmap, b, t,
                                               mg->cpart, tr, st));
        if (L.assembled && mg->nu2 > 0 && mg_sweep_coarse_pays(nc, nf)) {
            T *nxt = other();
            FE_CHECK_HIP(mg_sweep_coarse<T>(L.grid, C.grid, S, D, b, cur, nc, nf, pos, mg->cpart,
                                            L.nmask, nxt, om, tr, st));
            cur = nxt;
            post = 1;
        } else {
            FE_CHECK_HIP(mg_coarse_sum<T>(nc, nf, pos, mg->cpart, xc, st));
        }
    }
    if (post == 0) {
        if (L.assembled && mg->nu2 > 0) {
            T *nxt = other();
            FE_CHECK_HIP(mg_sweep_prolong<T>(L.grid, C.grid, S, D, b, cur, xc, L.nmask, nxt, om, tr,
                                             st));
            cur = nxt;
            post = 1;
        } else {
            FE_CHECK_HIP(mg_prolong_add<T>(L.grid, C.grid, xc, L.nmask, cur, st));
        }
    }
    for (int it = post; it < mg->nu2; ++it) FE_CHECK_HIP(sweep());
    if (cur != x) FE_CHECK_HIP(mg_copy<T>(cur, x, L.ndof, st));
    return FE_OK;
}

int mg_apply64(Mg *mg, const double *v, double *z, bool tr, hipStream_t st)
{
    return vcycle<double>(mg, 0, v, z, tr, st);
}

int mg_apply32(Mg *mg, const double *v, float *z, bool tr, hipStream_t st)
{
    return vcycle<float>(mg, 0, mg->lev[0].b32, z, tr, st, false, v);
}

}  // namespace fe
