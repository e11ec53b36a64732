// Band LU of the coarsest multigrid level's matrix, on the host (internal).
#pragma once

#include <algorithm>
#include <cmath>
#include <cstdint>

namespace fe {

// Row i of the band matrix holds columns i - kl - LU_NB .. i + kl + ku + LU_NB (the
// fill of row swaps, and a panel's width on both sides), row after row.
constexpr int LU_NB = 8;
inline int64_t lu_row(int64_t kl, int64_t ku) { return 2 * kl + ku + 2 * LU_NB + 1; }

struct BandMatrix {
    double *a;
    int64_t step, off;
    BandMatrix(double *w, int64_t kl, int64_t ku) : a(w), step(lu_row(kl, ku) - 1), off(kl + LU_NB) {}
    double *row(int64_t i) const { return a + i * step + off; }  // indexed by column
};

// r[0 .. n) -= sum_c l[c] u[c ustep + 0 .. n), c < LU_NB: V doubles at a time.  Every
// column adds the even and the odd c apart, fused, whatever V is and however many columns
// are left over: the factors are the same on every host.
template <typename V>
__attribute__((always_inline)) static inline void lu_update(double *r, const double *l,
                                                            const double *u, int64_t ustep,
                                                            int64_t n)
{
    constexpr int W = sizeof(V) / sizeof(double);
    typedef V U __attribute__((aligned(8)));
    V lv[LU_NB];
    for (int c = 0; c < LU_NB; ++c) lv[c] = l[c] - V{};
    int64_t j = 0;
    for (; j + 2 * W <= n; j += 2 * W) {
        V s0{}, s1{}, t0{}, t1{};
#pragma unroll
        for (int c = 0; c < LU_NB; c += 2) {
            s0 += lv[c] * *(const U *)(u + c * ustep + j);
            s1 += lv[c] * *(const U *)(u + c * ustep + j + W);
            t0 += lv[c + 1] * *(const U *)(u + (c + 1) * ustep + j);
            t1 += lv[c + 1] * *(const U *)(u + (c + 1) * ustep + j + W);
        }
        *(U *)(r + j) = *(const U *)(r + j) - (s0 + t0);
        *(U *)(r + j + W) = *(const U *)(r + j + W) - (s1 + t1);
    }
    for (; j < n; ++j) {
        double s = 0.0, t = 0.0;
        for (int c = 0; c < LU_NB; c += 2) {
            s = std::fma(l[c], u[c * ustep + j], s);
            t = std::fma(l[c + 1], u[(c + 1) * ustep + j], t);
        }
        r[j] -= s + t;
    }
}
typedef double lu_v4 __attribute__((vector_size(32)));
typedef double lu_v8 __attribute__((vector_size(64)));

// Rows i0 .. i1 of the trailing matrix, columns j0 .. j0 + n - 1, less the panel's
// product: P holds the panel by columns (pr rows each), its first row is row k0.
#define FE_LU_TRAILING                                                                            \
    for (int64_t i = i0; i < i1; ++i) {                                                            \
        double l[LU_NB];                                                                           \
        bool any = false;                                                                          \
        for (int c = 0; c < LU_NB; ++c) {                                                          \
            l[c] = P[c * pr + (i - k0)];                                                           \
            any |= l[c] != 0.0;                                                                    \
        }                                                                                          \
        if (any) lu_update<V>(A.row(i) + j0, l, A.row(k0) + j0, A.step, n);                        \
    }
inline void lu_trailing(const BandMatrix &A, const double *P, int64_t pr, int64_t k0, int64_t i0,
                        int64_t i1, int64_t j0, int64_t n)
{
    typedef lu_v4 V;
    FE_LU_TRAILING
}
__attribute__((target("avx512f"))) inline void lu_trailing512(const BandMatrix &A, const double *P,
                                                              int64_t pr, int64_t k0, int64_t i0,
                                                              int64_t i1, int64_t j0, int64_t n)
{
    typedef lu_v8 V;
    FE_LU_TRAILING
}
#undef FE_LU_TRAILING

// Band LU with partial pivoting of the n x n matrix A, LU_NB columns at a time: the
// panel is factored in a buffer by columns, and its row operations are applied to the
// rest of the band together.  The GPU waits for this; one column at a time read and
// wrote the whole window, 200 KB, for every column: n = 632, kl = 110: 1.24 ms, here
// 0.60; n = 233, kl = 87: 0.24, here 0.13.  (One workgroup on the device, its window in
// registers, took 1.1 and 0.36 ms: a step's pivot search is a chain of instructions that
// nothing else on the CU fills.)  Lc, Uc, Ud, piv: the layout the device inverse reads
// (multipliers as they were in step k, before later swaps).  wide: the host
// has AVX-512 (n = 632: 877 us without).  False: zero or non-finite pivot.
inline bool band_lu_factor(int64_t n, int kl, int ku, double *Aw, double *Lc, double *Uc, double *Ud,
                           int *piv, double *panel, bool wide)
{
    const BandMatrix A(Aw, kl, ku);
    const int64_t w = kl + ku, pr = LU_NB + kl;
    double *P = panel;
    for (int64_t k0 = 0; k0 < n; k0 += LU_NB) {
        const int64_t nb = std::min<int64_t>(LU_NB, n - k0), j0 = k0 + nb;
        const int64_t m = std::min<int64_t>(n, j0 + kl) - k0;        // panel rows
        const int64_t nt = std::min<int64_t>(n, j0 + w) - j0;        // columns right of the panel
        for (int64_t i = 0; i < m; ++i)
            for (int64_t c = 0; c < nb; ++c) P[c * pr + i] = A.row(k0 + i)[k0 + c];
        for (int64_t c = 0; c < nb; ++c) {
            const int64_t k = k0 + c, ie = std::min<int64_t>(m, c + 1 + kl);
            double *pc = P + c * pr;
            int64_t p = c;
            double best = std::fabs(pc[c]);
            for (int64_t i = c + 1; i < ie; ++i)
                if (std::fabs(pc[i]) > best) {
                    best = std::fabs(pc[i]);
                    p = i;
                }
            piv[k] = (int)(k0 + p);
            if (best == 0.0 || !std::isfinite(best)) return false;
            if (p != c) {
                for (int64_t q = 0; q < nb; ++q) std::swap(P[q * pr + c], P[q * pr + p]);
                std::swap_ranges(A.row(k) + j0, A.row(k) + j0 + nt, A.row(k0 + p) + j0);
            }
            const double inv = 1.0 / pc[c];
            double *lc = Lc + k * kl;
            for (int64_t i = c + 1; i < ie; ++i) lc[i - c - 1] = pc[i] *= inv;
            for (int64_t i = ie - c - 1; i < kl; ++i) lc[i] = 0.0;
            for (int64_t q = c + 1; q < nb; ++q) {
                double *pq = P + q * pr;
                const double u = pq[c];
                if (u != 0.0)
                    for (int64_t i = c + 1; i < ie; ++i) pq[i] -= pc[i] * u;
            }
        }
        // the panel's rows of U right of it, and U by columns: Uc[k w + q] = U(k - 1 - q, k)
        for (int64_t c = 1; c < nb; ++c)
            for (int64_t q = 0; q < c; ++q) {
                const double l = P[q * pr + c], *rq = A.row(k0 + q) + j0;
                double *rc = A.row(k0 + c) + j0;
                if (l != 0.0)
                    for (int64_t j = 0; j < nt; ++j) rc[j] -= l * rq[j];
            }
        for (int64_t c = 0; c < nb; ++c) {
            Ud[k0 + c] = P[c * pr + c];
            for (int64_t q = 0; q < std::min(c, w); ++q) Uc[(k0 + c) * w + q] = P[c * pr + c - 1 - q];
            const double *rc = A.row(k0 + c) + j0;
            double *u = Uc + j0 * w + (nb - 1 - c);
            for (int64_t j = 0; j < std::min(nt, w - (nb - 1 - c)); ++j) u[j * (w + 1)] = rc[j];
        }
        if (nb < LU_NB) break;  // (the last panel: nothing below it)
        (wide ? lu_trailing512 : lu_trailing)(A, P, pr, k0, j0, k0 + m, j0, nt);
    }
    for (int64_t k = 0; k < std::min(n, w); ++k)
        std::fill(Uc + k * w + k, Uc + (k + 1) * w, 0.0);
    return true;
}

}  // namespace fe
