"""The coarsest multigrid level's band LU (host code, ``csrc/fe_band_lu.h``), compiled by
itself: both forms of the trailing update give the same factors bit for bit, the factors
invert the matrix, every factor is written, and nothing is written outside the buffers.

Bound of the inverse: elimination with partial pivoting by another order of the same sums,
so the residual |A X - I| is at most 100 times that of LAPACK's inverse.
"""
import ctypes
import os
import subprocess

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1508_04596_amd", "csrc")
NB = 8
GUARD = 64
SRC = """#include "fe_band_lu.h"
extern "C" int band_lu(int64_t n, int kl, int ku, double *A, double *Lc, double *Uc, double *Ud, int *piv,
                       double *panel, int wide)
{
    return fe::band_lu_factor(n, kl, ku, A, Lc, Uc, Ud, piv, panel, wide != 0);
}
extern "C" int has_wide() { return __builtin_cpu_supports("avx512f") ? 1 : 0; }
"""


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    d = tmp_path_factory.mktemp("band_lu")
    (d / "t.cpp").write_text(SRC)
    cxx = os.path.join(os.environ.get("ROCM_PATH", "/opt/rocm"), "bin", "amdclang++")
    # the library's host flags
    subprocess.run([cxx, "-O3", "-std=c++17", "-fPIC", "-shared", "-mavx2", "-mfma", "-I" + CSRC,
                    str(d / "t.cpp"), "-o", str(d / "t.so")], check=True)
    L = ctypes.CDLL(str(d / "t.so"))
    dp, ip = ctypes.POINTER(ctypes.c_double), ctypes.POINTER(ctypes.c_int)
    L.band_lu.argtypes = [ctypes.c_int64, ctypes.c_int, ctypes.c_int, dp, dp, dp, dp, ip, dp, ctypes.c_int]
    return L


def guarded(size, dtype=np.float64):
    """Buffer of `size` entries, not yet numbers, with a guard on both sides."""
    fill = np.nan if dtype is np.float64 else -7
    full = np.full(size + 2 * GUARD, fill, dtype)
    full[:GUARD] = full[GUARD + size:] = 12345
    return full, full[GUARD:GUARD + size]


def factor(L, A, kl, ku, wide):
    n = len(A)
    row = 2 * kl + ku + 2 * NB + 1
    buf = {"A": guarded(n * row), "Lc": guarded(n * kl), "Uc": guarded(n * (kl + ku)), "Ud": guarded(n),
           "piv": guarded(n, np.int32), "panel": guarded(NB * (NB + kl))}
    band = buf["A"][1]
    band[:] = 0.0
    for i in range(n):
        for j in range(max(0, i - kl), min(n, i + ku + 1)):
            band[i * row + kl + NB + j - i] = A[i, j]
    dp, ip = ctypes.POINTER(ctypes.c_double), ctypes.POINTER(ctypes.c_int)
    p = {k: v[1].ctypes.data_as(ip if k == "piv" else dp) for k, v in buf.items()}
    ok = L.band_lu(n, kl, ku, p["A"], p["Lc"], p["Uc"], p["Ud"], p["piv"], p["panel"], wide)
    for k, (full, inner) in buf.items():
        assert (full[:GUARD] == 12345).all() and (full[GUARD + inner.size:] == 12345).all(), k
    return ok, {k: buf[k][1].copy() for k in ("Lc", "Uc", "Ud", "piv")}


def inverse(n, kl, ku, f):
    """As the device forms it: swaps and eliminations in turn, then back substitution."""
    w = kl + ku
    Lc, Uc = f["Lc"].reshape(n, kl), f["Uc"].reshape(n, w)
    Y = np.eye(n)
    for k in range(n):
        p = f["piv"][k]
        Y[[k, p]] = Y[[p, k]]
        m = min(kl, n - 1 - k)
        Y[k + 1:k + 1 + m] -= np.outer(Lc[k, :m], Y[k])
        assert not Lc[k, m:].any()
    for k in reversed(range(n)):
        Y[k] /= f["Ud"][k]
        m = min(w, k)
        Y[k - m:k] -= np.outer(Uc[k, :m][::-1], Y[k])
        assert not Uc[k, m:].any()
    return Y


def matrix(n, kl, ku, seed):
    i, j = np.indices((n, n))
    A = np.random.default_rng(seed).standard_normal((n, n))
    return np.where((j - i <= ku) & (i - j <= kl), A, 0.0)


# one panel and less, whole panels, a rest; bands narrower than a panel, wider than the
# matrix; columns beside the panel that fill no vector, some, and a rest of them
SIZES = [(1, 1), (5, 1), (8, 2), (9, 12), (16, 3), (17, 5), (40, 7), (64, 21), (101, 9), (233, 87), (300, 110)]


@pytest.mark.parametrize("n,k", SIZES)
def test_factors(lib, n, k):
    A = matrix(n, k, k, 100 * n + k)
    ok, f = factor(lib, A, k, k, 0)
    assert ok
    X = inverse(n, k, k, f)
    lapack = np.abs(A @ np.linalg.inv(A) - np.eye(n)).max()
    assert np.abs(A @ X - np.eye(n)).max() <= 100 * max(lapack, np.finfo(float).eps)


@pytest.mark.parametrize("n,k", SIZES)
def test_same_factors_on_every_host(lib, n, k):
    if not lib.has_wide():
        pytest.skip("this host has one form of the update only")
    A = matrix(n, k, k, 100 * n + k)
    (ok0, a), (ok1, b) = factor(lib, A, k, k, 0), factor(lib, A, k, k, 1)
    assert ok0 and ok1
    for name in a:
        np.testing.assert_array_equal(a[name], b[name], err_msg=name)


@pytest.mark.parametrize("wide", [0, 1])
@pytest.mark.parametrize("bad", [0.0, np.nan, np.inf])
def test_no_pivot(lib, wide, bad):
    if wide and not lib.has_wide():
        pytest.skip("this host has one form of the update only")
    A = matrix(30, 4, 4, 3)
    A[:, 17] = np.where(A[:, 17] != 0.0, bad, 0.0)
    assert not factor(lib, A, 4, 4, wide)[0]
