"""FP64 operator passes at the edges of their tiling.

The passes march through tiles of 8x8xL elements, L chosen from the grid; a wave
holds two rows of eight elements.  The sizes below reach one layer per tile (with
a full and a nearly empty last tile), the largest L, an L that does not divide the
grid, and partial tiles in x and y.  The bound is the parity suite's 1e-11: the
sums have at most 8 elements x 8 Gauss points of terms of mixed sign, a few
hundred roundings of 1.1e-16 relative to the largest entry.
"""
import numpy as np
import pytest

import oracle
from paper_1508_04596_amd import inputs
from tests.helpers import assert_parity

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def fe():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1508_04596_amd import fe as fe_mod
    fe_mod.lib()
    return fe_mod


def dev(a, dtype=torch.float64):
    return torch.from_numpy(np.ascontiguousarray(a)).to("cuda", dtype)


def host(t):
    torch.cuda.synchronize()
    return t.double().cpu().numpy()


# (nx, ny, nz): layers per tile
SIZES = [(8, 8, 1), (9, 7, 2), (3, 2, 41), (16, 17, 65),  # 1
         (41, 33, 37),                                     # 3, last tile one layer
         (129, 129, 3), (131, 130, 16), (185, 184, 9)]     # 3, 16, 5 (last tile four)


@pytest.mark.parametrize("size", SIZES, ids=["x".join(map(str, s)) for s in SIZES])
def test_operators_at_tile_edges(fe, size):
    nx, ny, nz = size
    print(f"[elem64] {size}", flush=True)
    p = inputs.tiny_problem(nx, ny, nz, Gr=2e4, seed=11)
    m = p.mask_solve
    x = inputs.random_state(p, 2001, mask=m)
    v = np.random.default_rng(3).standard_normal(p.n_dof)
    prob = fe.Problem.from_inputs(p, mask="solve")
    g, s, xd, vd = dev(p.gamma), dev(p.s), dev(x), dev(v)
    assert_parity(host(fe.fe_residual(prob, xd, g, s)), oracle.residual(p, x, mask=m), what="R")
    jv = host(fe.fe_jvp(prob, xd, g, s, vd))
    assert_parity(jv, oracle.jvp(p, x, v, mask=m), what="J v")
    np.testing.assert_array_equal(jv[m.astype(bool)], v[m.astype(bool)])
    jt = host(fe.fe_adjoint_jtvp(prob, xd, g, s, vd))
    w = inputs.random_direction(p, 5, mask=m)
    a = float(np.dot(host(fe.fe_jvp(prob, xd, g, s, dev(w))), np.where(m, 0.0, v)))
    b = float(np.dot(w, np.where(m, 0.0, jt)))
    scale = float(np.linalg.norm(jv) * np.linalg.norm(w))
    assert abs(a - b) <= 1e-11 * scale, (a, b, scale)
