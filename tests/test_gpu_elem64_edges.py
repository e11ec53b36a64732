"""The FP64 passes in tiles of two layers (chosen where they leave a workgroup to a CU),
with a last tile of one and partial tiles in x and y.

The parity suite's 1e-11.
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


TWO = [(28, 28, 28), (32, 32, 32), (9, 9, 65), (128, 128, 2), (17, 31, 33)]


@pytest.mark.parametrize("size", TWO, ids=lambda s: "x".join(map(str, s)))
def test_tiles_of_two_layers(fe, size):
    print(f"[elem64] {size}", flush=True)
    p = inputs.tiny_problem(*size, Gr=2e4, seed=12)
    m = p.mask_solve
    x = inputs.random_state(p, 2002, mask=m)
    v = np.random.default_rng(3).standard_normal(p.n_dof)
    prob = fe.Problem.from_inputs(p, mask="solve")
    g, s, xd, vd = dev(p.gamma), dev(p.s), dev(x), dev(v)
    assert_parity(host(fe.fe_residual(prob, xd, g, s)), oracle.residual(p, x, mask=m), what="R")
    assert_parity(host(fe.fe_jvp(prob, xd, g, s, vd)), oracle.jvp(p, x, v, mask=m), what="J v")
    assert_parity(host(fe.fe_adjoint_jtvp(prob, xd, g, s, vd)), oracle.jtvp(p, x, v, mask=m), what="J^T w")
