"""The FP64 operator passes where |u_e|^2 overflows: tau and tauT are 1 / sqrt(inf) = 0
there, and a uniform velocity, which advects nothing, leaves every row finite.

|u|_i = 2^511: the sum of 24 squares is beyond 2^1024.  The residual's rows are alpha u and
below, some 1e157 h^3, plus whatever u (grad u) rounds to: at most |u|^2 times the parity
suite's 1e-11.  J v, scaled into range for the norms, is held to the 1e-11 itself.
"""
import numpy as np
import pytest

import oracle
from paper_1508_04596_amd import inputs
from tests.helpers import assert_parity

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def test_overflowing_speed_leaves_the_rows_finite():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1508_04596_amd import fe
    p = inputs.tiny_problem(9, 3, 4, Gr=1e3, seed=7)
    none = np.zeros(p.n_dof, dtype=np.uint8)
    x = np.zeros(p.n_dof).reshape(-1, 5)
    x[:, :3] = 2.0 ** 511
    x = x.reshape(-1)
    v = np.random.default_rng(4).standard_normal(p.n_dof)
    g, s, xd, vd = (torch.from_numpy(np.ascontiguousarray(a)).cuda() for a in (p.gamma, p.s, x, v))
    prob = fe.Problem.from_inputs(p, mask=None)
    r = fe.fe_residual(prob, xd, g, s).cpu().numpy()
    assert np.isfinite(r).all() and np.abs(r).max() <= 1e-11 * 2.0 ** 1022
    want = oracle.jvp(p, x, v, mask=none)
    assert np.isfinite(want).all()
    assert_parity(fe.fe_jvp(prob, xd, g, s, vd).cpu().numpy() * 1e-150, want * 1e-150, what="J v")
