"""The V-cycle's fused small-level kernels (first sweep with its own x, post sweep
with its own prolongation or coarse solution, restriction with the coarse solve's
first pass) against the cycle on matrix-free levels, which has none of them.

The two cycles are the same operator up to rounding, so solves to 1e-8 take the same
Newton steps, the same Krylov steps to within one each, and end within the solver's
tolerance of each other times the condition of the preconditioned system, taken as 100
(1e-6; adjoint, from two such states, 1e-5).

Sizes: two levels and three, even and odd (overhanging coarse elements), the finest
level just above the coarsest; coarsest levels on both sides of the rule for summing
its partials in the post sweep (4x3x2 and 4^3 inside, 5^3 outside); a last workgroup
of few nodes.  Sweeps: one and two before, none, one and two after.
"""
import numpy as np
import pytest

import oracle
from paper_1508_04596_amd import inputs
from tests.helpers import rel_norm

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def fe():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1508_04596_amd import fe as fe_mod
    fe_mod.lib()
    return fe_mod


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).to("cuda", torch.float64)


@pytest.mark.parametrize("sweeps", [(2, 1), (1, 1), (2, 0), (2, 2)], ids=lambda s: f"nu{s[0]}-{s[1]}")
@pytest.mark.parametrize("pc", ["FE_FP64", "FE_FP32"])
@pytest.mark.parametrize("dims", [(8, 6, 4), (10, 10, 10), (17, 13, 9), (16, 16, 15)],
                         ids=lambda d: "x".join(map(str, d)))
def test_fused_small_levels(fe, dims, pc, sweeps):
    p = inputs.scaled_config(*dims, 1e4, seed=77)
    g, s = dev(p.gamma), dev(p.s)
    out = {}
    for asm in (0, -1):
        print(f"[vcycle] {dims} {pc} {sweeps} mg_assembled_nodes={asm}", flush=True)
        prob = fe.Problem.from_inputs(p, mask="solve")
        kw = dict(precond="multigrid", mg_assembled_nodes=asm, mg_nu=sweeps[0],
                  mg_nu_post=sweeps[1], pc_prec=getattr(fe, pc))
        x = torch.zeros(p.n_dof, dtype=torch.float64, device="cuda")
        rep = fe.newton_solve(prob, g, s, x, fe.solve_opts(rtol_newton=1e-8, **kw))
        c = torch.empty_like(x)
        fe.fe_compliance(prob, x, s, c)
        lam, arep = fe.fe_adjoint_solve(prob, x, g, s, c, opts=fe.solve_opts(rtol_lin=1e-8, **kw))
        torch.cuda.synchronize()
        out[asm] = (x.cpu().numpy(), rep, lam.cpu().numpy(), arep)
        prob.close()
    (x0, r0, l0, a0), (x1, r1, l1, a1) = out[0], out[-1]
    assert r0["mg_levels"] == r1["mg_levels"] >= 2
    assert r0["newton_its"] == r1["newton_its"]
    assert all(abs(a - b) <= 1 for a, b in zip(r0["lin_its"], r1["lin_its"]))
    assert abs(a0["lin_its_total"] - a1["lin_its_total"]) <= 1
    assert rel_norm(x1, x0) <= 1e-6
    assert rel_norm(l1, l0) <= 1e-5


# coarsest level (half the fine counts) whose half bandwidth takes each slot count of the
# register-resident inverse: 21, 46, 65, 101, 138, 175, 212, 249; then 671 unknowns, which
# it takes two columns per wave for
@pytest.mark.parametrize("dims", [(4, 4, 24), (4, 10, 8), (6, 8, 6), (6, 14, 8), (8, 14, 8), (10, 14, 8),
                                  (12, 14, 6), (14, 14, 6), (10, 10, 14)],
                         ids=lambda d: "x".join(map(str, d)))
def test_coarsest_level_bands(fe, dims):
    """An exact coarse solve on two levels: 20 Krylov steps reduce a Newton system's
    residual enough, and the states reach the oracle's residual (the bounds of the
    two-level slab in the solver's tests)."""
    print(f"[coarse] {dims}", flush=True)
    p = inputs.scaled_config(*dims, 2e3, seed=404)
    prob = fe.Problem.from_inputs(p, mask="solve")
    x = torch.zeros(p.n_dof, dtype=torch.float64, device="cuda")
    rep = fe.newton_solve(prob, dev(p.gamma), dev(p.s), x,
                          fe.solve_opts(rtol_newton=1e-8, precond="multigrid"))
    torch.cuda.synchronize()
    r0 = np.linalg.norm(oracle.residual(p, np.zeros(p.n_dof), mask="solve"))
    r = np.linalg.norm(oracle.residual(p, x.cpu().numpy(), mask="solve"))
    print(f"[coarse] newton {rep['newton_its']} lin {rep['lin_its']} rel {r / r0:.2e}")
    assert rep["mg_levels"] == 2
    assert r <= 1e-8 * r0 * 1.0001
    assert max(rep["lin_its"]) <= 20
    prob.close()
