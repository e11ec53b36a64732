"""The FP64 passes' other forms at the edges of their tiling: tiles of two layers (chosen
where they leave a workgroup to a CU) with a last tile of one, the batched passes, and the
direction stored in FP32 (the Krylov operator under an FP32 preconditioner).

Operators: the parity suite's 1e-11.  Batched J v: bit for bit the single one.  Solves: the
oracle's residual at the solver's target, and the batched server's solutions as far from
the single solve's as two solves to 1e-8 may be, times 100 for the system's condition.
"""
import numpy as np
import pytest

import oracle
from paper_1508_04596_amd import inputs
from tests.helpers import assert_parity, rel_norm

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


# one layer a tile (a last tile nearly empty in x), two, three with a last one of one, 16 and 5
MIX = [(9, 7, 2), (3, 2, 41), (32, 32, 31), (41, 33, 37), (131, 130, 16), (185, 184, 9)]


def test_batched_jvp_is_the_single_one(fe):
    items = []
    for k, size in enumerate(MIX):
        print(f"[elem64] {size}", flush=True)
        p = inputs.tiny_problem(*size, Gr=1e4, seed=40 + k)
        prob = fe.Problem.from_inputs(p, mask="solve")
        rng = np.random.default_rng(50 + k)
        items.append((prob, dev(0.1 * rng.standard_normal(p.n_dof)), dev(p.gamma), dev(p.s),
                      dev(rng.standard_normal(p.n_dof))))
    refs = [fe.fe_jvp(pr, x, g, s, v) for pr, x, g, s, v in items]
    for order in (range(len(items)), [5, 2, 0]):
        it = [items[i] for i in order]
        outs = [torch.full_like(i[4], float("nan")) for i in it]
        b = fe.JvpBatch(*([i[c] for i in it] for c in range(5)), outs)
        b.run()
        torch.cuda.synchronize()
        for o, i in zip(outs, order):
            assert torch.equal(o, refs[i]), MIX[i]
        b.close()


# finest levels that are matrix-free, so that the smoothing passes run on them: two layers
# and a last tile of one, partial tiles; three layers
@pytest.mark.parametrize("dims", [(33, 31, 29), (41, 33, 37)], ids=lambda s: "x".join(map(str, s)))
def test_fp32_direction_and_batched_smoothing(fe, dims):
    p = inputs.scaled_config(*dims, 1e4, seed=909)
    g, s = dev(p.gamma), dev(p.s)
    r0 = np.linalg.norm(oracle.residual(p, np.zeros(p.n_dof), mask="solve"))
    ph = fe.make_phys(p.Pr, p.Gr, p.Ck, p.qf, p.alpha_max, p.q_alpha, p.eg)
    for pc in ("fp64", "fp32"):
        print(f"[elem64] {dims} {pc}", flush=True)
        o = fe.solve_opts(rtol_newton=1e-8, pc_prec=pc)
        prob = fe.Problem.from_inputs(p, mask="solve")
        x = torch.zeros(p.n_dof, dtype=torch.float64, device="cuda")
        rep = fe.newton_solve(prob, g, s, x, o)
        assert rep["mg_levels"] >= 2
        with fe.Server(4 << 30, max_active=2, batched=True) as srv:
            tickets = [srv.submit(p.nx, p.ny, p.nz, p.h, ph, p.gamma, p.s, o) for _ in range(2)]
            xs = [srv.wait(t)[1] for t in tickets]
        for y in [host(x)] + [np.asarray(t) for t in xs]:
            assert np.linalg.norm(oracle.residual(p, y, mask="solve")) <= 1e-8 * r0 * 1.0001
            assert rel_norm(y, host(x)) <= 1e-6
        prob.close()
