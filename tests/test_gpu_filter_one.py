"""The density filter's one-launch iteration (grids up to 300,000 nodes): several tiles,
also several per workgroup (1x1x9000), against exact sparse solves; a zero field; a field that is not a number; and the sizes on
both sides of the limit, too large for a sparse factorisation here, by what F must keep
(constants, and <F u, v> = <u, F^T v>).

As for the tile edges, conjugate gradients stop at a relative residual of 1e-12 with a
condition number below 100: 1e-10 of the largest entry (of the norms' product).
"""
import numpy as np
import pytest

from oracle.filter import Filter as OFilter

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


@pytest.mark.parametrize("dims", [(2, 2, 1), (41, 41, 3), (23, 17, 21), (50, 4, 30), (1, 1, 9000)],
                         ids=lambda d: "x".join(map(str, d)))
def test_filter_one_launch(fe, dims):
    nx, ny, nz = dims
    print(f"[filter] {dims}", flush=True)
    h = 1.0 / max(dims)
    gam = np.random.default_rng(5).uniform(0.0, 1.0, nx * ny * nz)
    ref = OFilter(nx, ny, nz, h, 2.5 * h)
    f = fe.Filter(nx, ny, nz, h, 2.5 * h)
    for got, want in ((f.apply(dev(gam)), ref.apply(gam)),
                      (f.apply_transpose(dev(gam)), ref.apply_transpose(gam))):
        assert f.iterations % 8 == 0 and f.iterations > 0
        assert np.abs(got.cpu().numpy() - want).max() <= 1e-10 * np.abs(want).max()
    assert float(f.apply(dev(np.zeros(nx * ny * nz))).abs().max()) == 0.0 and f.iterations == 0
    gam[0] = np.nan
    with pytest.raises(fe.FeError):
        f.apply(dev(gam))
    f.close()


# several planes per tile; 299,880 and 302,379 nodes
@pytest.mark.parametrize("dims", [(48, 48, 96), (16, 125, 139), (16, 126, 139)],
                         ids=lambda d: "x".join(map(str, d)))
def test_filter_at_the_limit(fe, dims):
    nx, ny, nz = dims
    print(f"[filter] {dims}", flush=True)
    h = 1.0 / max(dims)
    f = fe.Filter(nx, ny, nz, h, 2.5 * h)
    ones = torch.ones(nx * ny * nz, dtype=torch.float64, device="cuda")
    assert float((f.apply(ones) - 1.0).abs().max()) <= 1e-10
    rng = np.random.default_rng(6)
    u, v = (dev(rng.uniform(-1.0, 1.0, nx * ny * nz)) for _ in range(2))
    a, b = float(f.apply(u) @ v), float(u @ f.apply_transpose(v))
    assert abs(a - b) <= 1e-10 * float(u.norm() * v.norm())
    f.close()
