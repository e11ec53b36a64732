"""The density filter at the edges of its tiling (tiles of up to 40 x 128 nodes,
at least two planes): one element, one full and one just overflowing tile width,
thin and long grids, a zero field, and the iteration count's multiple of eight.

CG stops at a relative residual of 1e-12 with a condition number below 100, so the
fields agree with exact sparse solves to 1e-10 of the largest entry.
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


DIMS = [(1, 1, 1), (39, 3, 2), (40, 5, 1), (2, 130, 4), (81, 7, 19), (5, 1, 67)]


@pytest.mark.parametrize("dims", DIMS, ids=["x".join(map(str, d)) for d in DIMS])
def test_filter_at_tile_edges(fe, dims):
    nx, ny, nz = dims
    print(f"[filter] {dims}", flush=True)
    h = 1.0 / max(dims)
    gam = np.random.default_rng(3).uniform(0.0, 1.0, nx * ny * nz)
    ref = OFilter(nx, ny, nz, h, 2.5 * h)
    f = fe.Filter(nx, ny, nz, h, 2.5 * h)
    for got, want in ((f.apply(dev(gam)), ref.apply(gam)),
                      (f.apply_transpose(dev(gam)), ref.apply_transpose(gam))):
        assert f.iterations % 8 == 0 and f.iterations > 0
        assert np.abs(got.cpu().numpy() - want).max() <= 1e-10 * np.abs(want).max()
    zero = f.apply(dev(np.zeros(nx * ny * nz)))
    assert f.iterations == 0 and float(zero.abs().max()) == 0.0
    f.close()
