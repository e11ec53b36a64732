"""The density filter's right-hand sides that end a solve at its first look: zero, not
finite, and so small that the squared residual has no range left below it.

A field of 1e-158 gives <r, r> of some 1e-314: rtol^2 = 1e-24 times that is no double, and
the terms of <r, r> underflow before the field is solved (a field 6e-3 off at 1e-160 once
passed as converged).  Such a solve is refused as not converged; a field whose <r, r>
itself is zero is the zero field.
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def fe():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1508_04596_amd import fe as fe_mod
    fe_mod.lib()
    return fe_mod


# one launch per iteration; two
@pytest.mark.parametrize("dims", [(16, 16, 16), (60, 70, 80)], ids=lambda d: "x".join(map(str, d)))
def test_first_look(fe, dims):
    print(f"[filter] {dims}", flush=True)
    n = dims[0] * dims[1] * dims[2]
    f = fe.Filter(*dims, 1.0, 2.5)
    e = torch.from_numpy(np.random.default_rng(9).uniform(0.5, 1.0, n)).cuda()
    for apply in (f.apply, f.apply_transpose):
        for scale in (0.0, 1e-170):
            assert float(apply(scale * e).abs().max()) == 0.0 and f.iterations == 0
        for scale in (1e-158, 1e-160):
            with pytest.raises(fe.FeError, match="not converged"):
                apply(scale * e)
        for bad in (float("nan"), float("inf"), 1e160):
            g = e.clone()
            g[n // 2] = bad
            with pytest.raises(fe.FeError, match="non-finite"):
                apply(g)
        # the solves after those are as before them; the scale down to 1e-140 takes no part
        want = apply(e)
        assert f.iterations > 0
        assert float((apply(1e-140 * e) * 1e140 - want).abs().max()) <= 1e-10
    f.close()
