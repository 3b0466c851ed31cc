"""How a mixed-precision solve stores its search direction does not hang on the value of a shift.

Two iterations on 18 columns (the last group of 16 is completed by padding), once with the shift 1 and once with
the next larger double.  The single-precision preconditioner sees the same shift, the operator one that
differs by 2e-16, so the two results differ by some 1e-15 relative; a direction rounded to single precision in
one of them alone would leave 6e-8 of the second step, far above the bound of 1e-12.
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

g = pytest.importorskip("paper_2605_24882_amd.gfield")


@pytest.mark.parametrize("ncols", [18, 32])
def test_direction_storage_does_not_depend_on_the_shift(ncols, monkeypatch):
    monkeypatch.setenv("GF_APPLY_SHAPE", "2,32")
    ctx = g.Context(0)
    sp = g.Space(ctx, g.Geometry(ctx, False), 2, 5)
    b = np.random.default_rng(2).standard_normal((ncols, sp.ndofs))
    kw = dict(precision=g.GF_PREC_MIXED, cheb_degree=1, rtol=3e-2)
    x, st = sp.solve_shifted(1.0, b, **kw)
    y, su = sp.solve_shifted(np.nextafter(1.0, 2.0), b, **kw)
    assert 2 <= st["max_iters"] <= 4 and st["max_iters"] == su["max_iters"], (st["max_iters"], su["max_iters"])
    assert np.abs(x - y).max() <= 1e-12 * np.abs(x).max()
