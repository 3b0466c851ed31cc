"""Columns with shifts of their own in every launch shape of the stencil kernel.

Seven shifts in seven columns (no aligned group of 16 shares one) and 18 columns of one shift (the last group
of 16 is completed by padding), strips of one, two and four rows.  The residual of every system is taken with
the sum-factorised operator, which shares no kernel with the stencils: it may exceed the solver's 1e-11 by the
rounding of the operator on the solution, eps |A| |x| / |b| <= eps cond(A) ~ 2e-16 x 1e5, in all 1e-10.
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

g = pytest.importorskip("paper_2605_24882_amd.gfield")


@pytest.fixture(scope="module")
def ctx():
    return g.Context(0)


@pytest.mark.parametrize("shape", ["1,16", "2,32", "4,64"])
@pytest.mark.parametrize("p,level,prec", [(1, 4, 0), (2, 4, 1), (3, 4, 0), (3, 4, 1), (4, 3, 0), (5, 3, 1)])
def test_shifts_per_column(ctx, p, level, prec, shape, monkeypatch):
    monkeypatch.setenv("GF_APPLY_SHAPE", shape)
    sp = g.Space(ctx, g.Geometry(ctx, True), p, level)
    rng = np.random.default_rng(p)
    for sigma in (np.array([9.0, 30.0, 1.0, 400.0, 50.0, 120.0, 77.0]), np.full(18, 40.0)):
        b = rng.standard_normal((len(sigma), sp.ndofs))
        x, _ = sp.solve_shifted(sigma, b, precision=prec, rtol=1e-11, max_iter=2000)
        for s, xi, bi in zip(sigma, x, b):
            r = bi - sp.apply(s, 1.0, xi, kind=g.GF_APPLY_SUMFACT)
            assert np.linalg.norm(r) <= 1e-10 * np.linalg.norm(bi), (s, np.linalg.norm(r) / np.linalg.norm(bi))
