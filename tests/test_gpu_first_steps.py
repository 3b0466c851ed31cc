"""The two smoothing steps after the start from zero, which take the right-hand side or the previous iterate
from z1 = c r / D in the combined-stencil kernel, against the sum-factorised kind, which reads both.

Both are the same preconditioner up to rounding, so the conjugate gradients need the same number of
iterations (one more or fewer when a residual lies at the threshold, and one per cent of them), and each
solution is within rtol sqrt(N) of the exact one, relative (the load is Gaussian: |x| is at least its share of the
lowest eigenvector), the two within twice that, taken twice again for the spread of the load.
Two steps end with the first of them, three with the second, sixteen is the most.
"""
import numpy as np
import pytest

from paper_2605_24882_amd import inputs

pytestmark = pytest.mark.gpu

g = pytest.importorskip("paper_2605_24882_amd.gfield")


@pytest.fixture(scope="module")
def ctx():
    return g.Context(0)


@pytest.mark.parametrize("deg", [2, 3, 16])
@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("surface,p,level", [("sphere", 1, 4), ("torus", 2, 3), ("perturbed", 3, 5)])
def test_first_steps_match_sum_factorised_kind(ctx, surface, p, level, prec, deg):
    geo = g.Geometry.nurbs(ctx, *inputs.torus_patches()) if surface == "torus" else g.Geometry(ctx, surface == "perturbed")
    sp = g.Space(ctx, geo, p, level)
    rng = np.random.default_rng(deg)
    # one shift for a group of 16 columns, then shifts that differ lane by lane, with padding columns
    for sigma in (np.repeat([30.0, 900.0], 16), np.array([1.0, 7.0, 50.0, 7.0, 1.0, 400.0, 2e4])):
        b = rng.standard_normal((len(sigma), sp.ndofs))
        (x, st), (y, su) = (sp.solve_shifted(sigma, b, precision=prec, rtol=1e-11, cheb_degree=deg, apply_kind=kind,
                                             max_iter=3000)
                            for kind in (g.GF_APPLY_STENCIL, g.GF_APPLY_SUMFACT))
        assert abs(st["max_iters"] - su["max_iters"]) <= 1 + 0.01 * su["max_iters"], (st, su)
        err = np.linalg.norm(x - y, axis=1) / np.linalg.norm(y, axis=1)
        assert err.max() <= 4e-11 * np.sqrt(sp.ndofs), err
