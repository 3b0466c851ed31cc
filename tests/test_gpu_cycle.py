"""The coarsest levels of the V-cycle in one launch against the same steps launched one by one.

The sum-factorised operator kind runs every level by separate launches; the stencil kind runs the
levels that fit a block's LDS in one.  Both are the same preconditioner up to rounding (1e-7 relative in
single precision), so the conjugate gradients need the same number of iterations (one more or fewer
when a residual lies at the threshold, and as many per cent over the hundreds of iterations that a
single smoothing step leaves at degrees 4 and 5) and give the same solutions.  For a Gaussian load b the solution
has |x| >= |b| / (lambda_min sqrt(N)) or so (its share of the lowest eigenvector), and a residual of rtol |b|
leaves an error of at most rtol |b| / lambda_min: each solve is within rtol sqrt(N) of the exact one,
relative, and the two within twice that (taken twice again for the spread of the load).
"""
import numpy as np
import pytest

from paper_2605_24882_amd import inputs

pytestmark = pytest.mark.gpu

g = pytest.importorskip("paper_2605_24882_amd.gfield")


@pytest.fixture(scope="module")
def ctx():
    return g.Context(0)


@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("surface,p,level,mg_levels", [
    ("sphere", 1, 1, 0),   # the dense solve alone below the finest level
    ("sphere", 1, 5, 0),
    ("sphere", 2, 4, 0),
    ("perturbed", 3, 4, 0),
    ("sphere", 3, 4, 2),   # a coarsest level of 726 patch coefficients (above the dense solve's staging)
    ("sphere", 4, 3, 0),
    ("sphere", 5, 3, 0),
    ("torus", 2, 3, 0),
    ("open", 2, 3, 0),     # boundary unknowns with a single copy
])
def test_one_launch_cycle_matches_separate_launches(ctx, surface, p, level, mg_levels, prec):
    if surface == "torus":
        geo = g.Geometry.nurbs(ctx, *inputs.torus_patches())
    elif surface == "open":
        from .open_surfaces import strip
        geo = g.Geometry.nurbs(ctx, *strip())
    else:
        geo = g.Geometry(ctx, surface == "perturbed")
    sp = g.Space(ctx, geo, p, level, mg_levels=mg_levels)
    rng = np.random.default_rng(1)
    # one shift for a group of 16 columns (32 columns of two shifts), then shifts that differ lane by lane, with
    # a partly filled last group and the padding's own shift 1 among them
    for sigma in (np.repeat([30.0, 900.0], 16), np.array([1.0, 7.0, 50.0, 7.0, 1.0, 400.0, 2e4])):
        b = rng.standard_normal((len(sigma), sp.ndofs))
        out = [sp.solve_shifted(sigma, b, precision=prec, rtol=1e-11, cheb_degree=deg, apply_kind=kind,
                                max_iter=3000)
               for deg in (1, 4) for kind in (g.GF_APPLY_STENCIL, g.GF_APPLY_SUMFACT)]
        for (x, st), (y, su) in (out[:2], out[2:]):
            assert abs(st["max_iters"] - su["max_iters"]) <= 1 + 0.01 * su["max_iters"], (st, su)
            err = np.linalg.norm(x - y, axis=1) / np.linalg.norm(y, axis=1)
            assert err.max() <= 4e-11 * np.sqrt(sp.ndofs), err


@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("surface,p,level", [("sphere", 1, 3), ("perturbed", 2, 2), ("sphere", 3, 2), ("torus", 1, 2),
                                             ("torus", 2, 2), ("open", 2, 2)])
def test_whole_cycle_in_one_launch_matches_separate_launches(ctx, surface, p, level, prec):
    # the smallest spaces, finest level included
    test_one_launch_cycle_matches_separate_launches(ctx, surface, p, level, 0, prec)


@pytest.mark.parametrize("level", [2, 4])
@pytest.mark.parametrize("prec", [0, 1])
def test_columns_without_load_stay_zero_after_a_batch_that_was_not_finite(ctx, prec, level):
    # sixteen columns without a load take no part in the coarse cycle; what an earlier batch left in its
    # buffers (here NaN, beside one column that is solved) must not reach their solutions
    sp = g.Space(ctx, g.Geometry(ctx, False), 2, level)
    b = np.random.default_rng(5).standard_normal((20, sp.ndofs))
    bad = b.copy()
    bad[:15] = np.nan
    with pytest.raises(RuntimeError):
        sp.solve_shifted(30.0, bad, precision=prec)
    ref, _ = sp.solve_shifted(30.0, b, precision=prec)
    with pytest.raises(RuntimeError):
        sp.solve_shifted(30.0, bad, precision=prec)
    b[:16] = 0.0
    x, _ = sp.solve_shifted(30.0, b, precision=prec)
    assert not x[:16].any()
    assert np.abs(x[16:] - ref[16:]).max() <= 1e-9 * np.abs(ref[16:]).max()
