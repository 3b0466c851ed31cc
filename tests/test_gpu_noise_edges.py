"""White noise and the layout conversions at the edges of their blocks.

White noise against the oracle's element factors: every degree, one element per patch and more, sample counts
around the four that a wavefront keeps in flight and the tile of 64 columns (1e-13 of the largest entry: sums
of at most (p+1)^2 products per element, in another order; at degrees 4 and 5 the factor of an element
matrix of condition c is itself only determined to eps c).  The conversions transpose 64 x 64 tiles: the
operator on 1, 63, 64, 65 and 130 vectors gives each vector what it gives alone, to rounding (the launch
shape may differ), and a NaN in one vector stays in it.
"""
import numpy as np
import pytest

from oracle import assembly, noise
from paper_2605_24882_amd import inputs

pytestmark = pytest.mark.gpu

g = pytest.importorskip("paper_2605_24882_amd.gfield")


@pytest.fixture(scope="module")
def ctx():
    return g.Context(0)


@pytest.mark.parametrize("p,level,nsamp", [(1, 0, 1), (1, 3, 5), (2, 1, 3), (2, 3, 66), (3, 0, 4), (3, 2, 17), (3, 3, 130),
                                           (4, 1, 5), (5, 1, 2)])
def test_white_noise_edges(ctx, p, level, nsamp):
    sp, d = g.Space(ctx, g.Geometry(ctx, True), p, level), assembly.Discretisation(p, level, True)
    z = inputs.noise_vectors(range(nsamp), sp.noise_length)
    b, ref = sp.white_noise(z), noise.load(d, z)
    tol = 1e-13 if p <= 3 else 2.3e-16 * max(np.linalg.cond(m) for m in d.el_M)
    assert np.abs(b - ref).max() <= tol * np.abs(ref).max()
    z[0, -1] = np.nan  # the last entry of an element factors into its last function only
    bad = np.isnan(sp.white_noise(z))
    assert bad.sum() == 1 and np.array_equal(bad, np.isnan(noise.load(d, z)) & bad)


@pytest.mark.parametrize("nvec", [1, 63, 64, 65, 130])
def test_layout_conversions(ctx, nvec):
    sp = g.Space(ctx, g.Geometry(ctx, False), 2, 2)
    x = np.random.default_rng(nvec).standard_normal((nvec, sp.ndofs))
    y = sp.apply(3.0, 1.0, x)
    for v in {0, nvec // 2, nvec - 1}:
        ref = sp.apply(3.0, 1.0, x[v:v + 1])
        assert np.abs(y[v] - ref[0]).max() <= 1e-13 * np.abs(ref).max()
    x[nvec - 1, 5] = np.nan
    y2 = sp.apply(3.0, 1.0, x)
    assert np.isnan(y2[nvec - 1]).any() and np.array_equal(y2[:nvec - 1], y[:nvec - 1])


@pytest.mark.parametrize("surface,p,level,mg", [("sphere", 1, 1, 0), ("torus", 2, 1, 0), ("torus", 3, 1, 0),
                                                ("sphere", 2, 3, 1)])
def test_coarse_inverse_sizes(ctx, surface, p, level, mg):
    """Dense solves of 8, 64, 144 and 488 unknowns (the last above the one-launch factorisation): the residual
    of every shift, taken with the sum-factorised operator, is the solver's (1e-11) to rounding."""
    geo = g.Geometry.nurbs(ctx, *inputs.torus_patches()) if surface == "torus" else g.Geometry(ctx, True)
    sp = g.Space(ctx, geo, p, level, mg_levels=mg)
    sigma = np.array([2.0, 40.0, 900.0])
    b = np.random.default_rng(0).standard_normal((3, sp.ndofs))
    x, st = sp.solve_shifted(sigma, b, rtol=1e-11)
    for s, xi, bi in zip(sigma, x, b):
        r = bi - sp.apply(s, 1.0, xi, kind=g.GF_APPLY_SUMFACT)
        assert np.linalg.norm(r) <= 1e-10 * np.linalg.norm(bi)
    assert mg != 1 or st["max_iters"] <= 2
