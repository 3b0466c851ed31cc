"""Shared unknowns inside the strips' launch (strips of one or two rows) against the interface kernel after it
(strips of four rows, and the sum-factorised kind).

The operator: a value is a sum of (2p + 1)^2 products per copy, rounded within (2p + 1)^2 eps of the sum of
their sizes, which for Gaussian vectors is within some ten times the largest value: 121 x 1.1e-16 x 10
is below 1e-12 (the sum-factorised kind sums over quadrature points, no more terms than that per
direction).  The solves: the same preconditioner up to rounding, so as many iterations (one more or
fewer, and one per cent of them), and each solution within rtol sqrt(N) of the exact one, relative; twice
that for the two, twice again for the spread of the load.
"""
import numpy as np
import pytest

from paper_2605_24882_amd import inputs

pytestmark = pytest.mark.gpu

g = pytest.importorskip("paper_2605_24882_amd.gfield")


@pytest.fixture(scope="module")
def ctx():
    return g.Context(0)


@pytest.mark.parametrize("surface,p,level", [("sphere", 1, 3), ("perturbed", 2, 4), ("sphere", 3, 3), ("torus", 2, 2),
                                             ("open", 3, 3), ("sphere", 4, 3), ("sphere", 5, 3)])
def test_interface_blocks_match_interface_kernel(ctx, monkeypatch, surface, p, level):
    if surface == "torus":
        geo = g.Geometry.nurbs(ctx, *inputs.torus_patches())
    elif surface == "open":
        from .open_surfaces import strip
        geo = g.Geometry.nurbs(ctx, *strip())
    else:
        geo = g.Geometry(ctx, surface == "perturbed")
    rng = np.random.default_rng(2)
    ref = g.Space(ctx, geo, p, level)
    for n in (1, 70):
        x = rng.standard_normal((n, ref.ndofs))
        y = ref.apply(9.0, 1.0, x, kind=g.GF_APPLY_SUMFACT)
        sigma = np.full(n, 30.0) if n == 1 else np.resize([1.0, 7.0, 900.0], n)  # one shift; lanes that differ
        u, su = ref.solve_shifted(sigma, x, apply_kind=g.GF_APPLY_SUMFACT, rtol=1e-11, cheb_degree=3, max_iter=3000)
        for shape in ("1,32", "2,64", "4,32"):
            monkeypatch.setenv("GF_APPLY_SHAPE", shape)
            sp = g.Space(ctx, geo, p, level)
            assert np.abs(sp.apply(9.0, 1.0, x) - y).max() <= 1e-12 * np.abs(y).max()
            for prec in (0, 1):
                v, st = sp.solve_shifted(sigma, x, precision=prec, rtol=1e-11, cheb_degree=3, max_iter=3000)
                if prec == 0:
                    assert abs(st["max_iters"] - su["max_iters"]) <= 1 + 0.01 * su["max_iters"], (st, su)
                err = np.linalg.norm(u - v, axis=1) / np.linalg.norm(u, axis=1)
                assert err.max() <= 4e-11 * np.sqrt(sp.ndofs), (shape, prec, err)
            monkeypatch.delenv("GF_APPLY_SHAPE")
