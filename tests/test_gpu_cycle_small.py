"""The smallest spaces whose whole V-cycle is one launch: 2 x 2 elements per patch.

One application of both forms of the preconditioner (a solve that stops after its first iteration returns a
multiple of it) agrees to rounding: some ten operator applications of at most 49 terms, below 1e-5 relative in
single and 1e-13 in double precision.  The numbers of iterations are no measure here: on 56 to 98 unknowns the
conjugate gradients end when the Krylov space does, and how soon depends on the rounding of the preconditioner
(degree 2, single precision, one smoothing step, to 1e-11: 28 iterations against 26; with every step launched
separately the two operator kinds differ as much).  The solutions agree as for larger spaces.
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

g = pytest.importorskip("paper_2605_24882_amd.gfield")


@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("p", [1, 2, 3])
@pytest.mark.parametrize("deg", [1, 4])
def test_level_one(p, deg, prec):
    ctx = g.Context(0)
    sp = g.Space(ctx, g.Geometry(ctx, False), p, 1)
    rng = np.random.default_rng(1)
    for sigma in (np.repeat([30.0, 900.0], 16), np.array([1.0, 7.0, 50.0, 7.0, 1.0, 400.0, 2e4])):
        b = rng.standard_normal((len(sigma), sp.ndofs))

        def both(rtol):
            return [sp.solve_shifted(sigma, b, precision=prec, rtol=rtol, cheb_degree=deg, apply_kind=kind)
                    for kind in (g.GF_APPLY_STENCIL, g.GF_APPLY_SUMFACT)]

        (x, st), (y, su) = both(0.999)
        assert st["max_iters"] == su["max_iters"] == 1
        assert np.abs(x - y).max() <= (1e-5 if prec else 1e-13) * np.abs(y).max()
        (x, _), (y, _) = both(1e-11)
        err = np.linalg.norm(x - y, axis=1) / np.linalg.norm(y, axis=1)
        assert err.max() <= 4e-11 * np.sqrt(sp.ndofs), err
