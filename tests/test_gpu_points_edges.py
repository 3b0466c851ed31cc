"""Point evaluation and its transpose at the edges of their point lists.

All points in one element, points repeated, on element borders and patch corners, no point in most elements,
point and vector counts around the blocks' 64, 256 and 1024 and the transpose's eight vectors: against the
oracle's sparse Phi, to 1e-13 of the largest entry times the points that meet in a coefficient (sums in
another order).  Out-of-range points are refused on device arrays as on host arrays.
"""
import numpy as np
import pytest

from oracle import assembly, evaluate

pytestmark = pytest.mark.gpu

g = pytest.importorskip("paper_2605_24882_amd.gfield")


@pytest.fixture(scope="module")
def ctx():
    return g.Context(0)


@pytest.mark.parametrize("p,level,npts,nvec,where", [
    (1, 0, 1, 1, "any"), (2, 2, 65, 9, "any"), (3, 3, 1025, 8, "any"), (3, 2, 700, 17, "one"), (2, 3, 257, 3, "grid"),
    (4, 1, 300, 5, "grid"), (5, 2, 90, 7, "any"), (2, 5, 40, 2, "one")])
def test_points(ctx, p, level, npts, nvec, where):
    import torch
    sp, d = g.Space(ctx, g.Geometry(ctx, True), p, level), assembly.Discretisation(p, level, True)
    rng = np.random.default_rng(npts)
    patch, st = rng.integers(0, 6, npts).astype(np.int32), rng.random((npts, 2))
    if where == "one":
        patch[:], st = 3, st * 0.5 ** level
        st[::3] = st[0]
    if where == "grid":  # element borders, patch edges and corners
        st = rng.integers(0, 2 ** level + 1, (npts, 2)) / 2 ** level
    Phi = evaluate.phi_matrix(d, patch, st[:, 0], st[:, 1])
    u, r = rng.standard_normal((nvec, d.N)), rng.standard_normal((nvec, npts))
    ref, back = (Phi @ u.T).T, (Phi.T @ r.T).T
    meet = max(1, int(np.diff(Phi.tocsc().indptr).max()))
    dev = [torch.from_numpy(a).cuda() for a in (patch, st, u, r)]
    for vals, out in ((sp.eval(patch, st, u), sp.eval_adjoint(patch, st, r)),
                      (sp.eval(*dev[:3]).cpu().numpy(), sp.eval_adjoint(dev[0], dev[1], dev[3]).cpu().numpy())):
        assert np.abs(vals - ref).max() <= 1e-13 * np.abs(u).max()
        assert np.abs(out - back).max() <= 1e-13 * np.abs(r).max() * meet
    for bad in ("patch", "st"):
        pb, sb = patch.copy(), st.copy()
        if bad == "patch":
            pb[-1] = 6
        else:
            sb[-1, 1] = np.nan
        for mk in (lambda a: a, lambda a: torch.from_numpy(a).cuda()):
            for f, x in ((sp.eval, u), (sp.eval_adjoint, r)):
                with pytest.raises(g.GfieldError) as e:
                    f(mk(pb), mk(sb), mk(x))
                assert e.value.status == g.GF_EINVAL
