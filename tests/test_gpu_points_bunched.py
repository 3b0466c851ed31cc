"""The transpose of point evaluation where many points meet in few coefficients of a large mesh.

Against the oracle's sparse Phi, to 1e-13 of the largest entry times the points that meet in a coefficient (sums
in another order): point counts around a wavefront's 64 lanes in one element, in neighbouring elements, on a patch
corner, beside points spread over the mesh; fewer points than elements.  The same bits on a second call.  And in
time: bunched points may take 30 times as long as spread ones (a coefficient's thread walking all of them
alone takes longer than that at 20000).
"""
import time

import numpy as np
import pytest

from oracle import assembly, evaluate

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

g = pytest.importorskip("paper_2605_24882_amd.gfield")


@pytest.fixture(scope="module")
def ctx():
    return g.Context(0)


@pytest.mark.parametrize("p,level,bunch,spread,nvec,where", [
    (1, 5, 63, 0, 1, "element"), (1, 5, 700, 40, 3, "corner"), (2, 4, 130, 300, 8, "element"), (2, 5, 3000, 1, 9, "elements"),
    (3, 5, 1000, 500, 1, "corner"), (3, 4, 1000, 0, 17, "elements"), (4, 4, 257, 5, 2, "corner"), (5, 4, 129, 0, 4, "element")])
def test_bunched_points(ctx, p, level, bunch, spread, nvec, where):
    sp, d = g.Space(ctx, g.Geometry(ctx, True), p, level), assembly.Discretisation(p, level, True)
    rng = np.random.default_rng(bunch)
    n = bunch + spread
    assert n < 6 * 4 ** level
    patch, st, h = rng.integers(0, 6, n).astype(np.int32), rng.random((n, 2)), 0.5 ** level
    here = rng.permutation(n)[:bunch]
    if where == "corner":
        patch[here], st[here] = 2, 1.0 - h * st[here]
        st[here[:5]] = 1.0
    else:
        patch[here], st[here] = 4, h * (3 + (1 if where == "element" else 5) * st[here])
    Phi = evaluate.phi_matrix(d, patch, st[:, 0], st[:, 1])
    r = rng.standard_normal((nvec, n))
    back = (Phi.T @ r.T).T
    meet = int(np.diff(Phi.tocsc().indptr).max())
    out = sp.eval_adjoint(patch, st, r)
    assert np.abs(out - back).max() <= 1e-13 * np.abs(r).max() * meet
    assert np.array_equal(sp.eval_adjoint(patch, st, r), out)


@pytest.mark.parametrize("nvec", [1, 16])
def test_bunched_points_in_time(ctx, nvec):
    sp, n = g.Space(ctx, g.Geometry(ctx, False), 3, 6), 20000
    rng = np.random.default_rng(1)
    st = rng.random((n, 2))
    r = torch.from_numpy(rng.standard_normal((nvec, n))).cuda()

    def seconds(patch, st):
        patch, st = torch.from_numpy(patch.astype(np.int32)).cuda(), torch.from_numpy(st).cuda()
        best = 1e30
        for _ in range(5):
            t = time.perf_counter()
            sp.eval_adjoint(patch, st, r)
            best = min(best, time.perf_counter() - t)
        return best

    spread, bunched = seconds(rng.integers(0, 6, n), st), seconds(np.full(n, 2), (3 + st) / 64)
    print(f"{n} points of {nvec}: spread {spread * 1e3:.3f} ms, in one element {bunched * 1e3:.3f} ms")
    assert bunched <= 30 * spread
