"""Reductions over batches whose last tile has few columns: their partial sums are shared out among the lanes.

Every column of a batch is the same system as in a batch of 64, up to the order of its sums: the two
solutions are within rtol sqrt(N) of the exact one each, relative (the load is Gaussian: |x| is at
least its share of the lowest eigenvector), twice that again for the spread of the load.  A repeated call gives the
same bits.
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

g = pytest.importorskip("paper_2605_24882_amd.gfield")


@pytest.mark.parametrize("n", [1, 2, 3, 16, 17, 32, 33, 63, 65, 80])
@pytest.mark.parametrize("prec", [0, 1])
def test_column_counts(n, prec):
    ctx = g.Context(0)
    sp = g.Space(ctx, g.Geometry(ctx, False), 2, 4)
    b = np.random.default_rng(8).standard_normal((128, sp.ndofs))
    kw = dict(precision=prec, rtol=1e-11)
    ref = np.concatenate([sp.solve_shifted(30.0, b[i:i + 64], **kw)[0] for i in (0, 64)])[:n]
    x, _ = sp.solve_shifted(30.0, b[:n], **kw)
    again, _ = sp.solve_shifted(30.0, b[:n], **kw)
    err = np.linalg.norm(x - ref, axis=1) / np.linalg.norm(ref, axis=1)
    assert err.max() <= 4e-11 * np.sqrt(sp.ndofs), err
    assert np.array_equal(x, again)
