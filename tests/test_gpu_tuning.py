"""What the library times on a space's first calls, read from its own log (GF_TUNE_LOG).

The launch shape of the smoothing step is timed on a step that reads the iterate and the right-hand side, between
the steps that read less and those that read more.  The smoothing degree is kept for batches of one width, number
of shifts, distribution of the shifts over the columns and powers of two of the extreme shifts; a call with the
degree of an earlier one gives the same solution to the solver's tolerance, and with a given degree the same bits.
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

g = pytest.importorskip("paper_2605_24882_amd.gfield")


@pytest.fixture(scope="module")
def ctx():
    return g.Context(0)


def tuned(capfd, what):
    return [line for line in capfd.readouterr().err.splitlines() if line.startswith(what)]


@pytest.mark.parametrize("prec", [0, 1])
def test_smoothing_shape_is_timed_on_a_step_with_a_right_hand_side(ctx, prec, capfd, monkeypatch):
    monkeypatch.setenv("GF_TUNE_LOG", "1")
    sp = g.Space(ctx, g.Geometry(ctx, False), 2, 5)
    b = np.random.default_rng(1).standard_normal((64, sp.ndofs))
    sp.solve_shifted(30.0, b, precision=prec, cheb_degree=4)
    lines = [x for x in tuned(capfd, "tune p=") if f"lev=5 T={4 if prec else 8} " in x and "kind=1 " in x]
    assert lines and all("step=5 " in x for x in lines), lines


def test_degree_is_timed_for_each_distribution_of_the_shifts(ctx, capfd, monkeypatch):
    monkeypatch.setenv("GF_TUNE_LOG", "1")
    sp = g.Space(ctx, g.Geometry(ctx, False), 2, 6)
    n = 448  # 448 x 25,352 unknowns: above the smallest batch that is timed
    b = np.random.default_rng(1).standard_normal((n, sp.ndofs))
    low = np.where(np.arange(n) < n - 16, 2.0, 1e6)
    high = np.where(np.arange(n) < 16, 2.0, 1e6)
    for sigma in (low, high):
        sp.solve_shifted(sigma, b, rtol=1e-6)
        assert tuned(capfd, "degree tune"), sigma
    sp.solve_shifted(1.01 * low, b, rtol=1e-6)
    assert not tuned(capfd, "degree tune")


def test_degree_of_an_earlier_call_keeps_the_tolerance(ctx, monkeypatch):
    monkeypatch.setenv("GF_APPLY_SHAPE", "2,32")
    rtol = 1e-10
    sp, fresh = (g.Space(ctx, g.Geometry(ctx, False), 2, 6) for _ in range(2))
    b = np.random.default_rng(1).standard_normal((20, sp.ndofs))
    kw = dict(k_minus=20, k_plus=20, rtol=rtol)
    for deg in (0, 3):
        sp.sample(15.0, 0.75, b, cheb_degree=deg, **kw)
        u, _ = sp.sample(12.0, 0.75, b, cheb_degree=deg, **kw)
        v, _ = fresh.sample(12.0, 0.75, b, cheb_degree=deg, **kw)
        if deg:
            assert np.array_equal(u, v)
        # every node's solution is within rtol sqrt(N) of the exact one, relative, and the weights are positive
        err = np.linalg.norm(u - v, axis=1) / np.linalg.norm(v, axis=1)
        assert err.max() <= 4 * rtol * np.sqrt(sp.ndofs), err
