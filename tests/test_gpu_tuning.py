"""What the library times on a space's first calls, read from its own log (GF_TUNE_LOG).

The launch shape of the smoothing step is timed on a step that reads the iterate and the right-hand side, between
the steps that read less and those that read more.
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
