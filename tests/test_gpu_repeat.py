"""The first call on a space gives bit for bit what the second one gives (the sums of a reduction are split the
same way from the first call on).  The launch shape is fixed: timing it is part of a space's first calls."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

g = pytest.importorskip("paper_2605_24882_amd.gfield")


@pytest.mark.parametrize("p,level", [(1, 3), (2, 3), (2, 4), (3, 4), (2, 5), (3, 5)])
def test_sqrt_mass_repeats_its_first_result(p, level, monkeypatch):
    monkeypatch.setenv("GF_APPLY_SHAPE", "2,32")
    ctx = g.Context(0)
    sp = g.Space(ctx, g.Geometry(ctx, True), p, level)
    y = np.random.default_rng(p + level).standard_normal((3, sp.ndofs))
    first = sp.sqrt_mass(y, khat=6)[0]
    for _ in range(2):
        assert np.array_equal(sp.sqrt_mass(y, khat=6)[0], first)
