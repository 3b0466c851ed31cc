"""What calls reuse -- blocks of device memory, captured graphs -- carries nothing from one call to the next.

Every call of a sequence on one context (blocks handed from call to call, graphs replayed for another
kappa, memory that held NaN) gives bit for bit what the same call gives as the first one on a context
and space of its own: the same kernels run on the same columns in the same order.  The launch shape is
fixed, because every space times its own, and the shape decides how an inner product is split into
partial sums.
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

g = pytest.importorskip("paper_2605_24882_amd.gfield")


def calls(sp, rng):
    """(name, call) of every entry point that takes blocks from the pool, inputs drawn from rng"""
    b = rng.standard_normal((5, sp.ndofs))
    z = rng.standard_normal((5, sp.noise_length))
    patch, st = rng.integers(0, 6, 40).astype(np.int32), rng.random((40, 2))
    r = rng.standard_normal((5, 40))
    kw = dict(k_minus=6, k_plus=6, rtol=1e-10)

    def tape(kappa):
        u, t, _ = sp.sample_tape(kappa, 1.6, b, precision=1, **kw)
        return np.concatenate([u.reshape(-1), t.grad_kappa(b)[0]])

    yield "apply", lambda: sp.apply(2.0, 1.0, b)
    yield "sumfact", lambda: sp.apply(2.0, 1.0, b, kind=g.GF_APPLY_SUMFACT)
    yield "noise", lambda: sp.white_noise(z)
    for i, kappa in enumerate((3.0, 7.0, 3.0, 4.5)):  # one graph, four sets of shifts
        yield f"sample{i}", lambda kappa=kappa: sp.sample(kappa, 0.6, b, precision=i % 2, **kw)[0]
    yield "two passes", lambda: sp.sample(3.0, 1.2, b, split=g.GF_SPLIT_IMPROVED, **kw)[0]
    yield "tape", lambda: tape(5.0)
    yield "tape2", lambda: tape(6.0)
    yield "eval", lambda: sp.eval(patch, st, b)
    yield "eval_adjoint", lambda: sp.eval_adjoint(patch, st, r)
    yield "sqrt", lambda: sp.sqrt_mass(b, khat=6)[0]
    yield "prolong", lambda: sp.transfer(sp.level, g.GF_PROLONG, np.ones((3, coarse(sp))), sp.ndofs)
    yield "restrict", lambda: sp.transfer(sp.level, g.GF_RESTRICT, b, coarse(sp))


def coarse(sp):
    n = 2 ** (sp.level - 1) + sp.degree
    return 6 * (n - 2) ** 2 + 12 * (n - 2) + 8


@pytest.mark.parametrize("p,level", [(2, 3), (3, 4)])
def test_calls_are_independent_of_earlier_calls(p, level, monkeypatch):
    monkeypatch.setenv("GF_APPLY_SHAPE", "2,32")
    ctx = g.Context(0)
    sp = g.Space(ctx, g.Geometry(ctx, True), p, level)
    nan = np.full((70, sp.ndofs), np.nan)
    names = [n for n, _ in calls(sp, np.random.default_rng(0))]
    for k, name in enumerate(names):
        for n in (5, 70):  # the blocks of the next call have held NaN
            sp.apply(1.0, 1.0, nan[:n])
            sp.white_noise(np.full((n, sp.noise_length), np.nan))
        got = dict(calls(sp, np.random.default_rng(0)))[name]()
        ctx1 = g.Context(0)
        sp1 = g.Space(ctx1, g.Geometry(ctx1, True), p, level)
        ref = dict(calls(sp1, np.random.default_rng(0)))[name]()
        assert np.array_equal(got, ref), name
