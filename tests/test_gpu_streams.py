"""Inputs that another stream is still writing when the call begins.

The library works on its context's stream; a caller's tensors may come from any other stream of the device (a
program under torch.cuda.stream, an autograd backward).  Every call waits for them: its result is bit for
bit that of the same call on finished inputs.  The input here is copied into place behind some 50 ms of
other work, and holds other finite values until then.
"""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
from paper_2605_24882_amd import gfield as g  # noqa: E402

pytestmark = pytest.mark.gpu


def late(good):
    """A tensor that becomes `good` on a side stream, after a while."""
    x = torch.zeros_like(good)
    busy = torch.ones(1 << 27, dtype=torch.float32, device="cuda")
    side = torch.cuda.Stream()
    torch.cuda.synchronize()
    with torch.cuda.stream(side):
        for _ in range(200):
            busy.mul_(1.0)  # half a gigabyte read and written
        x.copy_(good)
    return x, busy


def test_calls_wait_for_their_inputs(monkeypatch):
    monkeypatch.setenv("GF_APPLY_SHAPE", "2,32")
    ctx = g.Context(0)
    sp = g.Space(ctx, g.Geometry(ctx, False), 2, 4)
    gen = torch.Generator(device="cuda").manual_seed(3)
    v = torch.randn(5, sp.ndofs, dtype=torch.float64, device="cuda", generator=gen)
    z = torch.randn(5, sp.noise_length, dtype=torch.float64, device="cuda", generator=gen)
    r = torch.randn(5, 40, dtype=torch.float64, device="cuda", generator=gen)
    rng = np.random.default_rng(4)
    patch = torch.from_numpy(rng.integers(0, 6, 40).astype(np.int32)).cuda()
    st = torch.from_numpy(rng.random((40, 2))).cuda()
    n = 6 * 8 ** 2 + 12 * 8 + 8  # unknowns of the next coarser level
    kw = dict(k_minus=6, k_plus=6, rtol=1e-10, cheb_degree=3)
    u, tape, _ = sp.sample_tape(4.0, 1.6, v, **kw)
    calls = {
        "apply": (v, lambda x: sp.apply(2.0, 1.0, x)),
        "transfer": (v, lambda x: sp.transfer(4, g.GF_RESTRICT, x, n)),
        "white_noise": (z, lambda x: sp.white_noise(x)),
        "eval": (v, lambda x: sp.eval(patch, st, x)),
        "eval at late points": (st, lambda x: sp.eval(patch, x, v)),
        "eval_adjoint": (r, lambda x: sp.eval_adjoint(patch, st, x)),
        "sqrt_mass": (v, lambda x: sp.sqrt_mass(x, khat=6, lo=1e-4, hi=1.0)[0]),
        "sample": (v, lambda x: sp.sample(4.0, 0.6, x, **kw)[0]),
        "sample, integer": (v, lambda x: sp.sample(4.0, 1.0, x, **kw)[0]),
        "batch": (v, lambda x: g.sample_batch(ctx, [dict(space=sp, kappa=4.0, beta=0.6, b=x, k_minus=6, k_plus=6)],
                                              cheb_degree=3)[0][0]),
        "solve": (v, lambda x: sp.solve_shifted(30.0, x, cheb_degree=3)[0]),
        "tape": (v, lambda x: sp.sample_tape(4.0, 1.6, x, **kw)[0]),
        "grad": (v, lambda x: tape.grad_kappa(x)[0]),
    }
    wrong = []
    for name, (good, call) in calls.items():
        ref = call(good).clone()
        x, busy = late(good)
        got = call(x)
        torch.cuda.synchronize()
        del busy
        if not torch.equal(got, ref):
            wrong.append(name)
    assert not wrong
