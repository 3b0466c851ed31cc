"""Device arrays of one call that overlap: inputs are read before an output takes their place."""
import ctypes

import numpy as np
import pytest

torch = pytest.importorskip("torch")
from paper_2605_24882_amd import gfield as g  # noqa: E402

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    return g.Context(0)


def ptr(t):
    return ctypes.c_void_p(t.data_ptr())


def test_white_noise_over_its_input(ctx):
    # several passes over the samples (16 of 7 MB each at a time); the loads take the place of the last vectors
    sp = g.Space(ctx, g.Geometry(ctx, False), 2, 7)
    z = torch.randn(40, sp.noise_length, dtype=torch.float64, device="cuda",
                    generator=torch.Generator(device="cuda").manual_seed(1))
    ref = sp.white_noise(z)
    out = z.reshape(-1)[-ref.numel():]
    assert g._lib.gf_white_noise(sp.h, 40, ptr(z), ptr(out), g.GF_DEVICE) == g.GF_OK
    assert torch.equal(out, ref.reshape(-1))


def test_eval_into_the_points(ctx):
    sp = g.Space(ctx, g.Geometry(ctx, False), 3, 4)
    rng = np.random.default_rng(2)
    npts = 200000
    patch = torch.from_numpy(rng.integers(0, 6, npts).astype(np.int32)).cuda()
    st = torch.from_numpy(rng.random((npts, 2))).cuda()
    u = torch.from_numpy(rng.standard_normal((2, sp.ndofs))).cuda()
    ref = sp.eval(patch, st, u)
    assert g._lib.gf_eval(sp.h, npts, ptr(patch), ptr(st), 2, ptr(u), ptr(st), g.GF_DEVICE) == g.GF_OK
    assert torch.equal(st.reshape(-1), ref.reshape(-1))
