"""Degrees 4 and 5 factorise the element matrices once a call, whatever the number of samples.

One thread factorises an element there, which takes longer than all of a few dozen samples: on degree 5, 64 x 64
elements, 48 samples (170 MB of work space) may take up to twice as long as 8.  Factorising again for every 16
samples takes three times as long and more.
"""
import time

import pytest

torch = pytest.importorskip("torch")
from paper_2605_24882_amd import gfield as g  # noqa: E402

pytestmark = pytest.mark.gpu


def test_elements_are_factorised_once():
    ctx = g.Context(0)
    sp = g.Space(ctx, g.Geometry(ctx, False), 5, 6)

    def seconds(n):
        z = torch.randn(n, sp.noise_length, dtype=torch.float64, device="cuda")
        sp.white_noise(z)
        torch.cuda.synchronize()
        best = 1e30
        for _ in range(5):
            t = time.perf_counter()
            sp.white_noise(z)
            best = min(best, time.perf_counter() - t)
        return best

    few, many = seconds(8), seconds(48)
    print(f"8 samples {few * 1e3:.2f} ms, 48 samples {many * 1e3:.2f} ms")
    assert many <= 2.0 * few
