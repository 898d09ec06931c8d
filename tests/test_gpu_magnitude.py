"""|x| is the correctly rounded root of fmaf(re, re, im * im) in every vector
forward kernel: one tap of one on the second power gives the rounded product of
|x| and x, bit for bit."""
from fractions import Fraction

import numpy as np
import pytest
import torch

from paper_1802_06625_amd import ops

from gpu_util import announce

pytestmark = pytest.mark.gpu


def _rounded_sum(a, b, c):
    """float32 of a * b + c, exact inside (a * b is exact in 64 bits)."""
    out = np.empty(len(a), np.float32)
    for k in range(len(a)):
        exact = Fraction(float(a[k])) * Fraction(float(b[k])) + Fraction(float(c[k]))
        near = np.float32(float(exact))
        cand = [np.nextafter(near, np.float32(0)), near, np.nextafter(near, np.float32(np.inf))]
        # nearest, ties to even
        out[k] = min(cand, key=lambda v: (abs(Fraction(float(v)) - exact), int(v.view(np.uint32)) & 1))
    return out


@pytest.mark.parametrize("variant", [0, 1, 2, 3, 4, 5])
def test_rounding_of_the_magnitude(variant):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    announce(f"magnitude, variant {variant}")
    rng = np.random.default_rng(1)
    n = 3000
    x = (rng.standard_normal(n) + 1j * rng.standard_normal(n)).astype(np.complex64)
    re, im = x.real, x.imag
    r = np.sqrt(_rounded_sum(re, re, im * im))
    taps = np.zeros((1, 1, 2, 1), np.complex64)
    taps[0, 0, 1, 0] = 1
    ops.set_variant(variant)
    try:
        y = ops.fb_forward(torch.from_numpy(x[None]).cuda(), torch.from_numpy(taps).cuda(),
                           ops.frame_table([(0, 0, n, 2, 0)]), 2, (1,), n)[0].cpu().numpy()
    finally:
        ops.set_variant(0)
    assert np.array_equal(y.real, re * r) and np.array_equal(y.imag, im * r)
