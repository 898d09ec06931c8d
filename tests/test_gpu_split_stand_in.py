"""A split half-precision variant set on a bank below 25 taps: variant 1 runs in
its place, bit for bit, also without allocation where the work list of variant
1's tiles would not fit but the set variant's does."""
import numpy as np
import pytest
import torch

from paper_1802_06625_amd import _lib as L
from paper_1802_06625_amd import ops

from gpu_util import announce

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def _needs_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


def _c(rng, *shape):
    return torch.from_numpy((rng.standard_normal(shape) + 1j * rng.standard_normal(shape)).astype(np.complex64)).cuda()


def _with(variant, f):
    ops.set_variant(variant)
    try:
        return f().cpu().numpy()
    finally:
        ops.set_variant(0)


@pytest.mark.parametrize("variant", [6, 7, 8])
@pytest.mark.parametrize("bank_L", [(2,), (24,), (40, 24)])
def test_short_banks_run_variant_1(variant, bank_L):
    announce(f"stand-in of variant {variant}, banks {bank_L}")
    rng = np.random.default_rng(variant)
    x, taps = _c(rng, 1, 9000), _c(rng, 1, len(bank_L), 3, max(bank_L))
    x[0, 3000:3300] *= 1e-9
    full = (1 << 3 * len(bank_L)) - 1
    fr = ops.frame_table([(0, 0, 5000, full, 0), (0, 5000, 1, 1, 0), (0, 5001, 3999, full, 0)])
    f = lambda: ops.fb_forward(x, taps, fr, 3, bank_L, 5000)
    assert np.array_equal(_with(variant, f), _with(1, f))
    ops.set_variant(variant)
    try:
        assert ops.tuned_variant(x, fr, 3, bank_L, 5000) == 1
    finally:
        ops.set_variant(0)


@pytest.mark.parametrize("variant,max_len", [(6, 70000), (6, 262144), (7, 70000), (8, 65536)])
def test_without_allocation_beyond_the_stand_ins_list(variant, max_len):
    """8000 and more frames of which each may have max_len
    samples, though they are short: a list of 2048-output tiles would not fit."""
    announce(f"no-alloc stand-in of variant {variant}, up to {max_len}")
    rng = np.random.default_rng(variant)
    n_frames, n = 8192 if variant == 6 else 8000, 40
    x, taps = _c(rng, 1, max(n_frames * n, max_len)), _c(rng, 1, 1, 2, 3)
    x[0, ::7] *= 1e-9
    fr = ops.frame_table([(0, k * n, n, 3, 0) for k in range(n_frames)])
    tile = {6: 8192, 7: 4096, 8: 2048}[variant]

    def f():
        y = torch.zeros_like(x)
        return ops.fb_forward_noalloc(x, taps, fr, 2, (3,), max_len, y)
    if n_frames * -(-max_len // tile) > 262144:
        with pytest.raises(L.PruneError):
            _with(variant, f)
        return
    ref = _with(1, lambda: ops.fb_forward(x, taps, fr, 2, (3,), n))
    assert np.array_equal(_with(variant, f)[0, :n_frames * n], ref[0, :n_frames * n])
