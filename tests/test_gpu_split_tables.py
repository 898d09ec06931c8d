"""The tap tables that the split half-precision kernels keep from frame to
frame, with four banks of eight branches: bit 31 of a mask is a branch like any
other, so a mask of branches in bank 0 and that one is not the table of a
single bank.  Many short frames, so that every workgroup takes several.

Tolerances as for the kernels themselves: 2^-17 of sum |h| |u| an output
(forward), 2e-6 of the root of the sum of squares of the terms (grad_x)."""
import numpy as np
import pytest
import torch

from oracle.filterbank import fb_stream, fb_stream_adjoint
from paper_1802_06625_amd import ops

from gpu_util import announce

pytestmark = pytest.mark.gpu
KMAX, BANK_L = 8, (30, 64, 26, 49)


@pytest.fixture(autouse=True)
def _needs_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


def _c(rng, *shape):
    return ((rng.standard_normal(shape) + 1j * rng.standard_normal(shape)) * 0.3).astype(np.complex64)


def _case(frames, lens):
    rng = np.random.default_rng(frames)
    masks = [0xFF00, 0x80000001, 0xFF0000, 0x80000002, 0xFF000000, 0x80000003, 0x80000000, 0xFF]
    rows, t0 = [], 0
    for _ in range(frames):
        n = int(rng.choice(lens))
        rows.append((0, t0, n, masks[int(rng.integers(len(masks)))], 0))
        t0 += n
    taps = _c(rng, 1, 4, KMAX, max(BANK_L)) * 0.2
    return _c(rng, 1, t0), taps.astype(np.complex64), rows, rng


@pytest.mark.parametrize("variant", [6, 7, 8])
def test_forward_masks_with_the_last_branch(variant):
    announce(f"tap table, four banks of eight, variant {variant}")
    x, taps, rows, _ = _case(3000, [40, 41])
    ops.set_variant(variant)
    try:
        y = ops.fb_forward(torch.from_numpy(x).cuda(), torch.from_numpy(taps).cuda(), ops.frame_table(rows), KMAX,
                           BANK_L, 41).cpu().numpy()
    finally:
        ops.set_variant(0)
    fr = [r[1:] for r in rows]
    ref = fb_stream(x[0], fr, taps[0], BANK_L, KMAX)
    size = fb_stream(np.abs(x[0].astype(complex)), fr, np.abs(taps[0].astype(complex)), BANK_L, KMAX).real
    assert np.all(np.abs(y[0] - ref) <= 2.0 ** -17 * size)


def test_grad_x_masks_with_the_last_branch():
    announce("tap table of grad_x, four banks of eight")
    x, taps, rows, rng = _case(1500, [90, 97])
    g = _c(rng, *x.shape)
    ops.set_bwd_variant(2)
    try:
        gx, _ = ops.fb_backward(torch.from_numpy(x).cuda(), torch.from_numpy(taps).cuda(), ops.frame_table(rows),
                                torch.from_numpy(g).cuda(), KMAX, BANK_L, 97)
        gx = gx.cpu().numpy()
    finally:
        ops.set_bwd_variant(0)
    fr = [r[1:] for r in rows]
    ref, _ = fb_stream_adjoint(x[0], fr, taps[0], BANK_L, KMAX, g[0])
    size, r = np.zeros(x.shape[1]), np.abs(x[0].astype(complex))
    for (t0, n, m, _) in fr:
        for d in range(32):
            if (m >> d) & 1:
                h = np.abs(taps[0, d // KMAX, d % KMAX, :BANK_L[d // KMAX]].astype(complex)) ** 2
                sq = np.convolve(np.abs(g[0, t0:t0 + n].astype(complex)) ** 2, h[::-1])
                lo = max(0, t0 - len(h) + 1)
                sq = sq[lo - (t0 - len(h) + 1):]
                size[lo:lo + len(sq)] += sq * ((d % KMAX + 1) * r[lo:lo + len(sq)] ** (d % KMAX)) ** 2
    err = np.abs(gx[0] - ref)
    for k in range(0, len(err), 32):
        assert np.linalg.norm(err[k:k + 32]) <= 2e-6 * np.sqrt(np.sum(size[k:k + 32])), k
