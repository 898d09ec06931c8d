"""Split half-precision kernels where an output depends on operands far below
the largest of its wave's window: quiet stretches beside loud ones with the
high powers in front, masks and taps without the first power, taps that leave
the loud samples out, single samples in silence, stream starts and frame ends.

Forward, per output: |y - ref| <= 2^-17 sum |h| |u| and 1e-44 for fp32's
underflow.  110 roundings of 2^-24 make 2^-17.2 at worst, and an output that is
not evaluated again in fp32 may miss 2^-17 of itself at worst; both add up like
squares, to a tenth of the bound."""
import numpy as np
import pytest
import torch

from oracle.filterbank import fb_stream, fb_stream_adjoint
from paper_1802_06625_amd import ops

from gpu_util import announce

pytestmark = pytest.mark.gpu
BOUND = 2.0 ** -17


@pytest.fixture(autouse=True)
def _needs_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


def _c(rng, *shape):
    return (rng.standard_normal(shape) + 1j * rng.standard_normal(shape)).astype(np.complex64)


def _forward(variant, x, taps, rows, K, L, what):
    ops.set_variant(variant)
    try:
        y = ops.fb_forward(torch.from_numpy(x[None]).cuda(), torch.from_numpy(taps[None, None]).cuda(),
                           ops.frame_table([(0, *r, 0) for r in rows]), K, (L,), max(r[1] for r in rows))
        y = y[0].cpu().numpy().astype(np.complex128)
    finally:
        ops.set_variant(0)
    fr = [(*r, 0) for r in rows]
    ref = fb_stream(x, fr, taps[None], (L,), K)
    size = fb_stream(np.abs(x.astype(complex)), fr, np.abs(taps[None].astype(complex)), (L,), K).real
    off = np.abs(y - ref)
    worst = int(np.argmax(off / np.maximum(size, 1e-40)))
    assert np.all(off <= BOUND * size + 1e-44), (what, worst, off[worst] / max(size[worst], 1e-40))
    return y


@pytest.mark.parametrize("variant", [6, 8])
@pytest.mark.parametrize("L", [25, 64])
@pytest.mark.parametrize("sigma,step,K,zero", [(30, 5, 10, 0), (4, 4, 10, 0), (8, 5, 6, 0), (0.3, 9, 3, 1), (0.3, 9, 3, 2),
                                               (0.3, 12, 1, 0), (0.3, 25, 2, 0), (1, 1, 10, 9)])
def test_quiet_stretches(sigma, step, K, zero, L, variant):
    """Stretches of 300 samples at 2^-step of the rest; the taps of the first
    `zero` powers are zero though their branches are in the mask."""
    announce(f"quiet stretches sigma {sigma} step {step} K {K} zero {zero} L {L} variant {variant}")
    rng = np.random.default_rng(K + 100 * L)
    x = _c(rng, 5000) * np.float32(sigma)
    for a in (700, 2000, 3333):
        x[a:a + 300] *= np.float32(2.0 ** -step)
    taps = _c(rng, K, L)
    taps[:zero] = 0
    _forward(variant, x, taps, [(0, 5000, (1 << K) - 1)], K, L, "stretch")


@pytest.mark.parametrize("K", [5, 10])
@pytest.mark.parametrize("P", [4, 8, 16, 64])
def test_quiet_frame_after_a_loud_one(P, K):
    announce(f"quiet after loud, {P}:1, K {K}")
    rng = np.random.default_rng(P)
    x = np.exp(2j * np.pi * rng.uniform(size=1700)).astype(np.complex64)
    x[:64] *= P
    x[1000:1064] *= P
    _forward(6, x, _c(rng, K, 32), [(0, 1064, (1 << K) - 1), (1064, 300, (1 << K) - 1), (1364, 336, (1 << K) - 1)], K, 32,
             "frame")


@pytest.mark.parametrize("mask", [0x2, 0x200, 0x3FE, 0x2AA, 0x60])
def test_masks_without_the_first_power(mask):
    announce(f"mask {mask:#x}")
    rng = np.random.default_rng(mask)
    for sigma in (0.3, 1.0, 50.0):
        x = _c(rng, 4000) * np.float32(sigma)
        x[1500:1600] *= np.float32(0.05)
        _forward(7, x, _c(rng, 10, 30), [(0, 4000, mask)], 10, 30, sigma)


@pytest.mark.parametrize("share", [0.2, 0.002])   # whole waves, and outputs one by one
@pytest.mark.parametrize("taps_of", ["one", "first", "decaying", "two scales"])
def test_taps_that_leave_samples_out(taps_of, share):
    announce(f"taps {taps_of}, share {share}")
    rng = np.random.default_rng(7)
    K, L = 3, 40
    x = _c(rng, 4000)
    x[rng.uniform(size=4000) < share] *= np.float32(1e-9)
    taps = _c(rng, K, L)
    if taps_of == "one":
        taps[:, np.arange(L) != 11] = 0
    elif taps_of == "first":
        taps[:, 1:] = 0
    elif taps_of == "decaying":
        taps *= np.exp2(-2.0 * np.arange(L)).astype(np.float32)
    else:
        taps[:, ::2] *= np.float32(1e-11)
    _forward(6, x, taps, [(0, 4000, 7)], K, L, taps_of)


@pytest.mark.parametrize("variant", [6, 7, 8])
def test_beside_silence(variant):
    """A stream that begins with a tiny sample, tails before silence, single
    samples in it; outputs of silent windows are exact zeros."""
    announce(f"beside silence, variant {variant}")
    rng = np.random.default_rng(variant)
    K, L, n = 4, 25, 6000
    x = _c(rng, n) * np.float32(0.3)
    x[0] = 1e-9
    x[1000:1003] *= np.float32(1e-10)
    x[1003:1200] = 0
    x[2000:2300] = 0
    x[2100] = 1e-12 + 1e-13j
    x[3000:5100] = 0
    x[5100] *= np.float32(1e-11)
    x[n - 1] *= np.float32(1e-10)
    taps = _c(rng, K, L)
    y = _forward(variant, x, taps, [(0, 2050, 15), (2050, 1500, 15), (3550, n - 3550, 15)], K, L, "silence")
    for a, b in ((1003, 1200), (2000, 2100), (2101, 2300), (3000, 5100)):
        assert np.all(y[a + L - 1:b] == 0)
    assert np.all(_forward(variant, x, taps * 0, [(0, n, 15)], K, L, "no taps") == 0)


# ---- grad_x: per sample |grad - ref| <= 2^-16 sum_p (1 + p) r^p sum_l |h| |g|
# (2^-17 that may be missing of g's parts, and the roundings as above)
def _grad_x(x, g, taps, rows, K, L, what):
    ops.set_bwd_variant(2)
    try:
        gx, _ = ops.fb_backward(torch.from_numpy(x[None]).cuda(), torch.from_numpy(taps[None, None]).cuda(),
                                ops.frame_table([(0, *r, 0) for r in rows]), torch.from_numpy(g[None]).cuda(), K, (L,),
                                max(r[1] for r in rows))
        gx = gx[0].cpu().numpy().astype(np.complex128)
    finally:
        ops.set_bwd_variant(0)
    ref, _ = fb_stream_adjoint(x, [(*r, 0) for r in rows], taps[None], (L,), K, g)
    size, r = np.zeros(len(x)), np.abs(x.astype(complex))
    for (t0, n, m) in rows:
        for p in range(K):
            if (m >> p) & 1:
                G = np.convolve(np.abs(g[t0:t0 + n].astype(complex)), np.abs(taps[p].astype(complex))[::-1])
                lo = max(0, t0 - L + 1)
                G = G[lo - (t0 - L + 1):]
                size[lo:lo + len(G)] += G * (1 + p) * r[lo:lo + len(G)] ** p
    off = np.abs(gx - ref)
    worst = int(np.argmax(off / np.maximum(size, 1e-40)))
    assert np.all(off <= 2.0 ** -16 * size + 1e-44), (what, worst, off[worst] / max(size[worst], 1e-40))
    return gx


@pytest.mark.parametrize("L", [15, 40, 64])
@pytest.mark.parametrize("step", [8, 13, 17, 30])
def test_grad_x_quiet_cotangent(step, L):
    announce(f"grad_x, cotangent at 2^-{step}, L {L}")
    rng = np.random.default_rng(step + L)
    x, g, K = _c(rng, 5000) * np.float32(0.3), _c(rng, 5000), 6
    for a in (700, 2000, 3333):
        g[a:a + 300] *= np.float32(2.0 ** -step)
    _grad_x(x, g, _c(rng, K, L), [(0, 2800, 63), (2800, 2200, 62)], K, L, "cotangent")


@pytest.mark.parametrize("K", [1, 4])
def test_grad_x_beside_zeros(K):
    """Tiny last samples of a frame, single and tiny cotangents among zeros;
    gradients before zeros alone are exact zeros."""
    announce(f"grad_x beside zeros, K {K}")
    rng = np.random.default_rng(K)
    n, L = 6000, 25
    x, g = _c(rng, n) * np.float32(0.3), _c(rng, n)
    g[1500] *= np.float32(1e-10)
    g[1497:1500] = 0
    g[1999] *= np.float32(1e-12)
    g[3000:3300] = 0
    g[3100] = 1e-11
    g[4000:5500] = 0
    g[5500:5503] *= np.float32(1e-9)
    x[2500:2600] = 0
    gx = _grad_x(x, g, _c(rng, K, L), [(0, 2000, (1 << K) - 1), (2000, 1001, (1 << K) - 1),
                                      (3001, 2999, (1 << K) - 1)], K, L, "zeros")
    assert np.all(gx[4000:5500 - L] == 0) and np.all(gx[3101:3300 - L] == 0)


@pytest.mark.parametrize("mask", [0x3FF, 0x200, 0x2A4])
@pytest.mark.parametrize("what", ["units of 3000", "loud and quiet", "tiny", "one tap", "decaying taps"])
def test_grad_x_samples_and_taps(what, mask):
    announce(f"grad_x {what}, mask {mask:#x}")
    rng = np.random.default_rng(mask)
    K, L, n = 10, 30, 4000
    x, g, taps = _c(rng, n) * np.float32(0.3), _c(rng, n), _c(rng, K, L)
    if what == "units of 3000":
        x *= np.float32(1e4)
        taps[4:] *= np.float32(1e-20)
    elif what == "loud and quiet":
        x[500:900] *= 30
        x[1500:1600] *= np.float32(0.01)
    elif what == "tiny":
        x *= np.float32(1e-3)
    elif what == "one tap":
        taps[:, np.arange(L) != 11] = 0
        g[rng.uniform(size=n) < 0.1] *= np.float32(1e-9)
    else:
        taps *= np.exp2(-2.0 * np.arange(L)).astype(np.float32)
        g[rng.uniform(size=n) < 0.1] *= np.float32(1e-9)
    _grad_x(x, g, taps, [(0, n, mask)], K, L, what)


# ---- tap gradients: per entry |grad - ref| <= 2^-16 sum |g| |u|
@pytest.mark.parametrize("L", [1, 10, 20, 64])
@pytest.mark.parametrize("what", ["one in 700", "one in 64", "loud without cotangent", "quiet only", "masked", "faint ends", "comb"])
def test_grad_taps(what, L):
    announce(f"tap gradients {what}, L {L}")
    rng = np.random.default_rng(L)
    n, K = 9000, 10
    x, g, k = _c(rng, n) * np.float32(0.3), _c(rng, n), np.arange(n)
    if what == "one in 700":
        g[k % 700 != 650] = 0
    elif what == "one in 64":
        g[k % 64 != 5] = 0
    elif what == "loud without cotangent":
        x[(k // 100) % 2 == 0] *= 64
        g[(k // 100) % 2 == 0] = 0
    elif what == "quiet only":
        x[k % 2000 < 150] *= np.float32(2.0 ** -6)
        g[k % 2000 >= 150 - L] = 0
        g[k % 2000 < L] = 0
    elif what == "masked":
        g[(k // 1500) % 2 == 1] = 0
    elif what == "comb":   # most taps see faint cotangents only
        x[k % 8 != 0] = 0
        g[k % 8 != 0] *= np.float32(1e-10)
    else:
        x[k % 512 > 500] *= np.float32(1e-6)
        g[k % 512 < 400] *= np.float32(1e-9)
    rows = [(0, 0, 3, 0x3FF, 0), (0, 3, 2900, 0x3FF, 0), (0, 2903, 1, 0x201, 0), (0, 2904, n - 2904, 0x3FE, 0)]
    taps = _c(rng, 1, 1, K, L)
    ops.set_bwd_variant(2)
    try:
        _, gt = ops.fb_backward(torch.from_numpy(x[None]).cuda(), torch.from_numpy(taps).cuda(), ops.frame_table(rows),
                                torch.from_numpy(g[None]).cuda(), K, (L,), n, want_gx=False)
        gt = gt[0].cpu().numpy()
    finally:
        ops.set_bwd_variant(0)
    fr = [r[1:] for r in rows]
    _, ref = fb_stream_adjoint(x, fr, taps[0], (L,), K, g)
    _, size = fb_stream_adjoint(np.abs(x.astype(complex)), fr, taps[0], (L,), K, np.abs(g.astype(complex)))
    off = np.abs(gt - ref)
    assert np.all(off <= 2.0 ** -16 * np.real(size) + 1e-44), (what, L, np.max(off / np.maximum(np.real(size), 1e-40)))
