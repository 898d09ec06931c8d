"""Frames written on the null stream, pushed, and fired on another stream: the
fire comes after the writes, also while they are still in flight, in every
execution mode, for frames written in place and for copied ones."""
import numpy as np
import pytest
import torch

from paper_1802_06625_amd import _lib as L
from paper_1802_06625_amd.graph import PlainGraph

from gpu_util import announce

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def _needs_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


@pytest.mark.parametrize("copied", [False, True])
@pytest.mark.parametrize("mode", [L.BATCHED, L.BATCHED_GRAPH, L.PER_FIRING])
def test_fire_on_another_stream(mode, copied):
    announce(f"fire on another stream, mode {mode}, copied {copied}")
    rng = np.random.default_rng(mode)
    F, n, K = 8, 512, 2
    side = np.tile(np.array([[K, n, 0, 0]], np.uint32), (F, 1))
    taps = torch.from_numpy((rng.standard_normal((1, K, 4)) + 1j).astype(np.complex64)).cuda()
    frames = [torch.from_numpy((rng.standard_normal(F * n) + 1j * rng.standard_normal(F * n)).astype(np.complex64)).cuda()
              for _ in range(3)]
    other = torch.cuda.Stream()

    def outputs(stream, slow):
        pg = PlainGraph(K, (4,), n, F)
        g, x, out = pg.g, torch.zeros(F * n, dtype=torch.complex64, device="cuda"), []
        g.set_taps(pg.fb, taps)
        torch.cuda.synchronize()
        for f in frames:
            if slow:
                torch.cuda._sleep(20_000_000)
            (x if copied else pg.fifo_in).copy_(f)
            g.source_push(pg.src, x if copied else None, np.full(F, n))
            g.config_push(pg.cfg, side)
            g.fire(mode, 0 if mode == L.PER_FIRING else F, stream=stream)
            g.sync(stream=stream)
            torch.cuda.synchronize()
            out.append(pg.fifo_out.cpu().numpy().copy())
        return out
    for a, b in zip(outputs(None, False), outputs(other, True)):
        assert np.array_equal(a, b)
