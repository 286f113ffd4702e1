"""Launches of few tiles on eight work queues: the same values as on one queue, bit for
bit, and about the same time (as many workgroups take a tile): within half of it, where
a launch that keeps seven eighths of its workgroups idle takes two to four times as
long.  The least of eight launches each, one shape after the other."""
import numpy as np
import pytest

from gpu_helpers import say

pytestmark = pytest.mark.gpu
D2R = np.pi / 180


@pytest.mark.parametrize("tiles", [5, 250, 1024, 3000])
def test_eight_queues_as_one(tiles):
    import torch
    from paper_1908_05662_amd import NORM_PER_SAMPLE
    from paper_1908_05662_amd.api import Convolver

    say(f"case: shared tiles on eight queues, {tiles} tiles")
    nside, n = 512, 64 * tiles - 5
    rng = np.random.default_rng(tiles)
    t = np.arange(n)
    conv = Convolver(0)
    conv.set_ordering("given")
    conv.set_sky(nside, *(torch.from_numpy(rng.normal(size=12 * nside * nside).astype(np.float32)).cuda()
                          for _ in range(3)))
    T = np.tan(3 * D2R)
    u = np.linspace(-T, T, 61)
    b = np.exp(-0.5 * (u[:, None] ** 2 + 1.2 * u[None, :] ** 2) / (1 * D2R) ** 2).astype(np.float32)
    conv.set_beam_scalar(0, 61, T, b, 0.5, 0.45, 0.1)
    conv.set_detector(0, 0.4, 0.0, 3 * D2R, NORM_PER_SAMPLE, 1.0)
    conv.set_pointing(0, *(torch.from_numpy(x).cuda() for x in (1.2 + 0.7 * np.sin(2e-5 * t), 1e-4 * t, 1.0 + 3e-5 * t)))
    best, got = {1: 1e9, 8: 1e9}, {}
    a, z = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    for queues in (1, 8):
        conv.set_launch(xcd_queues=queues)
        got[queues] = conv.convolve(0).cpu().numpy()
        for _ in range(8):
            torch.cuda.synchronize()
            a.record()
            conv.convolve(0)
            z.record()
            torch.cuda.synchronize()
            best[queues] = min(best[queues], a.elapsed_time(z))
    say(f"  {1e3 * best[1]:.0f} us on one queue, {1e3 * best[8]:.0f} on eight")
    assert np.array_equal(got[1], got[8])
    assert best[8] <= 1.5 * best[1]
    conv.close()
