"""One launch over detectors of every path: discs of at most 16 rings (four samples a
wave), larger ones (a sample a wave) and coherent streams (the tile path).  The value of
a sample is that of its detector's own launch, bit for bit, for each kind of launch shape."""
import numpy as np
import pytest

from gpu_helpers import say

pytestmark = pytest.mark.gpu
D2R = np.pi / 180


@pytest.mark.parametrize("dtype", ["float32", "float64"])
@pytest.mark.parametrize("n", [1, 5, 1000])
def test_mixed_detectors(dtype, n):
    import torch
    from paper_1908_05662_amd import NORM_PER_SAMPLE, OUT_COUNT, OUT_STOKES, OUT_TOD
    from paper_1908_05662_amd.api import Convolver

    say(f"case: mixed detectors {dtype} n {n}")
    nside, tdt = 64, getattr(torch, dtype)
    rng = np.random.default_rng(n)
    conv = Convolver(0)
    conv.set_ordering("given")
    conv.set_sky(nside, *(torch.from_numpy(rng.normal(size=12 * nside * nside)).to(tdt).cuda() for _ in range(3)), dtype=tdt)
    for k, (deg, scan) in enumerate([(4.0, "random"), (8.0, "random"), (4.0, "slow"), (6.0, "slow"), (3.0, "random")]):
        T = np.tan(deg * D2R)
        u = np.linspace(-T, T, 41)
        b = np.exp(-0.5 * (u[:, None] ** 2 + 1.2 * u[None, :] ** 2) / (0.4 * deg * D2R) ** 2)
        conv.set_beam_scalar(k, 41, T, torch.from_numpy(b).to(tdt).cuda(), 0.5, 0.45, 0.1, dtype=tdt)
        conv.set_detector(k, 0.4 + k, 0.0, deg * D2R, NORM_PER_SAMPLE, 1.0)
        t = np.arange(n + 3 * k)
        th = np.arccos(rng.uniform(-1, 1, t.size)) if scan == "random" else 1.0 + 1e-5 * t
        ph = rng.uniform(0, 6, t.size) if scan == "random" else 1e-4 * t
        conv.set_pointing(k, *(torch.from_numpy(x).cuda() for x in (th, ph, 0.1 * t)))
    for kw in ({}, {"xcd_queues": 8}, {"algorithm": 0}, {"waves_per_group": 1, "samples_per_tile": 3}):
        conv.set_launch(**{"algorithm": 1, "samples_per_tile": 64, "waves_per_group": 4, "xcd_queues": 1, **kw})
        for mode in (OUT_TOD, OUT_STOKES, OUT_COUNT):
            whole = conv.convolve(-1, mode).cpu().numpy()
            each = np.concatenate([conv.convolve(k, mode).cpu().numpy() for k in range(5)])
            assert np.array_equal(whole, each), (kw, mode)
            if "samples_per_tile" not in kw:
                for k in range(5):
                    assert np.array_equal(conv.convolve_static(k, mode).cpu().numpy(), conv.convolve(k, mode).cpu().numpy())
    conv.close()
