"""A sample's value does not depend on the launch it is part of: not on how many tiles
the launch holds (few are shared by 2, 4 or 8 waves), not on the staged chunk, not on
the entry point.  The sky makes the order of the FP64 sums visible: a flat beam over
pixels of order one with a few of +-2^44, exact in FP32 and cancelling in many discs, so
that the sum before the cancellation keeps 2^-9 of a value of order ten and any other
order of the same terms changes the FP32 result in many samples.  Bit for bit, no
tolerance."""
import numpy as np
import pytest

from gpu_helpers import say

pytestmark = pytest.mark.gpu
D2R = np.pi / 180
# the first is not shared: the reference; then 8, 8, 4, 4, 2 or 4, 2 or 1, 1 or 2 waves a tile (256 compute units; Stokes with four channels fewer)
TILES = (5200, 1, 200, 300, 900, 1100, 1900, 2500)


def _stream(n, jumps):
    t = np.arange(n)
    th, ph = 1.2 + 0.7 * np.sin(2e-5 * t), 1e-4 * t
    if jumps:
        # every sixth group of 64 samples jumps half-way through: too spread for a tile
        th = np.where((t // 64 % 6 == 5) & (t % 64 >= 32), np.pi - th, th)
    return th, ph, 1.0 + 3e-5 * t


@pytest.mark.parametrize("kind", ["scalar", "per_sample", "full", "full_v", "full_per_sample", "plate", "annulus"])
@pytest.mark.parametrize("jumps", [False, True])
def test_value_independent_of_launch(kind, jumps):
    import torch
    from paper_1908_05662_amd import NORM_FIXED, NORM_PER_SAMPLE, OUT_STOKES, OUT_TOD
    from paper_1908_05662_amd.api import Convolver

    nside = 128
    rng = np.random.default_rng(3)
    npix = 12 * nside * nside
    I = rng.normal(size=npix)
    big = rng.random(npix) < 0.02
    I[big] = np.where(rng.random(big.sum()) < 0.5, 2.0 ** 44, -2.0 ** 44)
    zero = np.zeros(npix)
    conv = Convolver(0)
    conv.set_ordering("given")
    conv.set_sky(nside, *(torch.from_numpy(x.astype(np.float32)).cuda() for x in (I, zero, zero)),
                 V=torch.from_numpy(I.astype(np.float32)).cuda() if kind == "full_v" else None)
    T = np.tan(6 * D2R)
    one, none = np.ones((41, 41), np.float32), np.zeros((41, 41), np.float32)
    if kind.startswith("full"):
        conv.set_beam(0, 41, T, one, none, none, one, **({"bV": 0.5 * one} if kind == "full_v" else {}))
    else:
        conv.set_beam_scalar(0, 41, T, one, 0.5, 0.25, 0.125)
    conv.set_detector(0, 0.4, 2 * D2R if kind == "annulus" else 0.0, 6 * D2R,
                      NORM_PER_SAMPLE if kind.endswith("per_sample") else NORM_FIXED, 1.0)
    ref = {}
    for tiles in TILES:
        n = 64 * tiles
        say(f"case: order of the sums, {kind}, jumps {jumps}, {tiles} tiles")
        p = _stream(n, jumps)
        conv.set_pointing(0, *(torch.from_numpy(x).cuda() for x in p))
        if kind == "plate":
            conv.set_hwp(0, torch.from_numpy(0.1 * np.arange(n)).cuda())
        for mode in (OUT_TOD, OUT_STOKES):
            for chunk in (64, 128, 256):
                conv.set_launch(chunk=chunk)
                outs = [conv.convolve(0, mode).cpu().numpy()]
                if chunk == 64:
                    outs.append(conv.convolve_static(0, mode).cpu().numpy())
                for o in outs:
                    ref.setdefault(mode, o)
                    differ = np.flatnonzero((o != ref[mode][:n]).reshape(n, -1).any(1))
                    assert differ.size == 0, (mode, tiles, chunk, differ[:5], differ.size)
    small = np.abs(ref[OUT_STOKES].reshape(-1, 3)[:, 0]) < 1e3
    say(f"  {small.mean():.2f} of the samples cancel")
    assert small.mean() > 0.02
    conv.close()
