"""Launches of few tiles share each tile among the waves of a workgroup: a sample's
value may not depend on how many tiles the launch holds.  The terms are summed in
FP32 in the same groups and only the FP64 sums of the groups are split, so TODs and
pickups agree to one FP32 rounding (2^-23 of the value: two neighbouring floats),
counts exactly; the two entry points agree throughout.  Streams of 1, 256, 257, 1024, 1025, 3072, 3073 and 5121 tiles (the ends of
the 8-, 4- and 2-wave launches with 256 compute units), the last tile ragged."""
import numpy as np
import pytest

from gpu_helpers import say

pytestmark = pytest.mark.gpu
TILES = (1, 256, 257, 1024, 1025, 3072, 3073, 5121)
D2R = np.pi / 180


@pytest.mark.parametrize("kind", ["scalar", "full", "plate", "annulus"])
def test_tile_count_changes_no_sample(kind):
    import torch
    from paper_1908_05662_amd import NORM_FIXED, NORM_PER_SAMPLE, OUT_COUNT, OUT_STOKES, OUT_TOD
    from paper_1908_05662_amd.api import Convolver

    nside, n_max = 64, 64 * TILES[-1] - 7
    rng = np.random.default_rng(5)
    t = np.arange(n_max)
    th = 1.2 + 0.7 * np.sin(2e-5 * t)
    ph, ps = 1e-4 * t, 1.0 + 3e-5 * t
    conv = Convolver(0)
    conv.set_ordering("given")
    conv.set_sky(nside, *(torch.from_numpy(rng.normal(size=12 * nside * nside).astype(np.float32)).cuda()
                          for _ in range(3)))
    T = np.tan(6 * D2R)
    u = np.linspace(-T, T, 41)
    b = np.exp(-0.5 * (u[:, None] ** 2 + 1.2 * u[None, :] ** 2) / (2 * D2R) ** 2).astype(np.float32)
    if kind == "full":
        conv.set_beam(0, 41, T, b, 0.9 * b, 0.01 * b * np.sign(u)[None, :].astype(np.float32), b)
    else:
        conv.set_beam_scalar(0, 41, T, b, 0.5, 0.45, 0.1)
    inner = kind == "annulus"
    conv.set_detector(0, 0.4, 2 * D2R if inner else 0.0, 6 * D2R, NORM_FIXED if inner else NORM_PER_SAMPLE, 0.01 if inner else 1.0)
    ref = {}
    for tiles in reversed(TILES):
        n = 64 * tiles - 7
        say(f"case: shared tiles, {kind}, {tiles} tiles")
        conv.set_pointing(0, *(torch.from_numpy(x[:n]).cuda() for x in (th, ph, ps)))
        if kind == "plate":
            conv.set_hwp(0, torch.from_numpy(0.1 * t[:n]).cuda())
        for mode in (OUT_TOD, OUT_STOKES, OUT_COUNT):
            outs = [conv.convolve(0, mode).cpu().numpy(), conv.convolve_static(0, mode).cpu().numpy()]
            for o in outs:
                if mode not in ref:
                    ref[mode] = o
                    continue
                whole = 64 * (n // 64)        # a ragged tile is another tile: another centre
                want = ref[mode][:whole]
                tol = 0.0 if mode == OUT_COUNT else 2.0 ** -23
                assert np.all(np.abs(o[:whole] - want) <= tol * np.abs(want)), (mode, tiles)
            assert np.array_equal(*outs)
    conv.close()
