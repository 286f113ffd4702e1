"""Harmonic analysis and synthesis at the edges of their launch shapes, against the
FP64 oracle: every workgroup shape (ring pairs a lane, waves), l counts around the
blocks of 4, 8 and 64, the m that change evaluation (2 and 16), a map's single
ring pair, temperature alone.  FP64 on both sides: 1e-12 of the largest value, as
for the other a_lm tests (sums of up to 1e4 FP64 products).  On a map the oracle's
W and X, differences of terms 2 / s^2 times as large next to the poles (s = sin
theta), carry their roundings with that factor (2.9e-12 of the largest Q at nside
256, lmax 9, against the harmonics in extended precision): 8 eps x 2 / s^2 more."""
import numpy as np
import pytest

from oracle import spectra as S

from gpu_helpers import say

pytestmark = pytest.mark.gpu
TOL = 1e-12


@pytest.fixture(scope="module")
def conv():
    import torch
    from paper_1908_05662_amd.api import Convolver

    c = Convolver(0)
    yield c
    torch.cuda.synchronize()
    c.close()


def _close(got, want):
    return np.abs(got.cpu().numpy() - want).max() <= TOL * np.abs(want).max()


@pytest.mark.parametrize("nside,lmax", [(1, 0), (1, 4), (2, 7), (32, 63), (64, 64), (128, 65), (128, 130), (256, 1),
                                        (256, 67), (512, 15), (512, 18), (1024, 17)])
@pytest.mark.parametrize("pol", [True, False])
def test_analysis_shapes(conv, nside, lmax, pol):
    import torch
    from paper_1908_05662_amd.api import Spectra

    say(f"case: map2alm nside {nside} lmax {lmax} pol {pol}")
    maps = np.random.default_rng(nside + lmax).normal(size=(3 if pol else 1, 12 * nside * nside))
    sp = Spectra(conv, nside, lmax, pol=pol)
    cl = sp.anafast(*(torch.from_numpy(m).cuda() for m in maps))
    want = S.map2alm(maps[0], *(maps[1:] if pol else (None, None)), S.healpix_rings(nside), lmax)
    for g, o in zip(sp.alm, want):
        assert o is None or not np.any(o) or _close(g, o)
    pairs = ((0, 0), (1, 1), (2, 2), (0, 1), (1, 2), (0, 2)) if pol else ((0, 0),)
    cls = np.stack([S.alm2cl(want[a], want[b], lmax) for a, b in pairs])
    assert np.abs(cl.cpu().numpy() - cls).max() <= TOL * np.abs(cls).max()


@pytest.mark.parametrize("nside,lmax", [(1, 2), (2, 8), (64, 5), (128, 3), (128, 66), (256, 9), (512, 4), (1024, 3)])
@pytest.mark.parametrize("pol", [True, False])
def test_synthesis_shapes(conv, nside, lmax, pol):
    import torch
    from paper_1908_05662_amd.api import Spectra

    say(f"case: alm2map nside {nside} lmax {lmax} pol {pol}")
    rng = np.random.default_rng(nside + lmax)
    al = [rng.normal(size=S.alm_size(lmax)) + 1j * rng.normal(size=S.alm_size(lmax)) for _ in range(3 if pol else 1)]
    for a in al:
        zero = S.alm_index(lmax, np.arange(lmax + 1), 0)
        a[zero] = a[zero].real
    got = Spectra(conv, nside, lmax, pol=pol).alm2map(*(torch.from_numpy(a).cuda() for a in al))
    rings = S.healpix_rings(nside)
    want = S.alm2map(al[0], *(al[1:] if pol else (None, None)), rings, lmax)
    tol = TOL + 16 * np.finfo(float).eps / np.repeat(rings["s"] ** 2, rings["count"])
    for k, (g, o) in enumerate(zip(got, want)):
        if o is not None:
            assert np.all(np.abs(g.cpu().numpy() - o) <= (tol if k else TOL) * np.abs(o).max())
