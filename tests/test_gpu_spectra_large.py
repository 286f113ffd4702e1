"""Synthesis and refinement on large maps: two and four ring pairs a lane (nside 256,
512, 1024) over a full range of l, where rings start many powers of two below their
later values, the loop's steps are pipelined and the bands past the first take the
shorter form of the recurrences.  a_lm of a few m keep the oracle's work small.

Tolerances, of the largest value: the recurrences of both sides round a few eps at
each of lmax steps and a step's rounding grows like 1 / s (s = sin theta); W and X,
differences of terms 2 / s^2 times as large, carry the oracle's roundings with that
factor: 4 eps lmax / s^2 covers both.  Refined a_lm: 1e-12 as for one pass (sums of up
to 1e4 FP64 products), once for the pass and once for each step."""
import numpy as np
import pytest

from oracle import spectra as S

from gpu_helpers import say

pytestmark = pytest.mark.gpu
EPS = np.finfo(float).eps


@pytest.fixture(scope="module")
def conv():
    import torch
    from paper_1908_05662_amd.api import Convolver

    c = Convolver(0)
    yield c
    torch.cuda.synchronize()
    c.close()


def _maps_of(al, ms, rings, lmax):
    """T, Q, U of a_lm that are zero but for the m of `ms`."""
    nr = len(rings["z"])
    G = np.zeros((3, len(ms), nr), dtype=complex)
    for i, m in enumerate(ms):
        lam = S.lambda_block(m, lmax, rings["z"], rings["s"])
        W, X = S.spin2_block(m, lmax, rings["z"], rings["s"], lam)
        t, e, b = (a[S.alm_index(lmax, np.arange(m, lmax + 1), m)] for a in al)
        G[0, i] = t @ lam
        G[1, i] = -(e @ W + 1j * (b @ X))
        G[2, i] = -(b @ W - 1j * (e @ X))
    ring = np.repeat(np.arange(nr), rings["count"])
    j = np.arange(ring.size) - rings["first"][ring]
    out = np.zeros((3, ring.size))
    for i, m in enumerate(ms):
        # m phi, the ring part reduced exactly
        phi = m * rings["phi0"][ring] + 2 * np.pi * ((m * j) % rings["count"][ring]) / rings["count"][ring]
        out += (1 if m == 0 else 2) * (G[:, i, ring] * np.exp(1j * phi)).real
    return out


@pytest.mark.parametrize("nside,lmax", [(256, 767), (512, 1024), (512, 1535), (1024, 3071)])
def test_synthesis_full_range(conv, nside, lmax):
    import torch
    from paper_1908_05662_amd.api import Spectra

    say(f"case: alm2map of a few m, nside {nside} lmax {lmax}")
    ms = [0, 1, 2, 17, nside, 2 * nside - 1, lmax - 6]
    rng = np.random.default_rng(nside + lmax)
    al = [np.zeros(S.alm_size(lmax), dtype=complex) for _ in range(3)]
    for m in ms:
        k = S.alm_index(lmax, np.arange(m, lmax + 1), m)
        for a in al:
            a[k] = rng.normal(size=k.size) + (1j * rng.normal(size=k.size) if m else 0)
    dev = [torch.from_numpy(a).cuda() for a in al]
    rings = S.healpix_rings(nside)
    want = _maps_of(al, ms, rings, lmax)
    tol = np.repeat(4 * EPS * lmax / rings["s"] ** 2, rings["count"])
    sp = Spectra(conv, nside, lmax)
    for g, o in zip(sp.alm2map(*dev), want):
        assert np.all(np.abs(g.cpu().numpy() - o) <= tol * np.abs(o).max())
    T = sp.alm2map(dev[0])[0].cpu().numpy()
    assert np.all(np.abs(T - want[0]) <= tol * np.abs(want[0]).max())


@pytest.mark.parametrize("nside,lmax,steps", [(256, 20, 2), (512, 18, 1)])
@pytest.mark.parametrize("pol", [True, False])
def test_refinement_on_large_maps(conv, nside, lmax, steps, pol):
    import torch
    from paper_1908_05662_amd.api import Spectra

    say(f"case: refined map2alm nside {nside} lmax {lmax} steps {steps} pol {pol}")
    maps = np.random.default_rng(nside).normal(size=(3 if pol else 1, 12 * nside * nside))
    got = Spectra(conv, nside, lmax, pol=pol).map2alm(*(torch.from_numpy(m).cuda() for m in maps), iterations=steps)
    want = S.map2alm_iter(maps[0], *(maps[1:] if pol else (None, None)), S.healpix_rings(nside), lmax, steps)
    for g, o in zip(got, want):
        if o is not None:
            assert np.abs(g.cpu().numpy() - o).max() <= (1 + steps) * 1e-12 * np.abs(o).max()


@pytest.mark.parametrize("nside,lmax", [(8, 0), (8, 1), (512, 1)])
def test_no_polarisation_below_two(conv, nside, lmax):
    import torch
    from paper_1908_05662_amd.api import Spectra

    say(f"case: a^E, a^B of l < 2, nside {nside} lmax {lmax}")
    maps = np.random.default_rng(lmax).normal(size=(3, 12 * nside * nside))
    got = Spectra(conv, nside, lmax).map2alm(*(torch.from_numpy(m).cuda() for m in maps))
    assert not got[1].any() and not got[2].any() and got[0].any()
