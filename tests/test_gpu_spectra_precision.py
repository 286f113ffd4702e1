"""The a_lm against the harmonics in extended precision (80-bit, exact ring geometry):
the analysis is no further from them than the FP64 oracle, which forms W and X from
lambda_l and lambda_{l-1}.  Both sum thousands of products of one rounding each, and the
device's own recurrences of W +- X (m >= 2; 16 above nside 256) leave out the oracle's
cancellation next to the poles: the root mean square over l, taken over T, E and B, is
at most 1.25 times the oracle's (for the spread of two such sums of a few hundred
errors).  The columns m = 2 .. 16 of the largest map against the oracle itself, as for
the others: 1e-12 of the largest value."""
import numpy as np
import pytest

from oracle import spectra as S

from gpu_helpers import say

pytestmark = pytest.mark.gpu
LD = np.longdouble
PI = LD("3.14159265358979323846264338327950288")


@pytest.fixture(scope="module")
def conv():
    import torch
    from paper_1908_05662_amd.api import Convolver

    c = Convolver(0)
    yield c
    torch.cuda.synchronize()
    c.close()


def _exact_column(maps, rings, nside, lmax, m):
    """a^T, a^E, a^B of l = m..lmax by the recurrences of lambda and of W +- X in 80 bits."""
    i = np.arange(1, 4 * nside)
    k = np.minimum(np.minimum(i, 4 * nside - i), nside)
    cap = (i < nside) | (i > 3 * nside)
    t = LD(1) * k * k / (LD(3) * nside * nside)
    z = np.where(cap, np.where(i < nside, 1 - t, t - 1), (LD(4) * nside - LD(2) * i) / (LD(3) * nside))
    omz = np.where(cap, np.where(i < nside, t, 2 - t), (LD(2) * i - nside) / (LD(3) * nside))
    opz = 2 - omz
    s = np.sqrt(omz * opz)
    F = [S.ring_fourier(x, rings, m)[:, m].astype(np.clongdouble) * (4 * PI / (12 * nside * nside)) for x in maps]
    P, M = F[1] + 1j * F[2], F[1] - 1j * F[2]
    c = np.sqrt(np.prod([LD(2 * q + 1) / (2 * q) for q in range(1, m + 1)] + [LD(1)]) / (4 * PI))
    v, vp = (-1) ** m * c * s ** m, 0 * s
    if m >= 2:
        cc = np.sqrt(LD(m) * (m - 1) / ((m + 1) * (m + 2)))
        f0, g0 = cc * v * omz / opz, cc * v * opz / omz
    elif m == 1:
        cc = np.sqrt(5 / (16 * PI))
        f0, g0 = -cc * s * omz, cc * s * opz
    else:
        f0 = g0 = np.sqrt(15 / (32 * PI)) * s * s
    A = lambda l: np.sqrt((LD(l) * l - m * m) / (4 * LD(l) * l - 1))
    B = lambda l: A(l) * np.sqrt(LD(l) * l - 4) / l
    f = g = fp = gp = 0 * s
    out = np.zeros((3, lmax - m + 1), dtype=np.clongdouble)
    l0 = max(m, 2)
    for l in range(m, lmax + 1):
        if l > m:
            v, vp = (z * v - A(l - 1) * vp) / A(l), v
        if l == l0:
            f, g = f0, g0
        elif l > l0:
            q, b = LD(2) * m / (LD(l) * (l - 1)), B(l - 1) if l - 1 > l0 else 0
            f, fp = ((z + q) * f - b * fp) / B(l), f
            g, gp = ((z - q) * g - b * gp) / B(l), g
        out[0, l - m] = np.sum(v * F[0])
        if l >= 2:
            sp, sm = np.sum(f * P), np.sum(g * M)
            out[1, l - m], out[2, l - m] = -(sp + sm) / 2, 1j * (sp - sm) / 2
    return out


@pytest.mark.parametrize("nside,lmax", [(128, 383), (512, 1023)])
def test_analysis_precision(conv, nside, lmax):
    import torch
    from paper_1908_05662_amd.api import Spectra

    say(f"case: precision of map2alm nside {nside} lmax {lmax}")
    maps = np.random.default_rng(nside).normal(size=(3, 12 * nside * nside))
    got = [a.cpu().numpy() for a in Spectra(conv, nside, lmax).map2alm(*(torch.from_numpy(m).cuda() for m in maps))]
    rings, ms = S.healpix_rings(nside), [0, 1, 2, 5, 17, nside]
    want = S.map2alm(*maps, rings, lmax, mmax=max(ms), ms=ms)
    for m in ms:
        k = S.alm_index(lmax, np.arange(m, lmax + 1), m)
        exact = _exact_column(maps, rings, nside, lmax, m)
        rms = [np.sqrt(sum((np.abs(a[k] - e) ** 2).sum() for a, e in zip(side, exact)) / (np.abs(exact) ** 2).sum())
               for side in (got, want)]
        say(f"  m {m}: device {float(rms[0]):.2e}, oracle {float(rms[1]):.2e}")
        assert rms[0] <= 1.25 * rms[1]


def test_first_columns_of_the_largest_map(conv):
    import torch
    from paper_1908_05662_amd.api import Spectra

    nside, lmax, ms = 1024, 3071, [2, 5, 15, 16]
    say(f"case: map2alm columns {ms}, nside {nside} lmax {lmax}")
    maps = np.random.default_rng(7).normal(size=(3, 12 * nside * nside))
    got = Spectra(conv, nside, lmax).map2alm(*(torch.from_numpy(m).cuda() for m in maps))
    want = S.map2alm(*maps, S.healpix_rings(nside), lmax, mmax=16, ms=ms)
    for m in ms:
        k = S.alm_index(lmax, np.arange(m, lmax + 1), m)
        for g, o in zip(got, want):
            assert np.abs(g.cpu().numpy()[k] - o[k]).max() <= 1e-12 * np.abs(o[k]).max(), m
