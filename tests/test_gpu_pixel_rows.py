"""The pixel path's four-samples-a-wave form (discs of at most 16 rings, 3 nside rho_max)
and the walk over the work queues.  Tolerances are the suite's: 1e-12 of the largest
value in FP64, 1e-6 in FP32 (algorithm 0), against the oracle; counts exactly."""
import numpy as np
import pytest

import oracle
from synth import beams as B
from synth import workloads as W
from synth.workloads import Detector, Workload

from gpu_helpers import load_workload, oracle_detector, rel_err, say

pytestmark = pytest.mark.gpu
TOL = {np.float64: 1e-12, np.float32: 1e-6}


@pytest.fixture()
def conv():
    import torch
    from paper_1908_05662_amd.api import Convolver

    c = Convolver(0)
    yield c
    torch.cuda.synchronize()
    c.close()


def _workload(nside, rho, n, norm, rho_min=0.0, seed=3):
    """Random pointings with both poles, their neighbourhood and the cap edges among them."""
    rng = np.random.default_rng(seed)
    th = np.arccos(rng.uniform(-1, 1, n))
    edge = [0.0, np.pi, 1e-9, rho, np.pi - rho, rho * (1 + 1e-12), np.arccos(2 / 3), np.arccos(-2 / 3), np.pi / 2]
    th[:min(n, len(edge))] = edge[:n]
    ph, ps = rng.uniform(-8, 8, n), rng.uniform(-7, 7, n)
    T, u, v, r, sig = B.tangent_grid(41, rho)
    g = B.elliptical_gaussian(r, sig, 0.7 * rho, 0.1, 0.5)
    bs = B.with_qu_leakage(B.ideal_beamsor(g, T), g, 0.01)
    d = Detector(bs, B.DetectorParams(0.3, 0.02, 1.1), rho_min, rho, norm, 1.0, th, ph, ps)
    sky = tuple(rng.normal(size=12 * nside * nside) + off for off in (3.0, 0.0, 0.0))
    return Workload("rows", nside, sky, [d])


@pytest.mark.parametrize("dtype", [np.float64, np.float32])
@pytest.mark.parametrize("nside,rings", [(1, 3.0), (8, 15.99), (64, 5.0), (64, 15.99), (64, 16.01), (1024, 16.0)])
@pytest.mark.parametrize("n", [1, 3, 4, 5, 67])
def test_small_discs(conv, dtype, nside, rings, n):
    say(f"case: pixel rows {np.dtype(dtype).name} nside {nside} rings {rings} n {n}")
    from paper_1908_05662_amd import OUT_COUNT, OUT_STOKES, OUT_TOD

    conv.set_launch(algorithm=0)
    rho = min(rings / (3 * nside), 1.0)
    for norm, rmin in ((W.NORM_PER_SAMPLE, 0.0), (W.NORM_FIXED, 0.4 * rho)):
        w = _workload(nside, rho, n, norm, rmin)
        for beam in ("auto", "full"):
            load_workload(conv, w, dtype, beam=beam)
            for mode, omode in ((OUT_TOD, oracle.OUT_TOD), (OUT_STOKES, oracle.OUT_STOKES)):
                want = oracle_detector(w, 0, slice(None), dtype, out_mode=omode)
                if not np.abs(want).max() > 0:
                    continue
                got = conv.convolve(0, mode).cpu().numpy()
                static = conv.convolve_static(0, mode).cpu().numpy()
                assert np.array_equal(got, static)
                assert rel_err(got, want.reshape(got.shape)) <= TOL[dtype], (norm, beam, mode)
        count = conv.convolve(0, OUT_COUNT).cpu().numpy()
        th, ph = w.detectors[0].theta, w.detectors[0].phi
        if nside <= 64:
            t, p = oracle.pix2ang(nside, np.arange(12 * nside * nside))
            z, s = np.cos(t), np.sin(t)
            c = np.stack([s * np.cos(p), s * np.sin(p), z])
            b = np.stack([np.sin(th) * np.cos(ph), np.sin(th) * np.sin(ph), np.cos(th)], 1)
            dist = np.arccos(np.clip(b @ c, -1, 1))
            lo = ((dist < rho - 1e-7) & (dist >= rmin + 1e-7)).sum(1)
            hi = ((dist < rho + 1e-7) & (dist >= rmin - 1e-7)).sum(1)
            assert np.all(count >= lo) and np.all(count <= hi)


@pytest.mark.parametrize("n", [8192, 140_001])
def test_queue_walk(conv, n):
    """Waves own their first tile and pop the later ones: every tile is taken, for one and
    eight queues, tiles of 1 to 64 samples and few or many workgroups."""
    say(f"case: queue walk, {n} samples")
    w = _workload(16, 0.1, n, W.NORM_PER_SAMPLE)
    load_workload(conv, w, np.float64)
    ref = conv.convolve(0).cpu().numpy()
    idx = np.unique(np.concatenate([np.linspace(0, n - 1, 500).astype(np.int64), [0, 63, 64, n - 1]]))
    assert rel_err(ref[idx], oracle_detector(w, 0, idx, np.float64)) <= TOL[np.float64]
    for kw in ({"samples_per_tile": 1}, {"xcd_queues": 8}, {"xcd_queues": 8, "groups_per_cu": 1, "waves_per_group": 1},
               {"waves_per_group": 8, "samples_per_tile": 16}):
        conv.set_launch(algorithm=0, **kw)
        assert np.array_equal(conv.convolve(0).cpu().numpy(), ref), kw
