"""Performance cases: the work a user of the framework has it do, through its public entry points.

Six kinds of work, over the sizes the paper's simulations and this repository's workloads use:

  tod      one pass of pointing through the convolver (FP32 or FP64; one-grid or four-channel
           beams; with a half-wave plate; TOD or Stokes outputs), or, with "block", one block of a
           streaming program: new pointing handed over, then the allocation-free convolution
  apply    the far-sidelobe network evaluated over a pointing stream and added to a TOD
  grad     one batch of the network's training: loss and every gradient
  bin      TOD binned into I, Q, U maps (clear, accumulate per detector, solve)
  spectra  the angular power spectra (and a_lm) of maps, with Jacobi refinement steps
  synth    maps from a_lm

`prepare` makes inputs on the GPU from the seed; `exact` evaluates the same definitions in 64 bits
with plain torch and numpy.
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_1908_05662_amd import NORM_FIXED, NORM_PER_SAMPLE, OUT_STOKES, OUT_TOD
from paper_1908_05662_amd.api import Convolver, MapMaker, Mlp, Spectra

DEG = math.pi / 180.0
FWHM_TO_SIGMA = 1.0 / math.sqrt(8.0 * math.log(2.0))
#: (sample, pixel) pairs up to which `exact` evaluates a convolution (about ten seconds)
EXACT_PAIRS = 4e9
RCOND_MIN = 1e-3


def _tod(name, **kw):
    c = {"name": name, "kind": "tod", "nside": 1024, "detectors": 1, "samples": 1000, "disc_deg": 2.0, "inner_deg": 0.0,
         "grid": 201, "fwhm_deg": 0.5, "ring": False, "beam": "scalar", "plate": False, "scan": "ces", "dtype": "f32",
         "out": "tod", "block": False}
    c.update(kw)
    return c


def listed():
    return [
        # a serving loop that simulates a detector as it scans: ten seconds of 100 Hz data per call
        _tod("stream_block", nside=512, samples=1024, block=True),
        # the whole-experiment run: 64 detectors of a focal plane, ragged streams of 1e5 to 1e6 samples
        _tod("focal_plane", detectors=64, samples=1_000_000),
        # measured beams with cross-polar leakage: four independent channels per detector
        _tod("full_beam", nside=512, detectors=16, samples=65_537, beam="full"),
        # a modulated experiment: a rotating half-wave plate before every detector
        _tod("plate", nside=1024, detectors=16, samples=100_000, plate=True),
        # a validation run in double precision: coarse sky, wide beam, pointings all over the sky
        _tod("double", nside=64, samples=100_000, disc_deg=4.5, grid=101, fwhm_deg=1.5, scan="sweep", dtype="f64"),
        # training targets of the far-sidelobe network: Stokes pickup of a wide annulus at random pointings
        _tod("annulus", nside=256, samples=65_536, disc_deg=20.0, inner_deg=5.0, grid=401, fwhm_deg=1.0, ring=True,
             scan="sphere", out="stokes"),
        # the paper's benchmark: a detector pair at every nside-128 pixel centre and three angles
        _tod("whole_sky", nside=128, detectors=2, samples=589_824, disc_deg=10.0, fwhm_deg=1.5, scan="centres"),
        # the network in place of the far sidelobe over a million samples
        {"name": "network", "kind": "apply", "width": 256, "layers": 4, "samples": 1_000_000},
        # one training batch of the full-scale network
        {"name": "training", "kind": "grad", "width": 512, "layers": 10, "batch": 8192},
        # the map of a modulated focal plane's TOD
        {"name": "maps", "kind": "bin", "nside": 1024, "detectors": 16, "samples": 250_000, "plate": True,
         "scan": "ces", "dtype": "f32"},
        # spectra of the paper's nside-128 output maps, refined as its estimator refines them
        {"name": "spectra_small", "kind": "spectra", "nside": 128, "lmax": 383, "pol": True, "iterations": 3},
        # spectra of the experiment's nside-1024 maps, one pass
        {"name": "spectra_large", "kind": "spectra", "nside": 1024, "lmax": 3071, "pol": True, "iterations": 0},
    ]


def _log(rng, lo, hi):
    return math.exp(rng.uniform(math.log(lo), math.log(hi)))


def draw(rng):
    kind = rng.choices(["tod", "block", "apply", "grad", "bin", "spectra", "synth"], [8, 2, 2, 2, 2, 3, 1])[0]
    if kind in ("tod", "block"):
        dtype = "f64" if kind == "tod" and rng.random() < 0.2 else "f32"
        nside = rng.choice([64, 128, 256] if dtype == "f64" else [128, 256, 512, 1024, 2048])
        # discs of about 60 to 20000 pixels, between half a degree and twenty
        pixels = _log(rng, 60.0, 20_000.0)
        disc = min(20.0, max(0.5, math.acos(max(-1.0, 1.0 - 2.0 * pixels / (12.0 * nside * nside))) / DEG))
        disc = round(disc, 2)
        case = _tod("", nside=nside, disc_deg=disc, grid=2 * rng.randrange(25, 201) + 1,
                    fwhm_deg=round(disc / rng.uniform(3.0, 6.0), 3), dtype=dtype,
                    beam="full" if rng.random() < 0.25 else "scalar", plate=rng.random() < 0.2,
                    scan=rng.choice(["ces", "ces", "sweep", "sphere"]), block=kind == "block")
        if rng.random() < 0.2:
            case.update(out="stokes", plate=False)
        pairs = _log(rng, 1e5, 2e9 if dtype == "f64" else 2e10)
        if kind == "block":
            case.update(scan="ces", samples=max(1, int(_log(rng, 50, 30_000))))
        else:
            case["detectors"] = rng.choice([1, 1, 2, 4, 16])
            case["samples"] = max(1, min(int(pairs / _disc_pixels(case) / case["detectors"]), 3_000_000))
        del case["name"]
        return case
    if kind == "apply":
        return {"kind": kind, "width": 64 * rng.randrange(1, 9), "layers": rng.randrange(2, 11),
                "samples": int(_log(rng, 300, 1_000_000))}
    if kind == "grad":
        return {"kind": kind, "width": 64 * rng.randrange(1, 9), "layers": rng.randrange(2, 11),
                "batch": 64 * int(_log(rng, 2, 256))}
    if kind == "bin":
        # a scan's consecutive samples share a pixel and, without a plate, an angle: the condition number of such a
        # pixel is rounding noise, so scans are modulated here; random pointings are not always
        scan = rng.choice(["ces", "ces", "sphere"])
        return {"kind": kind, "nside": rng.choice([64, 128, 256, 512, 1024]), "detectors": rng.choice([1, 2, 8]),
                "samples": int(_log(rng, 3_000, 1_000_000)), "plate": scan == "ces" or rng.random() < 0.3,
                "scan": scan, "dtype": rng.choice(["f32", "f64"])}
    nside = rng.choice([16, 32, 64, 128, 256, 512])
    case = {"kind": kind, "nside": nside, "lmax": int(nside * rng.uniform(1.0, 4.0)), "pol": rng.random() < 0.75}
    if kind == "spectra":
        case["iterations"] = rng.choice([0, 0, 1, 3])
    return case


# -- inputs -----------------------------------------------------------------------------------


def _generator(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(0x9E3779B1 * (int(seed) + 1) % (1 << 62))
    return g


def _rand(g, n):
    return torch.rand(n, generator=g, device="cuda", dtype=torch.float64)


def _dtype(case):
    return torch.float64 if case["dtype"] == "f64" else torch.float32


def _ring_table(nside):
    """Per RING-scheme ring (Gorski et al. 2005): z, sin theta, pixel count, first pixel, first longitude (numpy)."""
    n = int(nside)
    i = np.arange(1, 4 * n, dtype=np.int64)
    k = np.minimum(np.minimum(i, 4 * n - i), n)
    cap = (i < n) | (i > 3 * n)
    t = k.astype(np.float64) ** 2 / (3.0 * n * n)
    z = np.where(cap, np.where(i < n, 1.0 - t, t - 1.0), (4.0 * n - 2.0 * i) / (3.0 * n))
    s = np.sqrt(np.where(cap, t * (2.0 - t), (2.0 * i - n) * (7.0 * n - 2.0 * i) / (9.0 * n * n)))
    count = 4 * k
    first = np.concatenate([[0], np.cumsum(count)[:-1]])
    shifted = cap | (((i - n) & 1) == 0)
    phi0 = np.where(shifted, math.pi / count, 0.0)
    return z, s, count, first, phi0


def _maps(nside, g, dtype, fields=3):
    """Stokes maps: I of order one with large-scale structure and pixel noise, Q and U a tenth of that."""
    z, s, count, first, phi0 = _ring_table(nside)
    reps = torch.from_numpy(count).cuda()
    zz = torch.repeat_interleave(torch.from_numpy(z).cuda(), reps)
    out = []
    for f in range(fields):
        c = torch.randn(3, generator=g, device="cuda", dtype=torch.float64)
        m = 0.3 * torch.randn(zz.numel(), generator=g, device="cuda", dtype=torch.float64)
        m += c[0] + c[1] * zz + c[2] * zz * zz
        out.append(((1.0 if f == 0 else 0.1) * m).to(dtype))
    return out


def _counts(case):
    """Samples of each detector: a full stream for one, ragged from a tenth up for several."""
    n, k = case["samples"], case["detectors"]
    if k == 1 or case["scan"] == "centres":
        return [n] * k
    return [max(1, int(n * (0.1 + 0.9 * ((i * 0.6180339887) % 1.0)))) for i in range(k)]


def _pointing(case, n, k, g):
    """theta, phi, psi (float64, GPU) of detector k."""
    if case["scan"] == "centres":
        z, s, count, first, phi0 = _ring_table(case["nside"])
        reps = torch.from_numpy(count).cuda()
        ring = torch.repeat_interleave(torch.arange(len(z), device="cuda"), reps)
        j = torch.arange(ring.numel(), device="cuda") - torch.from_numpy(first).cuda()[ring]
        th = torch.acos(torch.from_numpy(z).cuda())[ring]
        ph = torch.from_numpy(phi0).cuda()[ring] + 2.0 * math.pi * j.double() / reps[ring]
        i = torch.arange(n, device="cuda")
        return th[i % th.numel()], ph[i % ph.numel()], (i // th.numel()).double() * (45.0 * DEG) + _rand(g, 1)
    if case["scan"] in ("sphere", "sweep"):
        psi = 2.0 * math.pi * _rand(g, n)
        if case["scan"] == "sphere":
            return torch.acos(2.0 * _rand(g, n) - 1.0), 2.0 * math.pi * _rand(g, n), psi
        dec = 60.0 * DEG * (2.0 * _rand(g, n) - 1.0)
        return 0.5 * math.pi - dec, 2.0 * math.pi * torch.arange(n, device="cuda", dtype=torch.float64) / n, psi
    # constant-elevation scan: 720 deg sweeps at 0.01 deg a sample, 100 Hz, boresight steps of 15 deg
    r = _rand(g, 3).tolist()
    t = torch.arange(n, device="cuda", dtype=torch.float64) + int(2_000_000 * r[0])
    lat = (2.0 * r[1] - 1.0) * 45.0 * DEG
    half = 72_000.0
    ph = torch.remainder(t, 2.0 * half)
    az = torch.where(ph < half, ph, 2.0 * half - ph) * (0.01 * DEG) + 0.7 * DEG * (k % 8 - 3.5)
    el = 45.0 * DEG + 0.7 * DEG * (k // 8 % 8 - 3.5)
    lst = 2.0 * math.pi * (r[2] + t / 100.0 / 86164.0905)
    sl, cl, se, ce = math.sin(lat), math.cos(lat), math.sin(el), math.cos(el)
    dec = torch.asin((se * sl + ce * cl * torch.cos(az)).clamp(-1.0, 1.0))
    ha = torch.atan2(-torch.sin(az) * ce, se * cl - ce * sl * torch.cos(az))
    q = torch.atan2(torch.sin(ha), math.tan(lat) * torch.cos(dec) - torch.sin(dec) * torch.cos(ha))
    step = (torch.floor(t / 100_000.0) % 7.0 - 3.0) * (15.0 * DEG)
    return 0.5 * math.pi - dec, torch.remainder(lst - ha, 2.0 * math.pi), torch.remainder(q + step, 2.0 * math.pi)


def _plate_angle(n, g):
    """A plate turning twice a second at 100 Hz sampling."""
    t = torch.arange(n, device="cuda", dtype=torch.float64)
    return torch.remainder(2.0 * math.pi * (t * 0.02) + 2.0 * math.pi * _rand(g, 1), 2.0 * math.pi)


def _beam(case, g):
    """Channel grids [v][u] of one detector: b alone, or (bI, bQ, bU, bT)."""
    n, T = case["grid"], math.tan(case["disc_deg"] * DEG)
    ax = torch.linspace(-T, T, n, device="cuda", dtype=torch.float64)
    v, u = torch.meshgrid(ax, ax, indexing="ij")
    rho, sig = torch.atan(torch.hypot(u, v)), torch.atan2(v, u)
    e, orient = (_rand(g, 2) * torch.tensor([0.1, math.pi], device="cuda", dtype=torch.float64)).tolist()
    s0, r = case["fwhm_deg"] * DEG * FWHM_TO_SIGMA, math.sqrt((1.0 + e) / (1.0 - e))
    x, y = rho * torch.cos(sig - orient), rho * torch.sin(sig - orient)
    b = torch.exp(-0.5 * ((x / (s0 * r)) ** 2 + (y * r / s0) ** 2))
    if case["ring"]:
        b = b + 1e-4 * torch.exp(-0.5 * ((rho - 0.5 * case["disc_deg"] * DEG) / (2.0 * DEG * FWHM_TO_SIGMA)) ** 2)
    b = b.to(_dtype(case))
    if case["beam"] == "scalar":
        return b
    cross = (0.01 * b * torch.cos(2.0 * sig)).to(b.dtype)
    eps = 1e-3
    return [(0.5 * (1.0 + eps) * b), (0.5 * (1.0 - eps) * b), (0.5 * (1.0 - eps) * cross), b]


def _weights():
    """(wI, wQ, wU, wT) of a one-grid detector with polarisation efficiency 1 - 1e-3."""
    return 0.5 * 1.001, 0.5 * 0.999, 0.0, 1.0


def _zeta(case, k):
    if case["out"] == "stokes":
        return 0.0
    return ((0.0 if (k // 2) % 2 == 0 else 45.0) - (90.0 if k % 2 else 0.0)) * DEG


def _norm(case):
    """A fixed constant for the sidelobe annulus (pixel over beam solid angle), else unit normalisation per sample."""
    if case["inner_deg"] > 0.0:
        s0 = case["fwhm_deg"] * DEG * FWHM_TO_SIGMA
        return NORM_FIXED, 4.0 * math.pi / (12.0 * case["nside"] ** 2) / (2.0 * math.pi * s0 * s0)
    return NORM_PER_SAMPLE, 1.0


def _tod_inputs(case, seed):
    g = _generator(seed)
    sky = _maps(case["nside"], g, _dtype(case))
    dets = []
    for k, n in enumerate(_counts(case)):
        d = {"beam": _beam(case, g), "pointing": _pointing(case, n, k, g), "zeta": _zeta(case, k)}
        d["plate"] = _plate_angle(n, g) if case["plate"] else None
        dets.append(d)
    return sky, dets


def _network_params(case, seed):
    """Weights of the scale a trained network has: 1.5 / sqrt(fan in), small biases (one float32 array, W_l then b_l)."""
    g = _generator(seed + 7)
    dims = [5] + [case["width"]] * case["layers"] + [3]
    parts = []
    for a, b in zip(dims, dims[1:]):
        parts.append(torch.randn(a * b, generator=g, device="cuda") * (1.5 / math.sqrt(a)))
        parts.append(torch.randn(b, generator=g, device="cuda") * 0.1)
    return torch.cat(parts), dims


def _grad_inputs(case, seed):
    g = _generator(seed)
    x = _features(torch.acos(2.0 * _rand(g, case["batch"]) - 1.0), 2.0 * math.pi * _rand(g, case["batch"]),
                  2.0 * math.pi * _rand(g, case["batch"])).float().contiguous()
    t = torch.randn(case["batch"], 3, generator=g, device="cuda")
    return x, t


def _features(th, ph, ps):
    return torch.stack([torch.sin(th) * torch.cos(ph), torch.sin(th) * torch.sin(ph), torch.cos(th), torch.sin(ps),
                        torch.cos(ps)], 1)


APPLY_SCALES = ([0.1, -0.2, 0.3], [0.5, 1.5, 0.7], [0.5, 0.25, -0.125])   # mean, std, coef


def _bin_inputs(case, seed):
    g = _generator(seed)
    dets = []
    for k, n in enumerate(_counts(case)):
        p = _pointing(case, n, k, g)
        tod = (1.0 + 0.3 * torch.randn(n, generator=g, device="cuda", dtype=torch.float64)).to(_dtype(case))
        zeta = ((0.0 if (k // 2) % 2 == 0 else 45.0) - (90.0 if k % 2 else 0.0)) * DEG
        dets.append((p, tod, zeta, _plate_angle(n, g) if case["plate"] else None))
    return dets


def _alm_inputs(case, seed):
    """a_lm with a falling spectrum, m-major, a_l0 real, E and B without l < 2."""
    g = _generator(seed)
    lmax = case["lmax"]
    m = torch.repeat_interleave(torch.arange(lmax + 1, device="cuda"), torch.arange(lmax + 1, 0, -1, device="cuda"))
    first = m * (2 * lmax + 1 - m) // 2
    l = torch.arange(m.numel(), device="cuda") - first
    out = []
    for f in range(3 if case["pol"] else 1):
        a = torch.complex(torch.randn(m.numel(), generator=g, device="cuda", dtype=torch.float64),
                          torch.randn(m.numel(), generator=g, device="cuda", dtype=torch.float64))
        a = a / (l.double() + 1.0)
        a = torch.where(m == 0, torch.complex(a.real, torch.zeros_like(a.real)), a)
        out.append(torch.where(l < 2, torch.zeros_like(a), a) if f else a)
    return out


def prepare(case, seed):
    kind = case["kind"]
    conv = Convolver(0)
    state = {"kind": kind, "conv": conv}
    if kind == "tod":
        sky, dets = _tod_inputs(case, seed)
        dtype = _dtype(case)
        conv.set_sky(case["nside"], *sky, dtype=dtype)
        T = math.tan(case["disc_deg"] * DEG)
        mode, scale = _norm(case)
        for k, d in enumerate(dets):
            if case["beam"] == "scalar":
                conv.set_beam_scalar(k, case["grid"], T, d["beam"], *_weights(), dtype=dtype)
            else:
                conv.set_beam(k, case["grid"], T, *d["beam"], dtype=dtype)
            conv.set_detector(k, d["zeta"], case["inner_deg"] * DEG, case["disc_deg"] * DEG, mode, scale)
            conv.set_pointing(k, *d["pointing"])
            if d["plate"] is not None:
                conv.set_hwp(k, d["plate"])
        state["block"] = dets[0]["pointing"] if case["block"] else None
        state["mode"] = OUT_STOKES if case["out"] == "stokes" else OUT_TOD
    elif kind == "apply":
        g = _generator(seed)
        # the network reads a ready detector's pointing: any sky and beam make one
        conv.set_sky(16, *(torch.zeros(12 * 16 * 16, device="cuda") for _ in range(3)), dtype=torch.float32)
        conv.set_beam_scalar(0, 3, 0.1, torch.ones(9, device="cuda"), *_weights(), dtype=torch.float32)
        conv.set_detector(0, 0.0, 0.0, 0.05, NORM_PER_SAMPLE, 1.0)
        conv.set_pointing(0, *_pointing({"scan": "sphere"}, case["samples"], 0, g))
        state["net"] = Mlp(conv, case["width"], case["layers"], max_batch=64, seed=1)
        state["net"].set_params(_network_params(case, seed)[0])
        state["tod"] = torch.randn(case["samples"], generator=g, device="cuda")
    elif kind == "grad":
        state["net"] = Mlp(conv, case["width"], case["layers"], max_batch=case["batch"], seed=1)
        state["net"].set_params(_network_params(case, seed)[0])
        state["x"], state["t"] = _grad_inputs(case, seed)
    elif kind == "bin":
        state["dets"] = _bin_inputs(case, seed)
        state["maker"] = MapMaker(conv, case["nside"])
    else:
        state["sp"] = Spectra(conv, case["nside"], case["lmax"], case["pol"])
        if kind == "spectra":
            state["maps"] = _maps(case["nside"], _generator(seed), torch.float64, 3 if case["pol"] else 1)
            state["iterations"] = case["iterations"]
        else:
            state["alm"] = _alm_inputs(case, seed)
    return state


def run(state):
    kind = state["kind"]
    if kind == "tod":
        if state["block"] is not None:
            state["conv"].set_pointing(0, *state["block"])
            return state["conv"].convolve_static(0, state["mode"])
        return state["conv"].convolve(-1, state["mode"])
    if kind == "apply":
        return state["net"].apply(0, *APPLY_SCALES, state["tod"].clone())
    if kind == "grad":
        return state["net"].gradient(state["x"], state["t"])
    if kind == "bin":
        mk = state["maker"]
        mk.clear()
        for (th, ph, ps), tod, zeta, plate in state["dets"]:
            mk.add(th, ph, ps, tod, zeta=zeta, eps=1e-3, hwp=plate)
        maps, rcond = mk.solve(RCOND_MIN)
        return {"maps": maps, "rcond": rcond, "sums": mk.accum}
    if kind == "spectra":
        cl = state["sp"].anafast(*state["maps"], iterations=state["iterations"])
        return {"cl": cl, "alm": list(state["sp"].alm)}
    return [m for m in state["sp"].alm2map(*state["alm"]) if m is not None]


# -- the work no implementation can do without --------------------------------------------------


def _disc_pixels(case):
    caps = math.cos(case["inner_deg"] * DEG) - math.cos(case["disc_deg"] * DEG)
    return max(1.0, 6.0 * case["nside"] ** 2 * caps)


def work(case):
    kind = case["kind"]
    if kind == "tod":
        word = 8 if case["dtype"] == "f64" else 4
        n, width = sum(_counts(case)), 3 if case["out"] == "stokes" else 1
        channels = 4 if case["beam"] == "full" else 1
        sky = min(12.0 * case["nside"] ** 2, n * _disc_pixels(case)) * 3 * word
        beams = case["detectors"] * channels * word * case["grid"] ** 2
        # per pair: offsets and projection 15, cell lookup and interpolation 12 (9 more a channel), angle and terms 20
        flops = 47.0 + 9.0 * (channels - 1) + (6.0 if case["plate"] else 0.0)
        return {"bytes": sky + beams + n * (24.0 + word * width + (8.0 if case["plate"] else 0.0)),
                "flops": flops * n * _disc_pixels(case)}
    if kind == "apply":
        h, n = case["width"], case["samples"]
        macs = 5 * h + (case["layers"] - 1) * h * h + 3 * h
        return {"bytes": n * 32.0 + 2.0 * macs, "flops": 2.0 * macs * n}
    if kind == "grad":
        h, n = case["width"], case["batch"]
        macs = 5 * h + (case["layers"] - 1) * h * h + 3 * h
        return {"bytes": 6.0 * macs + n * 32.0, "flops": 6.0 * macs * n}
    npix = 12.0 * case["nside"] ** 2
    if kind == "bin":
        n = sum(_counts(case))
        return {"bytes": n * (24.0 + (8 if case["dtype"] == "f64" else 4) + (8.0 if case["plate"] else 0.0)) + npix * 112.0,
                "flops": 60.0 * n}
    fields, lmax = 3 if case["pol"] else 1, case["lmax"]
    nalm = 0.5 * (lmax + 1) * (lmax + 2)
    passes = 1 if kind == "synth" else 1 + 2 * case["iterations"]
    # recurrence 4 flops and 4 a field component's real and imaginary sums; spin-2 functions 8 more
    per = 8.0 + (8.0 + 16.0 if case["pol"] else 0.0)
    return {"bytes": fields * (8.0 * npix + 16.0 * nalm), "flops": passes * per * nalm * 2.0 * case["nside"]}


# -- the same definitions in 64 bits ------------------------------------------------------------


def exact(case, seed):
    kind = case["kind"]
    if kind == "tod":
        return _exact_tod(case, seed) if sum(_counts(case)) * _disc_pixels(case) <= EXACT_PAIRS else None
    if kind == "apply":
        g = _generator(seed)
        p = _pointing({"scan": "sphere"}, case["samples"], 0, g)
        tod = torch.randn(case["samples"], generator=g, device="cuda").double()
        mean, std, coef = (torch.tensor(v, device="cuda", dtype=torch.float64) for v in APPLY_SCALES)
        out = []
        for lo in range(0, case["samples"], 1 << 16):
            y = _network(case, seed, _features(*(t[lo:lo + (1 << 16)] for t in p)))[0]
            out.append(tod[lo:lo + (1 << 16)] + ((mean + std * y) * coef).sum(1))
        return torch.cat(out)
    if kind == "grad":
        x, t = _grad_inputs(case, seed)
        y, params = _network(case, seed, x.double(), True)
        loss = ((y - t.double()) ** 2).mean()
        loss.backward()
        return loss.detach().reshape(1), params.grad
    if kind == "bin":
        return _exact_bin(case, seed)
    if kind == "spectra":
        if case["nside"] >= 512 and case["iterations"] > 0:
            return None
        maps = _maps(case["nside"], _generator(seed), torch.float64, 3 if case["pol"] else 1)
        alm = _analysis(case, maps)
        for _ in range(case["iterations"]):
            back = _synthesis(case, alm)
            alm = [a + d for a, d in zip(alm, _analysis(case, [m - b for m, b in zip(maps, back)]))]
        return {"cl": _spectra(case["lmax"], alm), "alm": alm}
    return _synthesis(case, _alm_inputs(case, seed))


def _network(case, seed, x, grad=False):
    flat, dims = _network_params(case, seed)
    flat = flat.double().requires_grad_(grad)
    o, a = 0, x
    for i, (n_in, n_out) in enumerate(zip(dims, dims[1:])):
        w = flat[o:o + n_in * n_out].reshape(n_out, n_in)
        b = flat[o + n_in * n_out:o + n_in * n_out + n_out]
        o += n_in * n_out + n_out
        a = a @ w.t() + b
        if i < len(dims) - 2:
            a = a * torch.sigmoid(a)
    return a, flat


def _vectors(th, ph):
    st, ct, sp, cp = torch.sin(th), torch.cos(th), torch.sin(ph), torch.cos(ph)
    return (torch.stack([st * cp, st * sp, ct], -1), torch.stack([ct * cp, ct * sp, -st], -1),
            torch.stack([-sp, cp, torch.zeros_like(sp)], -1))


def _flatten(counts):
    """(owner, place) of `counts[i]` entries for each i."""
    owner = torch.repeat_interleave(torch.arange(counts.numel(), device="cuda"), counts)
    start = torch.cumsum(counts, 0) - counts
    return owner, torch.arange(owner.numel(), device="cuda") - start[owner]


def _exact_tod(case, seed):
    sky, dets = _tod_inputs(case, seed)
    sky = [m.double() for m in sky]
    z, s, count, first, phi0 = (torch.from_numpy(a).cuda() for a in _ring_table(case["nside"]))
    ring_th = torch.atan2(s, z)
    rmax, rmin = case["disc_deg"] * DEG, case["inner_deg"] * DEG
    T, n = math.tan(rmax), case["grid"]
    h = 2.0 * T / (n - 1)
    mode, scale = _norm(case)
    step = max(1, int(6e6 / _disc_pixels(case) / 1.4))
    out = []
    for d in dets:
        beams = d["beam"] if isinstance(d["beam"], list) else [d["beam"]]
        beams = [b.double().reshape(-1) for b in beams]
        th_all, ph_all, ps_all = d["pointing"]
        cz, sz = math.cos(d["zeta"]), math.sin(d["zeta"])
        for lo in range(0, th_all.numel(), step):
            th, ph, ps = (t[lo:lo + step] for t in (th_all, ph_all, ps_all))
            # candidate pixels: rings within the disc's colatitudes, on each the longitudes the cap can reach
            r0 = torch.searchsorted(ring_th, th - rmax - 1e-9)
            r1 = torch.searchsorted(ring_th, th + rmax + 1e-9, right=True)
            own, place = _flatten(r1 - r0)
            ring = r0[own] + place
            st = torch.sin(th)[own] * s[ring]
            c = (math.cos(rmax) - torch.cos(th)[own] * z[ring]) / st.clamp_min(1e-300)
            half = torch.acos(c.clamp(-1.0, 1.0)) + 1e-6
            dphi = 2.0 * math.pi / count[ring].double()
            j0 = torch.floor((ph[own] - half - phi0[ring]) / dphi).long()
            j1 = torch.ceil((ph[own] + half - phi0[ring]) / dphi).long()
            many = torch.minimum(j1 - j0 + 1, count[ring])
            lengths = torch.zeros_like(r0).index_add(0, own, many)
            own2, place2 = _flatten(many)
            t, ring = own[own2], ring[own2]
            j = torch.remainder(j0[own2] + place2, count[ring])
            pixel = first[ring] + j
            pp, pt, pf = _vectors(ring_th[ring], phi0[ring] + 2.0 * math.pi * j.double() / count[ring])
            p, a, b = _vectors(th, ph)
            cs, sn = torch.cos(ps)[:, None], torch.sin(ps)[:, None]
            tp, fp = cs * a + sn * b, cs * b - sn * a
            dot = (pp * p[t]).sum(-1)
            keep = dot >= math.cos(rmax)
            if rmin > 0.0:
                keep &= dot < math.cos(rmin)
            dot = torch.where(keep, dot, 1.0)
            x, y = (pp * tp[t]).sum(-1), (pp * fp[t]).sum(-1)
            # the boresight's theta' carried along the great circle to the pixel
            e = tp[t] - (x / (1.0 + dot))[:, None] * (p[t] + pp)
            cg, sg = (e * pt).sum(-1), (e * pf).sum(-1)
            cx, sx = cg * cz - sg * sz, sg * cz + cg * sz
            c2, s2 = cx * cx - sx * sx, 2.0 * cx * sx
            u, v = (x / dot + T) / h, (y / dot + T) / h
            inside = keep & (u >= 0) & (u <= n - 1) & (v >= 0) & (v <= n - 1)
            iu, iv = (w.floor().clamp(0, n - 2).long() for w in (u, v))
            fu, fv, base = u - iu, v - iv, iv * n + iu
            vals = [inside * ((g[base] * (1 - fu) + g[base + 1] * fu) * (1 - fv)
                              + (g[base + n] * (1 - fu) + g[base + n + 1] * fu) * fv) for g in beams]
            if len(vals) == 1:
                vals = [w * vals[0] for w in _weights()]
            si, sq, su = (m[pixel] for m in sky)
            if case["plate"]:
                f4 = 4.0 * d["plate"][lo:lo + step][t]
                c2, s2 = c2 * torch.cos(f4) - s2 * torch.sin(f4), s2 * torch.cos(f4) + c2 * torch.sin(f4)
            rq, ru = c2 * sq + s2 * su, c2 * su - s2 * sq
            if case["out"] == "stokes":
                terms = [vals[3] * si, vals[3] * rq, vals[3] * ru]
            else:
                terms = [vals[0] * si + vals[1] * rq + (-1.0 if case["plate"] else 1.0) * vals[2] * ru]
            sums = [torch.segment_reduce(w, "sum", lengths=lengths, axis=0, unsafe=True) for w in terms]
            if mode == NORM_PER_SAMPLE:
                nb = torch.segment_reduce(vals[3], "sum", lengths=lengths, axis=0, unsafe=True)
                sums = [torch.where(nb != 0.0, scale * w / torch.where(nb != 0.0, nb, 1.0), 0.0) for w in sums]
            else:
                sums = [scale * w for w in sums]
            out.append(torch.stack(sums, -1) if len(sums) == 3 else sums[0])
    return torch.cat(out)


def _ring_pixel(nside, th, ph):
    """RING pixel holding each direction (Gorski et al. 2005, Sec. 4)."""
    z = torch.cos(th)
    t = torch.remainder(ph * (2.0 / math.pi), 4.0)
    up = torch.floor(nside * (0.5 + t) - 0.75 * nside * z).long()
    dn = torch.floor(nside * (0.5 + t) + 0.75 * nside * z).long()
    r = nside + 1 + up - dn
    k = torch.remainder((up + dn - nside + 1 + (1 - (r & 1))) >> 1, 4 * nside)
    belt = 2 * nside * (nside - 1) + (r - 1) * 4 * nside + k
    w = nside * torch.sqrt(3.0 * (1.0 - z.abs()))
    tp = t - torch.floor(t)
    rc = (torch.floor(tp * w) + torch.floor((1.0 - tp) * w) + 1).long().clamp(max=nside)
    kc = torch.remainder(torch.floor(t * rc).long(), 4 * rc)
    cap = torch.where(z > 0, 2 * rc * (rc - 1) + kc, 12 * nside * nside - 2 * rc * (rc + 1) + kc)
    return torch.where(z.abs() <= 2.0 / 3.0, belt, cap)


def _exact_bin(case, seed):
    nside = case["nside"]
    npix = 12 * nside * nside
    sums = torch.zeros(npix, 10, device="cuda", dtype=torch.float64)
    for (th, ph, ps), tod, zeta, plate in _bin_inputs(case, seed):
        a = 2.0 * (ps + zeta) + (0.0 if plate is None else 4.0 * plate)
        w = [torch.full_like(a, 0.5 * 1.001), 0.5 * 0.999 * torch.cos(a), 0.5 * 0.999 * torch.sin(a)]
        d = tod.double()
        rows = [w[0] * w[0], w[0] * w[1], w[0] * w[2], w[1] * w[1], w[1] * w[2], w[2] * w[2], w[0] * d, w[1] * d, w[2] * d,
                torch.ones_like(d)]
        sums.index_add_(0, _ring_pixel(nside, th, ph), torch.stack(rows, 1))
    hit = torch.nonzero(sums[:, 9] > 0).reshape(-1)
    A = sums[hit].cpu().numpy()
    M = A[:, [0, 1, 2, 1, 3, 4, 2, 4, 5]].reshape(-1, 3, 3)
    ev = np.linalg.eigvalsh(M)
    rc = ev[:, 0] / ev[:, 2]
    m = np.zeros((3, hit.numel()))
    m[0] = A[:, 6] / A[:, 0]
    good = rc >= RCOND_MIN
    m[:, good] = np.linalg.solve(M[good], A[good, 6:9, None])[:, :, 0].T
    maps = torch.zeros(3, npix, device="cuda", dtype=torch.float64)
    maps[:, hit] = torch.from_numpy(m).cuda()
    # rcond: exactly 0 in every pixel hit once, where double precision gives rounding noise
    return {"maps": maps, "rcond": None, "sums": sums.reshape(-1)}


def _legendre(case, visit):
    """Calls visit(j, lam, W, X) for j = l - m = 0..lmax: the harmonics' colatitude functions of every m <= lmax - j (rows)
    on the north rings and the equator (columns); W and X (spin 2) None without polarisation."""
    N, lmax = case["nside"], case["lmax"]
    z, s = (torch.from_numpy(a[:2 * N]).cuda() for a in _ring_table(N)[:2])
    m = torch.arange(lmax + 1, device="cuda", dtype=torch.float64)[:, None]
    k = torch.arange(1, lmax + 1, device="cuda", dtype=torch.float64)
    c = torch.cat([torch.ones(1, device="cuda", dtype=torch.float64), torch.cumprod((2 * k + 1) / (2 * k), 0)])
    lg = m * (torch.log(s) / math.log(2.0)) + 0.5 * torch.log2(c / (4.0 * math.pi))[:, None]
    e = torch.floor(lg / 256.0)
    v = torch.exp2(lg - 256.0 * e) * (1.0 - 2.0 * torch.remainder(m, 2.0))
    vp = torch.zeros_like(v)
    s2 = s * s
    for j in range(lmax + 1):
        rows = lmax + 1 - j
        mm = m[:rows]
        l = mm + j
        v, vp, e = v[:rows], vp[:rows], e[:rows]
        if j > 0:
            a = torch.sqrt((4 * l * l - 1) / (l * l - mm * mm))
            b = torch.sqrt(((l - 1) ** 2 - mm * mm).clamp_min(0.0) / (4 * (l - 1) ** 2 - 1)) if j > 1 else 0.0
            v, vp = a * (z * v - b * vp), v
            big = v.abs() > 2.0 ** 256
            if bool(big.any()):
                f = torch.exp2(-256.0 * big.double())
                v, vp, e = v * f, vp * f, e + big
        f = torch.exp2(256.0 * e.clamp_min(-4.0))
        lam, lamp = v * f, vp * f
        W = X = None
        if case["pol"]:
            nl = torch.where(l >= 2, 2.0 / torch.sqrt(((l - 1) * l * (l + 1) * (l + 2)).clamp_min(1.0)), 0.0)
            cl = torch.sqrt((2 * l + 1) * j / ((2 * l - 1).clamp_min(1.0) * (l + mm).clamp_min(1.0)))
            W = nl * (-((l - mm * mm) / s2 + l * (l - 1) / 2) * lam + (l + mm) * cl * (z / s2) * lamp)
            X = nl * (mm / s2) * (-(l - 1) * z * lam + (l + mm) * cl * lamp)
        visit(j, lam, W, X)


def _alm_places(lmax, j):
    m = torch.arange(lmax + 1 - j, device="cuda")
    return m * (2 * lmax + 1 - m) // 2 + m + j


def _analysis(case, maps):
    N, lmax = case["nside"], case["lmax"]
    _, _, count, first, phi0 = _ring_table(N)
    m = np.arange(lmax + 1)
    halves = []                       # per field: north + south and north - south ring sums [m][ring]
    for x in maps:
        x = x.cpu().numpy()
        F = np.empty((4 * N - 1, lmax + 1), dtype=np.complex128)
        for r in range(4 * N - 1):
            F[r] = np.exp(-1j * m * phi0[r]) * np.fft.fft(x[first[r]:first[r] + count[r]])[m % count[r]]
        F = torch.from_numpy(F * (4.0 * math.pi / (12.0 * N * N))).cuda()
        north, south = F[:2 * N].t().contiguous(), F.flip(0)[:2 * N].t().contiguous()
        south[:, 2 * N - 1] = 0.0     # the equator is its own mirror
        halves.append((north + south, north - south))
    alm = [torch.zeros((lmax + 1) * (lmax + 2) // 2, device="cuda", dtype=torch.complex128) for _ in maps]

    def total(func, F):
        return torch.complex((func * F.real[:func.shape[0]]).sum(1), (func * F.imag[:func.shape[0]]).sum(1))

    def visit(j, lam, W, X):
        at, p = _alm_places(lmax, j), j & 1
        alm[0][at] = total(lam, halves[0][p])
        if case["pol"]:
            (Qa, Qb), (Ua, Ub) = ((h[p], h[1 - p]) for h in halves[1:])
            alm[1][at] = -(total(W, Qa) + 1j * total(X, Ub))
            alm[2][at] = -(total(W, Ua) - 1j * total(X, Qb))

    _legendre(case, visit)
    return alm


def _synthesis(case, alm):
    N, lmax = case["nside"], case["lmax"]
    _, _, count, first, phi0 = _ring_table(N)
    G = [[torch.zeros(lmax + 1, 2 * N, device="cuda", dtype=torch.complex128) for _ in range(2)] for _ in alm]

    def visit(j, lam, W, X):
        at, p, rows = _alm_places(lmax, j), j & 1, lmax + 1 - j
        a = [x[at][:, None] for x in alm]
        G[0][p][:rows] += a[0] * lam
        if case["pol"]:
            G[1][p][:rows] -= a[1] * W
            G[1][1 - p][:rows] -= 1j * a[2] * X
            G[2][p][:rows] -= a[2] * W
            G[2][1 - p][:rows] += 1j * a[1] * X

    _legendre(case, visit)
    m = np.arange(lmax + 1)
    out = []
    for even, odd in G:
        rings = torch.cat([(even + odd), (even - odd).flip(1)[:, 1:]], 1).t().contiguous().cpu().numpy()
        x = np.empty(12 * N * N)
        for r in range(4 * N - 1):
            n = int(count[r])
            h = np.where(m == 0, 1.0, 2.0) * rings[r] * np.exp(1j * m * phi0[r])
            h = np.concatenate([h, np.zeros(-len(h) % n, dtype=h.dtype)]).reshape(-1, n).sum(0)
            x[first[r]:first[r] + n] = (np.fft.ifft(h) * n).real
        out.append(torch.from_numpy(x).cuda())
    return out


def _spectra(lmax, alm):
    pairs = [(0, 0), (1, 1), (2, 2), (0, 1), (1, 2), (0, 2)] if len(alm) == 3 else [(0, 0)]
    cl = torch.zeros(len(pairs), lmax + 1, device="cuda", dtype=torch.float64)
    l = torch.arange(lmax + 1, device="cuda")
    m = torch.repeat_interleave(l, torch.arange(lmax + 1, 0, -1, device="cuda"))
    which = torch.arange(m.numel(), device="cuda") - m * (2 * lmax + 1 - m) // 2
    for i, (x, y) in enumerate(pairs):
        p = (alm[x] * alm[y].conj()).real * torch.where(m == 0, 1.0, 2.0)
        cl[i].index_add_(0, which, p)
    return cl / (2.0 * l.double() + 1.0)
