"""Performance cases of the RadioLensfit hot path on one MI355X.

Every case is one thing that a program using this package does over and over,
through the public binding (paper_2203_14071_amd.rlf): predict or subtract a
sky model, extract and fit a field, fit facets in the other modes the library
offers, run the serial refinement of the sky model, replay a captured pass,
form network inputs, train the network.  Sizes come from the package's
configurations (synth.CONFIGS: a 20-antenna array with 11,400 rows and 10
sources, the 9,266,880-row array with 1000 sources in FP64 and mixed
precision, the eight-channel field) and from reduced and ragged versions of
them; populations and noise are those configurations' own, the noise scaled
with the number of visibilities so that the sources keep their
signal-to-noise ratio.

listed() names the cases, draw() gives further ones of the same ranges,
prepare() makes what a program holds before the call, run() is one pass,
work() what a pass cannot do without, exact() its outputs in 64 bits.
"""
from __future__ import annotations

import dataclasses
import math

import numpy as np
import torch

from paper_2203_14071_amd import rlf, surrogate, synth

DEV = "cuda:0"
ARCSEC = math.pi / 648000.0
N_E, E_STEP, N_KNOTS, FRAC = 81, 0.02, 20, 0.05
N_GRID = 6333                       # grid points with |e| < 1 after the integer test (200-odd short of a circle's area)
MEAN_CELLS = {"tiny": 70, "mid": 300, "wide": 800}
FIT_KEYS = ("e1", "e2", "s1", "s2", "c12", "lmax")


# ---- the cases -----------------------------------------------------------------

def listed():
    return [
        # the smallest call: one residual of the 20-antenna array (a test field, or one step of an interactive session)
        dict(name="model_tiny_f64", op="model", field="tiny", rows=11400, chan=1, src=10, mixed=False, mode="residual"),
        # the residual of the 1000-source field, the first stage of a measurement
        dict(name="model_field_f64", op="model", field="mid", rows=9266880, chan=1, src=1000, mixed=False, mode="residual"),
        # simulating an eight-channel observation in mixed precision
        dict(name="model_8ch_mixed", op="model", field="wide", rows=579181, chan=8, src=1000, mixed=True, mode="write"),
        # measuring the shapes of the 10-source field in one go: sky model, extraction, full-grid fit
        dict(name="measure_tiny_f64", op="measure", field="tiny", rows=11400, chan=1, src=10, mixed=False, fused=True),
        # the same on a ragged few-channel observation with a few tiles of sources, replayed as a captured pass
        dict(name="pass_mid_f64", op="pass", field="mid", rows=400321, chan=2, src=150, mixed=False),
        # extraction and full-grid fit of the 1000-source field, the residual given
        dict(name="measure_field_f64", op="measure", field="mid", rows=9266880, chan=1, src=1000, mixed=False, fused=False),
        # the likelihood grid of the 1000-source field in mixed precision, surfaces kept
        dict(name="fit_field_mixed", op="fit", field="mid", rows=9266880, chan=1, src=1000, mixed=True, how="full",
             surface=True, noise=1.0),
        # the lattice-seeded narrowed fit on a part of the field
        dict(name="fit_lattice_f64", op="fit", field="mid", rows=1158361, chan=1, src=300, mixed=False, how="lattice",
             surface=False, noise=1.0),
        # bright, well-localised sources: position-marginalised fit and the adaptive refinement around the maximum
        dict(name="fit_positions_f64", op="fit", field="mid", rows=1158361, chan=1, src=100, mixed=False, how="positions",
             surface=False, noise=0.2),
        # the serial refinement of the sky model, one source at a time
        dict(name="sequential_f64", op="sequential", field="mid", rows=1158361, chan=1, src=24, mixed=False, chunk=1),
        # network inputs of an eight-channel field: sky model, extraction, feature rows
        dict(name="features_8ch_mixed", op="features", field="wide", rows=289591, chan=8, src=600, mixed=True, fused=True),
        # sixteen steps of the training recipe (batch 512) and the weights for the next checkpoint
        dict(name="train_512", op="train", batch=512, steps=16),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    op = rng.choice(["model", "model", "measure", "measure", "pass", "fit", "fit", "fit", "sequential", "features", "train"])
    if op == "train":
        return dict(op=op, batch=_log_int(rng, 32, 4096), steps=rng.randint(4, 16))
    field = rng.choice(["tiny", "mid", "mid", "wide"])
    chan = rng.choice([1, 1, 1, 2, 3, 4, 8])
    if field == "tiny":
        rows, src = _log_int(rng, 600, 11400), _log_int(rng, 1, 70)
    elif op == "sequential":
        rows, src = _log_int(rng, 20000, 1158361), _log_int(rng, 3, 24)
    else:
        rows, src = _log_int(rng, 20000, 9266880), _log_int(rng, 2, 1000)
    cap = {"model": 4e9, "measure": 2e9, "fit": 4e9, "pass": 5e8, "features": 5e8, "sequential": 6e7}[op]
    while rows * chan * src > cap:
        rows = max(600, int(rows * 0.73))
        src = max(1, int(src * 0.81))
    case = dict(op=op, field=field, rows=rows, chan=chan, src=src, mixed=rng.random() < 0.3)
    if op == "model":
        case["mode"] = rng.choice(["residual", "write", "accumulate"])
    elif op == "measure":
        case["mixed"] = False
        case["fused"] = rows * chan * src <= 5e8 and rng.random() < 0.5
    elif op == "fit":
        case["how"] = rng.choice(["full", "lattice", "positions"])
        case["surface"] = rng.random() < 0.3
        case["noise"] = 0.2 if case["how"] == "positions" else 1.0
        if case["how"] == "positions":
            case["src"], case["mixed"] = min(src, 100), False
        if case["how"] == "lattice":
            case["mixed"] = False
    elif op == "sequential":
        case["mixed"] = False
        case["chunk"] = rng.choice([1, 1, 4, 8, 10])
    elif op == "pass":
        case["mixed"] = False
    elif op == "features":
        case["mixed"], case["fused"] = True, rng.random() < 0.5
    return case


# ---- inputs ---------------------------------------------------------------------

_BASE = {"tiny": 0, "mid": 1, "wide": 3}


def _config(case):
    base = synth.CONFIGS[_BASE[case["field"]]]
    bl = -(-case["rows"] // base.n_time)
    n_ant = 2
    while n_ant * (n_ant - 1) // 2 < bl:
        n_ant += 1
    freq = tuple(base.freq_hz[c % base.n_chan] if base.n_chan > 1 else base.freq_hz[0] - 25.0e6 * c
                 for c in range(case["chan"]))
    n_vis0, n_vis = base.n_rows * base.n_chan, case["rows"] * case["chan"]
    sigma = base.noise_sigma_jy * math.sqrt(n_vis / n_vis0) * case.get("noise", 1.0)
    return dataclasses.replace(base, n_ant=n_ant, n_src=case["src"], freq_hz=freq, noise_sigma_jy=sigma)


def _tracks(cfg, enu, rows):
    """(u, v, w) in metres on the GPU, baseline-major, time fastest, the first `rows` of them (Earth rotation of
    the antenna pairs, hour angles centred on transit)."""
    lat, dec = math.radians(synth.SITE_LAT_DEG), math.radians(cfg.dec_deg)
    x = -math.sin(lat) * enu[:, 1] + math.cos(lat) * enu[:, 2]
    y = enu[:, 0]
    z = math.cos(lat) * enu[:, 1] + math.sin(lat) * enu[:, 2]
    i, j = np.triu_indices(cfg.n_ant, k=1)
    n = -(-rows // cfg.n_time)
    bx, by, bz = (torch.from_numpy(np.ascontiguousarray((a[j] - a[i])[:n])).to(DEV)[:, None] for a in (x, y, z))
    t = torch.arange(cfg.n_time, dtype=torch.float64, device=DEV) - 0.5 * (cfg.n_time - 1)
    ha = t * (cfg.dt_s * 2.0 * math.pi / synth.SIDEREAL_DAY_S)
    sh, ch = torch.sin(ha)[None, :], torch.cos(ha)[None, :]
    u = sh * bx + ch * by
    v = -math.sin(dec) * ch * bx + math.sin(dec) * sh * by + math.cos(dec) * bz
    w = math.cos(dec) * ch * bx - math.cos(dec) * sh * by + math.sin(dec) * bz
    return tuple(a.reshape(-1)[:rows].contiguous() for a in (u, v, w))


def _sky(uvw, freq, cat, sources, ref_hz=1.4e9, beta=-0.7):
    """Eq. 1 summed over `sources` of a catalogue, complex128 [rows * chan], in plain torch."""
    out = torch.zeros((uvw[0].shape[0], len(freq)), dtype=torch.complex128, device=DEV)
    for c, f in enumerate(freq):
        u, v, w = (a * (f / synth.C_LIGHT) for a in uvw)
        acc_r, acc_i = torch.zeros_like(u), torch.zeros_like(u)
        for s in sources:
            ph = _phase(u, v, w, cat.l[s], cat.m[s])
            amp = cat.flux_jy[s] * _profile(u, v, cat.alpha_arcsec[s], cat.e1[s], cat.e2[s])
            acc_r.addcmul_(amp, torch.cos(ph))
            acc_i.addcmul_(amp, torch.sin(ph))
        out[:, c] = torch.complex(acc_r, acc_i) * (f / ref_hz) ** beta
    return out.reshape(-1)


def _phase(u, v, w, l, m):
    """2 pi (u l + v m + w n), reduced to one turn before the factor 2 pi."""
    t = (u * float(l)).add_(v, alpha=float(m)).add_(w, alpha=math.sqrt(1.0 - l * l - m * m) - 1.0)
    return (t - torch.round(t)).mul_(2.0 * math.pi)


def _profile(u, v, alpha_arcsec, e1, e2):
    det = 1.0 - e1 * e1 - e2 * e2
    a11, a12, a22 = (1.0 + e1) / det, e2 / det, (1.0 - e1) / det
    c = 4.0 * math.pi ** 2 * (alpha_arcsec * ARCSEC) ** 2
    q = (u * float(a11) + v * float(a12)).square_() + (u * float(a12) + v * float(a22)).square_()
    return (q * float(c) + 1.0).pow_(-1.5)


def _inputs(case, seed):
    """Observation, catalogues (as handed to the library, and with the true shapes) and the noise-only residual."""
    cfg = _config(case)
    g = np.random.Generator(np.random.PCG64(seed))
    uvw = _tracks(cfg, synth.antennas(cfg, g), case["rows"])
    true = synth.catalogue(cfg, g, case["src"])
    tg = torch.Generator(device=DEV).manual_seed(int(seed) + 1)
    n_vis = case["rows"] * case["chan"]
    noise = torch.randn((n_vis, 2), generator=tg, dtype=torch.float64, device=DEV).mul_(cfg.noise_sigma_jy)
    noise = torch.view_as_complex(noise)
    weight = torch.full((n_vis,), 1.0 / cfg.noise_sigma_jy ** 2, dtype=torch.float64, device=DEV)
    weight[torch.randint(n_vis, (n_vis // 100,), generator=tg, device=DEV)] = 0.0         # flagged samples
    return cfg, uvw, true, noise, weight


def _circular(cat):
    return cat.with_shape(np.zeros(cat.n_src), np.zeros(cat.n_src))


def _isolated(case):
    """Whether the case works on a given residual (each source's own model plus noise) instead of the sky's data."""
    return case["op"] == "fit" or (case["op"] in ("measure", "features") and not case["fused"])


def _data(case, seed):
    """What the case's observation holds: (cfg, uvw, catalogue given, vis, weight) with vis in FP64.  Cases on a given
    residual hold noise and the true catalogue; the others noise plus the true sky, and the circular catalogue."""
    cfg, uvw, true, noise, weight = _inputs(case, seed)
    if case["op"] == "model":
        return cfg, uvw, true, noise, weight
    if _isolated(case):
        return cfg, uvw, true, noise, weight
    vis = noise + _sky(uvw, cfg.freq_hz, true, range(case["src"]))
    return cfg, uvw, _circular(true), vis, weight


def _fit_out(n, surface=False):
    out = {k: torch.zeros(n, dtype=torch.float64, device=DEV) for k in FIT_KEYS}
    for k in ("argmax", "n_above", "flags"):
        out[k] = torch.zeros(n, dtype=torch.int32, device=DEV)
    if surface:
        out["surface"] = torch.zeros((n, N_E * N_E), dtype=torch.float64, device=DEV)
    return out


def _train_inputs(case, seed):
    """A batch of network inputs (cells inside a facet's disk, signal and noise), targets, and the state of a network
    in the middle of its training."""
    tg = torch.Generator(device=DEV).manual_seed(int(seed))
    b = case["batch"] * 2
    r = torch.arange(64, device=DEV, dtype=torch.float32) - 32
    rad = torch.sqrt(r[:, None] ** 2 + r[None, :] ** 2).reshape(1, 4096)
    size = torch.rand((b, 1), generator=tg, device=DEV) * 10 + 5
    re = torch.exp(-rad / size) + 0.3 * torch.randn((b, 4096), generator=tg, device=DEV)
    im = 0.3 * torch.randn((b, 4096), generator=tg, device=DEV)
    x = (torch.cat([re * (rad < 2 * size), im * (rad < 2 * size)], dim=1)).clamp_(-4, 4).to(torch.bfloat16)
    target = torch.randn((b, 3), generator=tg, device=DEV) * 0.3
    shapes = [(8192, 512), (512, 512), (512, 512), (512, 6)]
    parts = []
    for k, (i, o) in enumerate(shapes):
        parts += [torch.randn(i * o, generator=tg, device=DEV) * (math.sqrt(2.0 / i) * (1e-2 if k == 3 else 1.0)),
                  torch.randn(o, generator=tg, device=DEV) * 0.01]
    params = torch.cat(parts)
    m = torch.randn(params.shape, generator=tg, device=DEV) * 1e-4
    v = torch.rand(params.shape, generator=tg, device=DEV) * 1e-6 + 1e-6
    return x, target, params, m, v


# ---- prepare and run -----------------------------------------------------------

_MODE = {"write": rlf.RLF_MODEL_WRITE, "accumulate": rlf.RLF_MODEL_ACCUMULATE, "residual": rlf.RLF_MODEL_RESIDUAL}
POS_SIDE, POS_STEP = 5, 0.1
STRIDE = 4
LR = 3e-4
STEP0 = 5000


def prepare(case, seed):
    st = {"case": case}
    if case["op"] == "train":
        x, target, params, m, v = _train_inputs(case, seed)
        st["ctx"] = rlf.Context(0, torch.cuda.current_stream().cuda_stream)
        st["net"] = rlf.Mlp(st["ctx"], case["batch"])
        st["net"].set_state(params.cpu().numpy(), m.cpu().numpy(), v.cpu().numpy(), STEP0)
        st["x"], st["target"] = x.split(case["batch"]), target.split(case["batch"])
        st["loss"] = torch.zeros(case["steps"], dtype=torch.float64, device=DEV)
        st["params"] = torch.zeros(params.shape, dtype=torch.float32, pin_memory=True)
        return st
    cfg, uvw, cat, vis, weight = _data(case, seed)
    mixed = case["mixed"]
    if mixed:
        vis, weight = vis.to(torch.complex64), weight.to(torch.float32)
    st["cat"] = cat
    st["obs"] = obs = rlf.Obs(*uvw, np.asarray(cfg.freq_hz), vis, weight)
    st["ctx"] = ctx = rlf.Context(0, torch.cuda.current_stream().cuda_stream,
                                  rlf.params(precision=rlf.RLF_MIXED if mixed else rlf.RLF_FP64))
    op = case["op"]
    if op == "model":
        st["out"] = torch.zeros_like(vis)
        return st
    if op != "sequential":
        st["facets"] = ctx.facets_create(obs, cat)
    if op == "features":
        st["net"] = rlf.Mlp(ctx, 64)
        st["x"] = torch.zeros((case["src"], surrogate.N_IN), dtype=torch.bfloat16, device=DEV)
        return st
    st["out"] = _fit_out(case["src"], case.get("surface", False))
    if op == "fit":
        ctx.extract_facets(obs, cat, vis, st["facets"])
        if case["how"] == "positions":
            ctx.set_positions(st["facets"], POS_SIDE, POS_STEP)
    if op == "pass":
        st["pass"] = ctx.pass_create(obs, cat, st["facets"], st["out"])
    return st


def run(st):
    case = st["case"]
    op = case["op"]
    ctx = st["ctx"]
    if op == "model":
        ctx.model_vis(st["obs"], st["cat"], st["out"], _MODE[case["mode"]])
        return st["out"]
    if op == "measure":
        ctx.extract_facets(st["obs"], st["cat"], None if case["fused"] else st["obs"].vis, st["facets"])
        ctx.fit_sources(st["facets"], st["out"])
        return st["out"]
    if op == "pass":
        st["pass"].launch()
        return st["out"]
    if op == "fit":
        if case["how"] == "lattice":
            ctx.fit_sources(st["facets"], st["out"], mode=2, check_stride=STRIDE, want_surface=case["surface"])
        else:
            ctx.fit_sources(st["facets"], st["out"], want_surface=case["surface"])
        if case["how"] == "positions":
            ctx.refine_sources(st["facets"], st["out"])
        return st["out"]
    if op == "sequential":
        e1, e2 = ctx.fit_sequential(st["obs"], st["cat"], case["chunk"], st["out"])
        return {"fit": st["out"], "e1": e1, "e2": e2}
    if op == "features":
        ctx.extract_facets(st["obs"], st["cat"], None if case["fused"] else st["obs"].vis, st["facets"])
        st["net"].features(st["facets"], st["x"])
        return st["x"]
    for k in range(case["steps"]):
        st["net"].train_step(st["x"][k % 2], st["target"][k % 2], LR, st["loss"][k:k + 1])
    # the FP32 weights alone, into page-locked host memory (rlf_mlp_get_state skips what is NULL)
    ctx._check(rlf.lib().rlf_mlp_get_state(st["net"].h, st["params"].data_ptr(), None, None, None, None))
    return {"loss": st["loss"], "params": st["params"]}


# ---- what a pass cannot do without ----------------------------------------------

# floating-point operations per unit (an FMA counts two, an elementary function one): a (visibility, source) pair
# of the sky model and of the extraction, a (cell, grid point, knot) of the likelihood
PAIR_MODEL, PAIR_EXTRACT, UNIT_FIT = 20.0, 31.0, 7.5


def work(case):
    op = case["op"]
    if op == "train":
        p1, p = 8192 * 512, 8192 * 512 + 2 * 512 * 512 + 512 * 6
        b, n = case["batch"], case["steps"]
        return {"bytes": n * (b * 8192 * 2 + p * 4 * 6) + p * 4, "flops": n * b * (4.0 * p + 2.0 * (p - p1))}
    n_vis, n = case["rows"] * case["chan"], case["src"]
    pairs = float(n_vis) * n
    cpx, wt = (8, 4) if case["mixed"] else (16, 8)
    obs = case["rows"] * 24 + n_vis * (cpx + wt)
    units = float(n) * MEAN_CELLS[case["field"]] * N_GRID * N_KNOTS
    fit_out = n * 60.0
    if op == "model":
        reads = case["rows"] * 24 + (0 if case["mode"] == "write" else n_vis * cpx)
        return {"bytes": reads + n_vis * cpx, "flops": pairs * PAIR_MODEL}
    if op in ("measure", "pass"):
        fused = op == "pass" or case["fused"]
        return {"bytes": obs + fit_out, "flops": pairs * (PAIR_EXTRACT + (PAIR_MODEL if fused else 0)) + units * UNIT_FIT}
    if op == "fit":
        per = {"full": UNIT_FIT, "lattice": UNIT_FIT / 4, "positions": UNIT_FIT - 2 + 2 * POS_SIDE ** 2}[case["how"]]
        out = fit_out + (n * N_E * N_E * 8.0 if case["surface"] else 0)
        return {"bytes": n * MEAN_CELLS[case["field"]] * 32.0 + out, "flops": units * per}
    if op == "sequential":
        steps = -(-n // case["chunk"])
        return {"bytes": obs * float(steps), "flops": pairs * (PAIR_EXTRACT + 3 * PAIR_MODEL) + units * UNIT_FIT}
    return {"bytes": obs + n * 8192 * 2.0, "flops": pairs * (PAIR_EXTRACT + (PAIR_MODEL if case["fused"] else 0))}


# ---- the same in 64 bits ----------------------------------------------------------

def _grid():
    c = (N_E - 1) // 2
    i = torch.arange(N_E, device=DEV) - c
    i1, i2 = i[:, None].expand(N_E, N_E).reshape(-1), i[None, :].expand(N_E, N_E).reshape(-1)
    ok = i1 * i1 + i2 * i2 < round(1.0 / E_STEP) ** 2
    return i1[ok].double() * E_STEP, i2[ok].double() * E_STEP, ok


def _knots():
    a = 0.3 + (3.5 - 0.3) * (np.arange(N_KNOTS) / (N_KNOTS - 1)) ** 2
    h = np.diff(a)
    n = N_KNOTS
    t = np.zeros((n - 2, n - 2))                        # second derivatives of the natural cubic spline
    r = np.zeros((n - 2, n))
    for i in range(1, n - 1):
        t[i - 1, i - 1] = 2 * (h[i - 1] + h[i])
        if i > 1:
            t[i - 1, i - 2] = h[i - 1]
        if i < n - 2:
            t[i - 1, i] = h[i]
        r[i - 1, i - 1], r[i - 1, i], r[i - 1, i + 1] = 6 / h[i - 1], -6 / h[i - 1] - 6 / h[i], 6 / h[i]
    m = np.vstack([np.zeros(n), np.linalg.solve(t, r), np.zeros(n)])
    w = np.zeros(n)
    for i in range(n - 1):
        w[i] += h[i] / 2
        w[i + 1] += h[i] / 2
        w -= h[i] ** 3 * (m[i] + m[i + 1]) / 24
    return a, w


def _log_weights(flux):
    a, w = _knots()
    z = np.log(a) - (-0.93 + 0.33 * math.log(flux * 1e6))
    return np.log(w) - z ** 2 / (2 * 0.3136 ** 2) - np.log(a * 0.3136 * math.sqrt(2 * math.pi))


def _facet(lam, spec, resid, weight, cat, s, e1, e2):
    """Cells (ix, iy), weight sums and means of source s from the residual (flattened over rows and channels)."""
    u, v, w = lam
    ph = _phase(u, v, w, cat.l[s], cat.m[s])
    own = _profile(u, v, cat.alpha_arcsec[s], e1, e2).mul_(float(cat.flux_jy[s])).mul_(spec)
    cs, sn = torch.cos(ph), torch.sin(ph)
    zr = (resid.real * cs + resid.imag * sn + own) * weight
    zi = (resid.imag * cs - resid.real * sn) * weight
    theta = 38.0 * (cat.alpha_arcsec[s] * ARCSEC)
    ix, iy = torch.round(u * theta).long(), torch.round(v * theta).long()
    half = int(max(ix.abs().max(), iy.abs().max()))
    side = 2 * half + 1
    key = (iy + half) * side + ix + half
    n = side * side
    cnt = torch.bincount(key, weights=(weight > 0).double(), minlength=n)
    W, Zr, Zi = (torch.bincount(key, weights=t, minlength=n) for t in (weight, zr, zi))
    k = torch.nonzero(cnt > 0).reshape(-1)
    return (k % side - half).double(), (k // side - half).double(), W[k], Zr[k] / W[k], Zi[k] / W[k], theta


def _lnl(facet, flux, e1, e2, positions=False):
    ix, iy, W, vr, vi, theta = facet
    u, v = ix / theta, iy / theta
    det = (1.0 - e1 * e1 - e2 * e2)[:, None]
    q = (((1 + e1)[:, None] * u + e2[:, None] * v) / det).square() + ((e2[:, None] * u + (1 - e1)[:, None] * v) / det).square()
    if positions:
        p = (torch.arange(POS_SIDE, device=DEV) - (POS_SIDE - 1) // 2).double() * (POS_STEP * ARCSEC)
        ph = 2 * math.pi * (u[:, None, None] * p[None, :, None] + v[:, None, None] * p[None, None, :]).reshape(len(u), -1)
        G = W[:, None] * (vr[:, None] * torch.cos(ph) + vi[:, None] * torch.sin(ph))
    else:
        G = (W * vr)[:, None]
    a, _ = _knots()
    lw = _log_weights(flux)
    terms = []
    for k in range(N_KNOTS):
        t = (q * float(4 * math.pi ** 2 * (a[k] * ARCSEC) ** 2) + 1.0).rsqrt_()
        f = t * t * t
        D, M = f @ G, (f * f) @ W
        terms.append(D * D / (2 * M[:, None]) - 0.5 * torch.log(M)[:, None] + float(lw[k]))
    return torch.logsumexp(torch.cat(terms, dim=1), dim=1) - math.log(G.shape[1])


def _moments(L, x1, x2):
    best = L.max()
    on = L >= best + math.log(FRAC)
    w, a, b = torch.exp(L[on] - best), x1[on], x2[on]
    m1, m2 = (w * a).sum() / w.sum(), (w * b).sum() / w.sum()
    c11, c22 = (w * (a - m1) ** 2).sum() / w.sum(), (w * (b - m2) ** 2).sum() / w.sum()
    c12 = (w * (a - m1) * (b - m2)).sum() / w.sum()
    return dict(e1=m1, e2=m2, s1=c11.sqrt(), s2=c22.sqrt(), c12=c12, lmax=best), on


def _refined(facet, flux, L, est, on, ok):
    """The adaptive refinement of one source (nested grids down to 0.0025, at least 30 samples above the threshold)."""
    c = (N_E - 1) // 2
    flat = torch.nonzero(ok).reshape(-1)
    k1, k2 = flat // N_E - c, flat % N_E - c
    step, unit = E_STEP, round(1.0 / E_STEP)
    while step > 0.003 and int(on.sum()) < 30:
        step, unit = step / 2, unit * 2
        at, axes = int(L.argmax()), []
        for k in (k1, k2):
            lo, hi = 2 * int(k[on].min()) - 2, 2 * int(k[on].max()) + 2
            if hi - lo + 1 > 64:
                lo = 2 * int(k[at]) - 63 // 2
                hi = lo + 63
            axes.append(torch.arange(lo, hi + 1, device=DEV))
        k1, k2 = (t.reshape(-1) for t in torch.meshgrid(*axes, indexing="ij"))
        inside = k1 * k1 + k2 * k2 < unit * unit
        k1, k2 = k1[inside], k2[inside]
        L = _lnl(facet, flux, k1.double() * step, k2.double() * step, True)
        est, on = _moments(L, k1.double() * step, k2.double() * step)
    return est


def _lambda(uvw, freq):
    f = torch.tensor(list(freq), dtype=torch.float64, device=DEV)
    lam = tuple((a[:, None] * (f / synth.C_LIGHT)[None, :]).reshape(-1) for a in uvw)
    spec = ((f / 1.4e9) ** -0.7)[None, :].expand(uvw[0].shape[0], -1).reshape(-1)
    return lam, spec


def _stack(ests, extra=None):
    out = {k: torch.stack([e[k] for e in ests]) for k in FIT_KEYS}
    return {**out, "argmax": None, "n_above": None, "flags": None, **(extra or {})}


def _exact_train(case, seed):
    x, target, params, m, v = _train_inputs(case, seed)
    x, target, p, m, v = (t.double() for t in (x, target, params, m, v))
    sizes = [8192 * 512, 512, 512 * 512, 512, 512 * 512, 512, 512 * 6, 6]
    shapes = [(8192, 512), (512,), (512, 512), (512,), (512, 512), (512,), (512, 6), (6,)]
    losses = []
    for k in range(case["steps"]):
        p = p.detach().requires_grad_(True)
        q = [t.reshape(s) for t, s in zip(p.split(sizes), shapes)]
        rows = slice((k % 2) * case["batch"], (k % 2 + 1) * case["batch"])
        h = x[rows]
        for i in range(3):
            h = torch.nn.functional.gelu(h @ q[2 * i] + q[2 * i + 1])
        y = h @ q[6] + q[7]
        s = y[:, 3:].clamp(min=math.log(1e-3))
        loss = (0.5 * (s + (target[rows] - y[:, :3]) ** 2 * torch.exp(-s))).sum() / case["batch"]
        (g,) = torch.autograd.grad(loss, p)
        t = STEP0 + k + 1
        m, v = 0.9 * m + 0.1 * g, 0.999 * v + 0.001 * g * g
        p = p.detach() - LR * (m / (1 - 0.9 ** t)) / ((v / (1 - 0.999 ** t)).sqrt() + 1e-8)
        losses.append(loss.detach())
    return {"loss": torch.stack(losses), "params": p}


def exact(case, seed):
    op = case["op"]
    if op == "train":
        return _exact_train(case, seed)
    cfg, uvw, cat, vis, weight = _data(case, seed)
    if case["mixed"]:
        vis, weight = vis.to(torch.complex64).to(torch.complex128), weight.float().double()
    n = case["src"]
    if op == "model":
        if case["mode"] == "accumulate":
            return None                                 # the sum over as many passes as were made
        sky = _sky(uvw, cfg.freq_hz, cat, range(n))
        return vis - sky if case["mode"] == "residual" else sky
    lam, spec = _lambda(uvw, cfg.freq_hz)
    x1, x2, ok = _grid()

    def fit(s, e1, e2, resid):
        facet = _facet(lam, spec, resid, weight, cat, s, e1, e2)
        positions = case.get("how") == "positions"
        L = _lnl(facet, cat.flux_jy[s], x1, x2, positions)
        est, on = _moments(L, x1, x2)
        return _refined(facet, cat.flux_jy[s], L, est, on, ok) if positions else est, L

    if op == "sequential":
        e1, e2 = cat.e1.copy(), cat.e2.copy()
        resid = vis - _sky(uvw, cfg.freq_hz, cat, range(n))
        ests, bad = [None] * n, []

        def is_bad(e):
            det = e["s1"] ** 2 * e["s2"] ** 2 - e["c12"] ** 2
            return bool(e["s1"] <= 5e-3) or bool(e["s2"] <= 5e-3) or float(det.clamp(min=0).sqrt()) <= 5e-5

        for c0 in range(0, n, case["chunk"]):
            chunk = range(c0, min(n, c0 + case["chunk"]))
            for s in chunk:
                ests[s], _ = fit(s, e1[s], e2[s], resid)
            good = [s for s in chunk if not is_bad(ests[s])]
            bad += [s for s in chunk if s not in good]
            resid = resid + _sky(uvw, cfg.freq_hz, cat.with_shape(e1, e2), good)
            for s in good:
                e1[s], e2[s] = float(ests[s]["e1"]), float(ests[s]["e2"])
            resid = resid - _sky(uvw, cfg.freq_hz, cat.with_shape(e1, e2), good)
        again = {s: fit(s, e1[s], e2[s], resid)[0] for s in bad}
        for s, est in again.items():
            ests[s] = est
            e1[s], e2[s] = float(est["e1"]), float(est["e2"])
        return {"fit": _stack(ests), "e1": e1, "e2": e2}

    if not _isolated(case):
        vis = vis - _sky(uvw, cfg.freq_hz, cat, range(n))
    if op == "features":
        g = float(np.mean([(f / 1.4e9) ** -0.7 for f in cfg.freq_hz]))
        x = torch.zeros((n, surrogate.N_IN), dtype=torch.float64, device=DEV)
        for s in range(n):
            ix, iy, _, vr, vi, _ = _facet(lam, spec, vis, weight, cat, s, cat.e1[s], cat.e2[s])
            on = (ix >= -32) & (ix <= 31) & (iy >= -32) & (iy <= 31)
            at = ((iy + 32) * 64 + ix + 32)[on].long()
            x[s, at] = (vr[on] / (cat.flux_jy[s] * g)).clamp(-4, 4)
            x[s, 4096 + at] = (vi[on] / (cat.flux_jy[s] * g)).clamp(-4, 4)
        return x
    ests, surf = [], None
    if case.get("surface"):
        surf = torch.full((n, N_E * N_E), -math.inf, dtype=torch.float64, device=DEV)
    for s in range(n):
        est, L = fit(s, cat.e1[s], cat.e2[s], vis)
        ests.append(est)
        if surf is not None:
            surf[s, ok] = L
    if case.get("how") == "lattice":
        surf = None                                     # holds only the points that the narrowed fit evaluates
    return _stack(ests, {"surface": surf} if case.get("surface") else None)
