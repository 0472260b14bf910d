"""The measured workloads of the beamforming library: what a user's program calls, over the
range of sizes, options and storage types it calls them with.

Every case goes through the package's public entry points with the objects a program keeps
between frames already made (marshalled geometry, output planes, workspace, batch handle).
The acquisitions are those of this repository's workload configurations: a linear array of
0.3 mm pitch, a 5 MHz pulse sampled at 20 MHz (or 7.5 MHz at 50 MHz), plane waves steered
within +-10 degrees. Kinds of case:

  frame    one beamformed image (das, dmas, pdas), one angle or the compound, with the depth
           post-processing the caller asks for
  iq       the baseband path: demodulation of the records, then IQ-DAS or BB-DMAS
  fk       Stolt's or Lu's f-k migration
  batch    uneven frames in one batch launch
  metrics  contrast and resolution figures of an envelope image
"""

import math
import random

import numpy as np
import torch

import paper_2311_00482_amd as pwbf

PITCH = 0.3e-3
C_SOUND = 1540.0
FLOOR_DB = -70.0
DEV = "cuda:0"


# ------------------------------------------------------------------ the cases
def _frame(name, mode, **kw):
    case = {"name": name, "kind": "frame", "mode": mode, "channels": 128, "samples": 4096,
            "angles": 1, "span_deg": 10.0, "angle": -1, "nx": 512, "nz": 512, "width": 19.0e-3,
            "z_min": 5e-3, "z_max": 45e-3, "fs": 20e6, "f0": 5e6, "dtype": "float32",
            "apod": "hann", "planes": "rf,env,log", "bandpass": False, "p": 2.0,
            "decimation": 1}
    case.update(kw)
    return case


def listed():
    return [
        # the smallest imaging grid of the timing study: a preview image, all launch latency
        _frame("preview_128x32", "das", channels=64, fs=50e6, f0=7.5e6, nx=128, nz=32,
               width=19.2e-3, z_min=1e-3, z_max=30e-3, dtype="int16"),
        # one plane wave per frame, as a live display shows it: 64 channels, 10-bit samples
        _frame("live_das_128x256", "das", channels=64, samples=2048, nx=128, nz=256, z_min=0.0,
               z_max=40e-3, dtype="int16"),
        # a single-shot DMAS image with its band-pass, every plane kept
        _frame("dmas_512x512", "dmas", z_min=13.6e-3, z_max=26.4e-3, dtype="int16",
               planes="rf,filtered,env,log", bandpass=True),
        # five-angle pDAS compound from records stored in half precision
        _frame("pdas_5a_512x512", "pdas", angles=5, width=38.4e-3, dtype="float16"),
        # research data: many angles, ragged sizes, no post-processing, boxcar aperture
        _frame("das_21a_301x777", "das", channels=96, samples=3000, angles=21, nx=301, nz=777,
               width=28.8e-3, z_max=50e-3, apod="boxcar", planes="rf"),
        # the headline workload: 11-angle coherent compound at full size
        _frame("das_11a_1024x1024", "das", angles=11, nx=1024, nz=1024, width=38.1e-3),
        # the baseband pipeline at the same size: demodulation and IQ-DAS
        _frame("iqdas_11a_1024x1024", "iqdas", kind="iq", angles=11, nx=1024, nz=1024,
               width=38.1e-3, planes="rf,imag,env,log"),
        # BB-DMAS from 10-bit records decimated by two, seven angles
        _frame("bbdmas_7a_d2_384x500", "bbdmas", kind="iq", channels=64, samples=2048, angles=7,
               nx=384, nz=500, width=19.2e-3, z_max=40e-3, dtype="int16", decimation=2,
               planes="rf,imag,env,log"),
        # f-k migration of the full compound
        _frame("stolt_11a_1024x1024", "stolt", kind="fk", angles=11, nx=1024, nz=1024,
               width=38.1e-3, planes="rf,imag,env,log"),
        # f-k migration of one steered wave of a 64-channel probe
        _frame("lu_1a_500x512", "lu", kind="fk", channels=64, samples=2048, angles=1,
               span_deg=8.0, nx=500, nz=512, width=19.2e-3, z_max=40e-3, dtype="int16",
               planes="rf,imag,env"),
        # frames of several probes and modes waiting together, in one batch launch
        {"name": "batch_16_uneven", "kind": "batch", "frames": 16, "frames_seed": 2000,
         "dtype": "int16"},
        # the evaluation figures of one compound image: three cysts, twenty point targets
        {"name": "metrics_1024x1024", "kind": "metrics", "nx": 1024, "nz": 1024, "cysts": 3,
         "targets": 20, "radius_min": 2e-3, "radius_max": 4e-3},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _draw_image(rng):
    mode = rng.choice(["das", "das", "das", "dmas", "pdas"])
    post = rng.random() < 0.7
    angles = rng.choice([1, 1, 1, rng.randint(2, 16), rng.randint(2, 16), rng.randint(17, 32)])
    case = _frame("", mode, angles=angles, channels=_log_int(rng, 16, 192),
                  samples=rng.choice([2048, 4096, rng.randint(1500, 6000)]),
                  nx=_log_int(rng, 24, 1024),
                  nz=2 ** rng.randint(5, 11) if post else _log_int(rng, 24, 1500),
                  dtype=rng.choice(["int16", "int16", "float16", "float32"]),
                  apod=rng.choice(["hann", "hann", "hann", "boxcar", "none"]),
                  planes=rng.choice(["rf,env,log", "rf,env", "rf,log"]) if post else "rf",
                  bandpass=post and mode == "dmas" and rng.random() < 0.7,
                  p=rng.choice([2.0, 2.0, 1.5]))
    if case["bandpass"]:
        case["planes"] = "rf,filtered,env,log"
    if angles > 1 and rng.random() < 0.2:
        case["angle"] = rng.randrange(angles)
    return case, {"das": 1.0, "dmas": 2.2, "pdas": 2.2}[mode]


def _draw_iq(rng):
    mode = rng.choice(["iqdas", "bbdmas"])
    case = _frame("", mode, kind="iq", angles=rng.choice([1, 1, rng.randint(2, 12), 5, 11]),
                  channels=_log_int(rng, 16, 160), samples=rng.choice([1024, 2048, 4096]),
                  nx=_log_int(rng, 24, 1024), nz=_log_int(rng, 24, 1024),
                  dtype=rng.choice(["int16", "int16", "float16", "float32"]),
                  apod=rng.choice(["hann", "hann", "boxcar"]),
                  decimation=rng.choice([1, 1, 2, 4]),
                  planes=rng.choice(["rf,imag,env,log", "rf,imag,env"]))
    return case, {"iqdas": 2.6, "bbdmas": 3.6}[mode]


def _draw_fk(rng):
    mode = rng.choice(["stolt", "lu"])
    case = _frame("", mode, kind="fk", angles=rng.choice([1, 1, rng.randint(2, 11)]),
                  channels=_log_int(rng, 16, 128), samples=rng.choice([1024, 2048, 4096]),
                  nx=_log_int(rng, 24, 1024), nz=_log_int(rng, 24, 1024),
                  dtype=rng.choice(["int16", "float16", "float32"]),
                  planes=rng.choice(["rf,imag,env,log", "rf,imag,env"]))
    return case, 1.0


def draw(rng):
    kind = rng.choice(["frame"] * 6 + ["iq", "iq", "fk", "fk", "batch", "metrics"])
    if kind == "batch":
        return {"kind": "batch", "frames": rng.randint(2, 12),
                "frames_seed": rng.randrange(1 << 30),
                "dtype": rng.choice(["int16", "float16", "float32"])}
    if kind == "metrics":
        return {"kind": "metrics", "nx": _log_int(rng, 128, 1024), "nz": _log_int(rng, 128, 1024),
                "cysts": rng.randint(1, 8), "targets": rng.randint(1, 32),
                "radius_min": 1.5e-3, "radius_max": 3.5e-3}
    case, cost = {"frame": _draw_image, "iq": _draw_iq, "fk": _draw_fk}[kind](rng)
    del case["name"]
    # pixels of 0.3 .. 1.6 samples along depth (at most c / (12 f0) for the band-pass), the
    # image over half to all of the array and inside the record's depth
    case["z_min"] = rng.uniform(0.0, 12e-3) if kind == "frame" else rng.uniform(3e-3, 12e-3)
    depth = 0.42 * case["samples"] * C_SOUND / case["fs"] - case["z_min"]
    dz = 25e-6 if case["bandpass"] else math.exp(rng.uniform(math.log(25e-6), math.log(120e-6)))
    dz = min(dz, depth / case["nz"])
    case["z_max"] = case["z_min"] + dz * case["nz"]
    array = case["channels"] * PITCH
    case["width"] = array * rng.uniform(0.5, 1.0)
    case["nx"] = max(case["nx"], int(math.ceil(case["width"] / 0.5e-3)))
    # no dearer than the full-size compound (pairs outside the aperture cost nothing there)
    if case["apod"] == "none":
        cost *= 2.5
    used = 1 if case["angle"] >= 0 else case["angles"]
    most = 1024 * 1024 * 128 * 11 / (cost * used * case["channels"] * case["nz"])
    if case["nx"] > most:
        case["nx"] = max(24, int(most))
        case["width"] = min(case["width"], case["nx"] * 0.5e-3)
    return case


# ------------------------------------------------------------------ geometry
class Geometry:
    """The attributes the binding reads, from a case's plain values."""

    def __init__(self, case):
        n, a = case["channels"], case["angles"]
        self.n_samples = case["samples"]
        self.elem_x = (np.arange(n, dtype=np.float64) - (n - 1) / 2.0) * PITCH
        span = math.radians(case["span_deg"])
        single = 0.0 if case["kind"] != "fk" else span
        self.angles_rad = np.linspace(-span, span, a) if a > 1 else np.array([single])
        self.c, self.fs, self.f0 = C_SOUND, case["fs"], case["f0"]
        self.nx, self.nz = case["nx"], case["nz"]
        self.dx = case["width"] / self.nx
        self.x0 = -0.5 * case["width"] + 0.5 * self.dx
        self.dz = (case["z_max"] - case["z_min"]) / self.nz
        self.z0 = case["z_min"] + 0.5 * self.dz
        self.f_number = 1.5
        self.apod = case["apod"]

    def first(self, a):
        return float(np.min(self.elem_x * math.sin(self.angles_rad[a])))


def _batch_frames(case):
    """The frames of a batch case: channels, angles, grid, samples and mode drawn per frame."""
    rng = random.Random(case["frames_seed"])
    out = []
    for i in range(case["frames"]):
        n, a = rng.choice([64, 128]), rng.choice([1, 1, 5, 11])
        nx, nz = rng.choice([256, 400, 512, 1024]), rng.choice([256, 512, 1024])
        mode = rng.choice(["das", "das", "dmas", "pdas"])
        if nx * nz * n * a > 512 * 1024 * 128 * 5:  # the largest frames go out on their own
            nx = 256
        z = (10e-3, 10e-3 + nz * 25e-6) if mode == "dmas" else (5e-3, 45e-3)
        out.append(_frame("", mode, channels=n, samples=rng.choice([2048, 4096]), angles=a, nx=nx,
                          nz=nz, width=n * PITCH, z_min=z[0], z_max=z[1], dtype=case["dtype"],
                          bandpass=mode == "dmas"))
    return out


# ------------------------------------------------------------------ inputs
def _records(case, g, seed, device=DEV):
    """Channel records of point targets and speckle with 30 dB of white noise, scaled to the
    10-bit range: the plane wave reaches a scatterer, its echo each element; the pulse is a
    Gaussian-windowed cosine at f0 with a two-cycle envelope."""
    host = np.random.default_rng(seed)
    A, N, Ns = case["angles"], case["channels"], case["samples"]
    w, h = case["width"], case["z_max"] - case["z_min"]
    points, speckle = 12, 160
    xs = np.concatenate([host.uniform(-0.45, 0.45, points) * w, host.uniform(-0.5, 0.5, speckle) * w])
    zs = case["z_min"] + h * np.concatenate([np.linspace(0.08, 0.95, points),
                                             host.uniform(0.0, 1.0, speckle)])
    amp = np.concatenate([np.full(points, 10.0), host.standard_normal(speckle)])
    f64 = dict(dtype=torch.float64, device=device)
    ex = torch.tensor(g.elem_x, **f64)
    th = torch.tensor(g.angles_rad, **f64)
    first = torch.tensor([g.first(a) for a in range(A)], **f64)
    sigma = 2.0 / case["f0"] / (2.0 * math.sqrt(2.0 * math.log(2.0)))
    half = int(math.ceil(3.5 * sigma * case["fs"]))
    taps = torch.arange(-half, half + 1, device=device)
    margin = half + 2
    rf = torch.zeros(A * N, Ns + 2 * margin, dtype=torch.float32, device=device)
    xs, zs, amp = (torch.tensor(v, **f64) for v in (xs, zs, amp))
    t = ((xs[:, None] * torch.sin(th) + zs[:, None] * torch.cos(th) - first)[:, :, None]
         + torch.sqrt((xs[:, None] - ex) ** 2 + zs[:, None] ** 2)[:, None, :]) / g.c
    t = t.reshape(len(xs), A * N) * case["fs"]  # [scatterer, record] in samples
    n0 = torch.round(t).clamp(-1, Ns)
    for k in range(len(xs)):  # one scatterer at a time: every position is written once
        d = ((n0[k] - t[k])[:, None] + taps) / case["fs"]
        v = amp[k] * torch.exp(-0.5 * (d / sigma) ** 2) * torch.cos(2.0 * math.pi * case["f0"] * d)
        at = n0[k].long()[:, None] + taps + margin
        rf.scatter_(1, at, rf.gather(1, at) + v.float())
    rf = rf[:, margin:margin + Ns]
    noise = torch.randn(rf.shape, dtype=torch.float32, device=device,
                        generator=torch.Generator(device=device).manual_seed(seed))
    rms = float(rf.double().square().mean().sqrt())
    rf = rf + noise * (rms * 10.0 ** (-30.0 / 20.0))
    rf = rf * (511.0 / float(rf.abs().max()))
    if case["dtype"] == "int16":
        rf = rf.round().clamp(-512, 511)
    return rf.reshape(A, N, Ns).to(getattr(torch, case["dtype"])).contiguous()


def _envelope(case, seed):
    """A speckle envelope with dark cysts and bright points, and the regions to read."""
    host = np.random.default_rng(seed)
    nx, nz = case["nx"], case["nz"]
    size_x, size_z = 38.1e-3, 40e-3
    dx, dz = size_x / nx, size_z / nz
    x = (torch.arange(nx, device=DEV) + 0.5) * dx - 0.5 * size_x
    z = 5e-3 + (torch.arange(nz, device=DEV) + 0.5) * dz
    gen = torch.Generator(device=DEV).manual_seed(seed)
    re, im = (torch.randn(nx, nz, device=DEV, generator=gen) for _ in range(2))
    env = 20.0 * torch.sqrt(re * re + im * im)
    cysts, targets = [], []
    for _ in range(case["cysts"]):
        r = host.uniform(case["radius_min"], case["radius_max"])
        cx, cz = host.uniform(-9e-3, 9e-3), host.uniform(14e-3, 36e-3)
        env = torch.where((x[:, None] - cx) ** 2 + (z - cz) ** 2 < r * r, 0.1 * env, env)
        side = -1.0 if cx > 0 else 1.0
        cysts.append(((cx, cz, 0.8 * r), (cx + side * 2.2 * r, cz, 0.8 * r)))
    for _ in range(case["targets"]):
        cx, cz = host.uniform(-17e-3, 17e-3), host.uniform(8e-3, 42e-3)
        peak = 4000.0 * torch.exp(-((x[:, None] - cx) / 0.35e-3) ** 2 - ((z - cz) / 0.15e-3) ** 2)
        env = env + peak
        targets.append((cx, cz, 1e-3))
    return env.contiguous(), cysts, targets, {"size_x": size_x, "size_z": size_z}


def _metrics_geometry(case, size):
    return Geometry(_frame("", "das", nx=case["nx"], nz=case["nz"], width=size["size_x"],
                           z_min=5e-3, z_max=5e-3 + size["size_z"]))


# ------------------------------------------------------------------ prepare and run
def _planes(case):
    return {k: torch.empty(case["nx"], case["nz"], dtype=torch.float32, device=DEV)
            for k in case["planes"].split(",")}


def _marshal(case, g):
    return pwbf.GeometryArg(g, bandpass=case["bandpass"], log_floor_db=FLOOR_DB,
                            pdas_p=case["p"], iq_decimation=case["decimation"])


def prepare(case, seed):
    if case["kind"] == "metrics":
        env, cysts, targets, size = _envelope(case, seed)
        g = pwbf.GeometryArg(_metrics_geometry(case, size))
        return {"case": case, "geom": g, "env": env, "cysts": cysts, "targets": targets}
    if case["kind"] == "batch":
        specs, outs = [], []
        for i, f in enumerate(_batch_frames(case)):
            g = Geometry(f)
            rf = _records(f, g, seed * 1000 + i)
            outs.append(_planes(f))
            specs.append(pwbf.FrameSpec(_marshal(f, g), rf, f["mode"], -1, outs[-1],
                                        f["bandpass"], None, f["p"]))
        return {"case": case, "batch": pwbf.Batch(specs), "outs": outs, "specs": specs}
    g = Geometry(case)
    arg = _marshal(case, g)
    rf = _records(case, g, seed)
    out = _planes(case)
    state = {"case": case, "geom": arg, "rf": rf, "out": out}
    if case["kind"] == "fk":
        need = pwbf.fk_workspace_bytes(arg, case["planes"].split(","), case["angle"],
                                       method=case["mode"])
    else:
        need = pwbf.workspace_bytes(arg, case["planes"].split(","), case["bandpass"])
    state["workspace"] = torch.empty(max(need, 256), dtype=torch.uint8, device=DEV)
    if case["kind"] == "iq":
        state["iq"] = torch.empty(arg.shape_iq, dtype=torch.complex64, device=DEV)
    return state


def run(state):
    case = state["case"]
    if case["kind"] == "metrics":
        c = pwbf.contrast_metrics(state["geom"], state["env"], state["cysts"])
        r = pwbf.resolution_metrics(state["geom"], state["env"], state["targets"])
        return {"contrast": _columns(c, ("n_in", "n_out")), "resolution": _columns(r, ("ix", "iz"))}
    if case["kind"] == "batch":
        state["batch"].launch()
        return state["outs"]
    want, out = state["out"].keys(), state["out"]
    if case["kind"] == "fk":
        pwbf.fk_migrate(state["geom"], state["rf"], case["angle"], want=want, out=out,
                        workspace=state["workspace"], log_floor_db=FLOOR_DB,
                        method=case["mode"])
        return out
    rf = state["rf"]
    if case["kind"] == "iq":
        rf = pwbf.iq_demodulate(state["geom"], rf, out=state["iq"])
    kw = dict(want=want, out=out, workspace=state["workspace"], bandpass=case["bandpass"],
              log_floor_db=FLOOR_DB)
    if case["angle"] >= 0 or case["angles"] == 1:
        pwbf.beamform(state["geom"], rf, case["mode"], max(case["angle"], 0), **kw)
    else:
        pwbf.compound(state["geom"], rf, case["mode"], **kw)
    return dict(out, iq=state["iq"]) if case["kind"] == "iq" else out


def _columns(rows, whole):
    """One array per figure from the list of dicts an entry point returns."""
    return {k: np.array([r[k] for r in rows], dtype=np.int32 if k in whole else np.float32)
            for k in rows[0]}


# ------------------------------------------------------------------ work
_ELEMENT = {"int16": 2, "float16": 2, "float32": 4}
# operations per gathered sample: delay, floor, fraction, interpolation, accumulate; the root
# modes' root and sign, the baseband modes' second interpolation and complex accumulate
_PER_GATHER = {"das": 6, "dmas": 10, "pdas": 9, "iqdas": 12, "bbdmas": 16}


def _pairs(case):
    """(pixel, channel) pairs inside the receive aperture."""
    if case["apod"] == "none":
        return case["nx"] * case["nz"] * case["channels"]
    g = Geometry(case)
    x = g.x0 + np.arange(g.nx) * g.dx
    half = np.maximum(g.z0 + np.arange(g.nz) * g.dz, 0.0) / (2.0 * g.f_number)
    hi = np.searchsorted(g.elem_x, x[:, None] + half, side="left")
    lo = np.searchsorted(g.elem_x, x[:, None] - half, side="right")
    return int(np.maximum(hi - lo, 0).sum())


def _fft_flops(n, rows):
    return 5.0 * n * math.log2(max(n, 2)) * rows


def _image_work(case):
    px = case["nx"] * case["nz"]
    used = 1 if case["angle"] >= 0 else case["angles"]
    records = used * case["channels"]
    planes = len(case["planes"].split(","))
    size = records * case["samples"] * _ELEMENT[case["dtype"]] + 4.0 * px * planes
    if case["kind"] == "fk":
        pad = 2 ** math.ceil(math.log2((2 if case["mode"] == "stolt" else 4) * case["channels"]))
        bins = case["samples"] // 2 + 1
        ops = _fft_flops(case["samples"], records) / 2 + 2 * _fft_flops(pad, bins * used)
        ops += _fft_flops(case["samples"], min(pad, case["channels"]) * used)
        ops += used * (bins * pad * 20.0 + px * 16.0)
        return size, ops
    pairs = _pairs(case)
    ops = pairs * (used * _PER_GATHER[case["mode"]] + 9.0)
    if case["kind"] == "iq":
        every = case["angles"] * case["channels"]
        kept = case["samples"] / case["decimation"]
        size += every * kept * 8.0 + (every - records) * case["samples"] * _ELEMENT[case["dtype"]]
        ops += every * 2.0 * 2.5 * case["samples"] * math.log2(case["samples"])
    elif planes > 1:
        ops += 2.0 * _fft_flops(case["nz"], case["nx"]) / 2
    return size, ops


def work(case):
    if case["kind"] == "batch":
        parts = [_image_work(f) for f in _batch_frames(case)]
        return {"bytes": sum(p[0] for p in parts), "flops": sum(p[1] for p in parts)}
    if case["kind"] == "metrics":
        area = math.pi * (0.8 * 0.5 * (case["radius_min"] + case["radius_max"])) ** 2
        px = case["nx"] * case["nz"] / (38.1e-3 * 40e-3)
        n = px * (2 * case["cysts"] * area + case["targets"] * math.pi * 1e-6)
        return {"bytes": 4.0 * n, "flops": 10.0 * n}
    size, ops = _image_work(case)
    return {"bytes": size, "flops": ops}


# ------------------------------------------------------------------ the same in 64 bits
def _grid(g):
    x = g.x0 + torch.arange(g.nx, dtype=torch.float64, device=DEV) * g.dx
    z = g.z0 + torch.arange(g.nz, dtype=torch.float64, device=DEV) * g.dz
    return x[:, None], z[None, :]


def _weights(g, d, z):
    if g.apod == "none":
        return torch.ones_like(d * z)
    a = z / (2.0 * g.f_number)
    inside = (d.abs() < a) & (z > 0)
    if g.apod == "boxcar":
        return inside.double()
    return torch.where(inside, 0.5 * (1.0 + torch.cos(math.pi * d.abs() / a)), 0.0 * a)


def _sample(rec, s):
    """Linear interpolation of the zero-extended record at positions s."""
    n = torch.floor(s)
    f = s - n
    last = rec.numel() + 1
    at = n.long()
    pad = torch.nn.functional.pad(torch.view_as_real(rec).T, (1, 1)).T if rec.is_complex() \
        else torch.nn.functional.pad(rec, (1, 1))
    pad = torch.view_as_complex(pad.contiguous()) if rec.is_complex() else pad
    lo, hi = pad[(at + 1).clamp(0, last)], pad[(at + 2).clamp(0, last)]
    return lo + f * (hi - lo)


def _beamform64(case, g, rec):
    """The image before post-processing; rec: float64 RF or complex128 baseband records."""
    mode, D = case["mode"], case["decimation"]
    x, z = _grid(g)
    angles = range(case["angles"]) if case["angle"] < 0 else [case["angle"]]
    kind = torch.complex128 if rec.is_complex() else torch.float64
    sums = [torch.zeros(g.nx, g.nz, dtype=kind, device=DEV) for _ in angles]
    squares = torch.zeros(g.nx, g.nz, dtype=torch.float64, device=DEV)
    for e in range(case["channels"]):
        d = x - g.elem_x[e]
        back = torch.sqrt(d * d + z * z)
        w = _weights(g, d, z)
        for k, a in enumerate(angles):
            th = float(g.angles_rad[a])
            s = g.fs / g.c * (x * math.sin(th) + z * math.cos(th) - g.first(a) + back)
            v = _sample(rec[a, e], s / D if rec.is_complex() else s)
            if rec.is_complex():
                ph = 2.0 * math.pi * g.f0 / g.fs * s
                v = v * torch.complex(torch.cos(ph), torch.sin(ph))
                if mode == "bbdmas":
                    v = v / v.abs().sqrt().clamp_min(1e-300)
                sums[k] += w * v
            elif mode == "das":
                sums[k] += w * v
            else:
                root = 2.0 if mode == "dmas" else case["p"]
                r = w * torch.sign(v) * v.abs() ** (1.0 / root)
                sums[k] += r
                if mode == "dmas":
                    squares += r * r
    if mode == "dmas":
        return 0.5 * (sum(t * t for t in sums) - squares)
    if mode == "pdas":
        return sum(torch.sign(t) * t.abs() ** case["p"] for t in sums)
    if mode == "bbdmas":
        return sum(t * t for t in sums)
    return sum(sums)


def _log64(env):
    top = float(env.max())
    if not top > 0:
        return torch.full_like(env, FLOOR_DB)
    return (20.0 * torch.log10(env / top)).clamp_min(FLOOR_DB)


def _analytic_weights(n):
    h = torch.zeros(n, dtype=torch.float64, device=DEV)
    h[0] = 1.0
    h[n // 2] = 1.0
    h[1:n // 2] = 2.0
    return h


def _post64(case, g, rf):
    want = case["planes"].split(",")
    out = {"rf": rf}
    if len(want) > 1:
        h = _analytic_weights(g.nz)
        if case["bandpass"]:
            k = torch.arange(g.nz, device=DEV)
            f = torch.minimum(k, g.nz - k).double() * (g.c / (2.0 * g.nz * g.dz))
            h = torch.where((f >= g.f0) & (f <= 3.0 * g.f0), h, 0.0 * h)
        col = torch.fft.ifft(torch.fft.fft(rf, dim=1) * h, dim=1)
        out.update(filtered=col.real, env=col.abs())
        out["log"] = _log64(out["env"])
    return {k: out[k] for k in want}


def _demodulate64(case, g, rf):
    n, D = case["samples"], case["decimation"]
    spec = torch.fft.fft(rf, dim=2) * _analytic_weights(n)
    if D > 1:
        k = torch.arange(n, device=DEV)
        keep = (k <= n // 2) & ((k.double() * g.fs / n - g.f0).abs() < g.fs / (2.0 * D))
        spec = torch.where(keep, spec, 0.0 * spec)
    t = torch.arange(n, dtype=torch.float64, device=DEV) * (2.0 * math.pi * g.f0 / g.fs)
    iq = torch.fft.ifft(spec, dim=2) * torch.complex(torch.cos(t), -torch.sin(t))
    return iq[:, :, ::D].contiguous()


def _complex_planes(case, y):
    out = {"rf": y.real, "imag": y.imag, "env": y.abs()}
    out["log"] = _log64(out["env"])
    return {k: out[k] for k in case["planes"].split(",")}


def _migrate64(case, g, rf, a):
    """Steps 1 to 5 of the library's reading of the f-k migrations, one angle."""
    stolt = case["mode"] == "stolt"
    th = float(g.angles_rad[a])
    sn, cs = math.sin(th), math.cos(th)
    N, Nt = case["channels"], case["samples"]
    K, Nx = Nt // 2 + 1, 1
    while Nx < (2 if stolt else 4) * N:
        Nx *= 2
    f64 = dict(dtype=torch.float64, device=DEV)
    bins = torch.arange(K, **f64)
    ex = torch.tensor(g.elem_x, **f64)
    fire = (ex * sn - g.first(a)) / g.c
    tau = fire if stolt else fire[:1]
    ph = 2.0 * math.pi * bins * (g.fs / Nt) * tau[:, None]
    spec = torch.fft.fft(rf[a], dim=1)[:, :K] * torch.complex(torch.cos(ph), torch.sin(ph))
    spec = torch.fft.fft(spec, n=Nx, dim=0)
    spec = torch.cat([spec, torch.zeros(Nx, 1, dtype=spec.dtype, device=DEV)], 1)  # [Nx, K + 1]
    m = torch.arange(Nx, **f64)
    kx = (torch.where(m < Nx // 2, m, m - Nx) / (Nx * PITCH))[:, None]
    df = g.fs / Nt
    row = torch.arange(Nx, device=DEV)[:, None]
    if stolt:
        v = g.c / (math.sqrt(2.0) * cs * cs)
        kz = (bins * df / v)[None, :]
        rho = torch.sqrt(kx * kx + kz * kz)
        u = v * rho / df
        ok = (rho > 0) & (u < K)
        i0 = torch.where(ok, torch.floor(u), 0.0 * u).long()
        w = u - i0
        val = (1.0 - w) * spec[row, i0] + w * spec[row, i0 + 1]
        jac = kz / rho.clamp_min(1e-300)
        step_z = v / g.fs
    else:
        kz = (2.0 * bins * df / g.c)[None, :]
        den = kx * sn + kz * cs
        k = torch.where(den > 0, (kx * kx + kz * kz) / (2.0 * den.clamp_min(1e-300)), 0.0 * den)
        kr = kz - k * cs
        u = k * g.c / df
        ok = (den > 0) & (kr >= 0) & (u < K)
        mf = torch.where(ok, (kx - k * sn) * (Nx * PITCH), 0.0 * u)
        m0 = torch.floor(mf)
        wm = mf - m0
        i0 = torch.where(ok, torch.floor(u), 0.0 * u).long()
        w = u - i0
        m0 = m0.long() % Nx
        m1 = (m0 + 1) % Nx
        val = (1.0 - wm) * ((1.0 - w) * spec[m0, i0] + w * spec[m0, i0 + 1]) \
            + wm * ((1.0 - w) * spec[m1, i0] + w * spec[m1, i0 + 1])
        jac = kr / den.clamp_min(1e-300)
        step_z = g.c / (2.0 * g.fs)
    img = torch.fft.ifft(torch.where(ok, val * jac, 0.0 * val), dim=0)
    img = torch.fft.ifft(torch.nn.functional.pad(torch.view_as_real(img).permute(2, 0, 1),
                                                 (0, Nt - K)).permute(1, 2, 0).contiguous()
                         .view(torch.complex128).squeeze(-1), dim=1)  # [Nx, Nt]
    x, z = _grid(g)
    if stolt:
        ux, uz = x + z * math.tan(th), math.sqrt(2.0) * z / cs + 0.0 * x
    else:
        ux, uz = x + 0.0 * z, z + 0.0 * x
    ux, uz = (ux - float(g.elem_x[0])) / PITCH, uz / step_z
    i0, j0 = torch.floor(ux), torch.floor(uz)
    out = torch.zeros(g.nx, g.nz, dtype=torch.complex128, device=DEV)
    for di, wx in ((0, 1.0 - (ux - i0)), (1, ux - i0)):
        for dj, wz in ((0, 1.0 - (uz - j0)), (1, uz - j0)):
            i, j = (i0 + di).long(), (j0 + dj).long()
            inside = (i >= 0) & (i < Nx) & (j >= 0) & (j < Nt)
            out += torch.where(inside, wx * wz, 0.0 * wx) * img[i.clamp(0, Nx - 1), j.clamp(0, Nt - 1)]
    return out


def _image64(case, seed):
    g = Geometry(case)
    rf = _records(case, g, seed).double()
    if case["kind"] == "fk":
        angles = range(case["angles"]) if case["angle"] < 0 else [case["angle"]]
        return _complex_planes(case, sum(_migrate64(case, g, rf, a) for a in angles))
    if case["kind"] == "iq":
        iq = _demodulate64(case, g, rf)
        return dict(_complex_planes(case, _beamform64(case, g, iq)), iq=iq)
    return _post64(case, g, _beamform64(case, g, rf))


def _disc(g, disc):
    """Pixels of a disc: the entry point's float32 rule, one rounding per operation."""
    cx, cz = np.float32((disc[0] - g.x0) / g.dx), np.float32((disc[1] - g.z0) / g.dz)
    sx, sz = np.float32(g.dx / disc[2]), np.float32(g.dz / disc[2])
    u = (np.arange(g.nx, dtype=np.float32) - cx) * sx
    v = (np.arange(g.nz, dtype=np.float32) - cz) * sz
    return (u * u)[:, None] + (v * v)[None, :] <= np.float32(1.0)


def _width64(line, at, half, step):
    i = j = at
    while i >= 0 and line[i] >= half:
        i -= 1
    while j < len(line) and line[j] >= half:
        j += 1
    if i < 0 or j >= len(line):
        return math.nan
    left = i + (half - line[i]) / (line[i + 1] - line[i])
    right = j - 1 + (half - line[j - 1]) / (line[j] - line[j - 1])
    return (right - left) * step


def _metrics64(case, seed):
    env, cysts, targets, size = _envelope(case, seed)
    g = _metrics_geometry(case, size)
    env = env.double().cpu().numpy()
    contrast, resolution = [], []
    for inner, outer in cysts:
        a, b = env[_disc(g, inner)], env[_disc(g, outer)]
        mu, sd = (a.mean(), b.mean()), (a.std(), b.std())
        contrast.append({"mu_in": mu[0], "mu_out": mu[1], "sigma_in": sd[0], "sigma_out": sd[1],
                         "cr_db": 20.0 * math.log10(mu[0] / mu[1]),
                         "cnr": (mu[0] - mu[1]) / math.sqrt(0.5 * (sd[0] ** 2 + sd[1] ** 2)),
                         "n_in": len(a), "n_out": len(b)})
    for t in targets:
        at = int(np.argmax(np.where(_disc(g, t), env, -np.inf)))
        ix, iz = at // g.nz, at % g.nz
        peak = env[ix, iz]
        resolution.append({"peak": peak, "fwhm_x": _width64(env[:, iz], ix, 0.5 * peak, g.dx),
                           "fwhm_z": _width64(env[ix], iz, 0.5 * peak, g.dz),
                           "ix": ix, "iz": iz})

    def columns(rows, whole):
        return {k: np.array([r[k] for r in rows], dtype=np.int32 if k in whole else np.float64)
                for k in rows[0]}
    return {"contrast": columns(contrast, ("n_in", "n_out")),
            "resolution": columns(resolution, ("ix", "iz"))}


def exact(case, seed):
    if case["kind"] == "metrics":
        return _metrics64(case, seed)
    if case["kind"] == "batch":
        return [_image64(f, seed * 1000 + i) for i, f in enumerate(_batch_frames(case))]
    return _image64(case, seed)
