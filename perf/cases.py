"""What this library is timed on: imaging frames as a user's program sends them.

A case is one pass through the public Python entry points (``Plan.envelope``,
``Plan.beamform``, ``Plan.matched_filter``, ``Server``) on pulse-echo or
near-field recordings made on the GPU from a seed. ``prepare`` holds what a
program keeps (the plan or the server) and the recordings it has in hand;
``run`` is the pass; ``exact`` is the same image in 64 bits in plain torch.

Fields of a case (``serve`` cases hold ranges of these per frame):
  kind      "image" (one frame), "pipeline" (raw channels -> matched filter ->
            image) or "serve" (several host frames through a Server)
  array     "disc" (random planar disc), "hex" (5 mm hexagonal lattice in a
            disc) or "grid" (rectangular, 1 cm pitch)
  mics      microphones (disc), aperture: its diameter in metres
  nx, ny    microphones of a rectangular grid; radius: of a hexagonal disc
  scan      "arc" (azimuths), "azel" (azimuth x elevation) or "voxels"
  n_az, n_el, n_z   scan points per axis (azimuths/x, elevations/y, depths)
  samples, order, cf, output, dtype, accumulate, linear, decimation: as Plan's
"""

from __future__ import annotations

import math

import numpy as np
import torch

from paper_2511_09165_amd import Plan, Server

C = 343.0
CF_EPS = 1e-20
FIR_LEN, FIR_HZ = 63, 5000.0
TORCH_DTYPE = {"f32": torch.float32, "f16": torch.float16, "bf16": torch.bfloat16}


def _image(name, **kw):
    case = dict(name=name, kind="image", array="disc", mics=32, aperture=0.12, nx=0, ny=0, radius=0.0,
                scan="azel", n_az=91, n_el=46, n_z=1, samples=16384, order=5, cf=True, output="envelope",
                dtype="f32", accumulate="f32", linear=False, decimation=1)
    case.update(kw)
    return case


def listed():
    return [
        # the smallest call: a handful of microphones and one azimuth sweep, as an obstacle detector
        # images every ping; launches and host time count
        _image("burst8-order2", mics=8, aperture=0.05, scan="arc", n_az=64, n_el=1, samples=1024, order=2),
        # a plain horizontal sweep of a small lattice, no coherence factor, a record of odd length
        # (beamwidth and dynamic-range studies run many of these)
        _image("hex19-order3-nocf", array="hex", radius=0.01, scan="arc", n_az=181, n_el=1, samples=3001,
               order=3, cf=False),
        # the eRTIS-like frame at 2 degrees and order 5: what a sonar head images per pulse
        _image("ertis32-order5", order=5),
        # the RF image of a half-length frame at order 3, for callers with a detector of their own
        _image("ertis32-order3-rf", n_az=64, n_el=32, samples=8192, order=3, output="beamform"),
        # a larger head storing FP16 channels, a small grid
        _image("disc64-order3-f16", mics=64, aperture=0.16, n_az=45, n_el=23, samples=8192, order=3, dtype="f16"),
        # even order on BF16 channels with a grid of odd sizes
        _image("disc48-order4-bf16", mics=48, aperture=0.10, n_az=61, n_el=31, samples=5003, order=4, dtype="bf16"),
        # many microphones, one horizontal sweep (the largest lattice of the beamwidth studies)
        _image("hex517-order2", array="hex", radius=0.06, scan="arc", n_az=361, n_el=1, samples=4096, order=2),
        # near-field volume of a 1024-microphone array: the largest frame
        _image("nearfield1024-order3", array="grid", nx=32, ny=32, scan="voxels", n_az=64, n_el=64, n_z=32,
               samples=2048, order=3),
        # interpolated delays at the headline order
        _image("ertis32-order5-linear", n_az=64, n_el=32, samples=8192, order=5, linear=True),
        # the accurate form: FP64 sums at a high order
        _image("ertis32-order7-f64sums", n_az=45, n_el=23, samples=4096, order=7, accumulate="f64"),
        # raw channels -> matched filter -> envelope of every 20th sample (a display's rate)
        _image("pipeline32-order5-dec20", kind="pipeline", n_az=64, n_el=32, decimation=20),
        # a burst of frames of different arrays, grids and orders through the request loop,
        # results brought back to the host
        dict(name="serve12-mixed", kind="serve", frames=12, max_mics=64, max_dirs=4096, max_samples=8192),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    what = rng.choice(["disc", "disc", "disc", "disc", "precise", "linear", "hex", "hex", "near", "near",
                       "pipeline", "serve"])
    if what == "serve":
        return {k: v for k, v in dict(kind="serve", frames=rng.randint(4, 20), max_mics=rng.choice([16, 32, 64]),
                                      max_dirs=_log_int(rng, 512, 4096),
                                      max_samples=_log_int(rng, 2048, 8192)).items()}
    case = _image("")
    del case["name"]
    case.update(order=rng.choice([1, 2, 3, 3, 4, 5, 5, 6, 7, 8]), cf=rng.random() < 0.8,
                output="envelope" if rng.random() < 0.75 else "beamform",
                dtype=rng.choice(["f32", "f32", "f16", "bf16"]), samples=_log_int(rng, 900, 16384))
    if what == "near":
        nx, ny = rng.randint(8, 32), rng.randint(8, 32)
        n_az, n_el, n_z = rng.randint(5, 48), rng.randint(5, 48), rng.randint(1, 12)
        case.update(array="grid", nx=nx, ny=ny, scan="voxels", n_az=n_az, n_el=n_el, n_z=n_z,
                    samples=_log_int(rng, 700, 3000))
        return case
    if what == "hex":
        case.update(array="hex", radius=rng.choice([0.01, 0.02, 0.03, 0.04, 0.05, 0.06]), scan="arc",
                    n_az=_log_int(rng, 61, 721), n_el=1, samples=_log_int(rng, 900, 8192))
        return case
    case.update(mics=_log_int(rng, 8, 64), aperture=round(rng.uniform(0.05, 0.20), 3))
    if rng.random() < 0.25:
        case.update(scan="arc", n_az=_log_int(rng, 40, 361), n_el=1)
    else:
        n = math.sqrt(_log_int(rng, 200, 8192) / 2.0)
        case.update(n_az=int(2 * n), n_el=max(2, int(n)))
    if what == "precise":
        case.update(cf=True, accumulate=rng.choice(["f64", "f64", "kahan"]), samples=min(case["samples"], 8192))
    elif what == "linear":
        case.update(cf=True, linear=True)
    elif what == "pipeline":
        case.update(kind="pipeline", dtype="f32", output="envelope", decimation=rng.randint(2, 24))
    return case


# -- geometry ---------------------------------------------------------------

def _disc(rng, mics, aperture):
    """Uniform points of a disc, kept apart."""
    apart = min(0.004, aperture / (2.5 * math.sqrt(mics)))
    pts = []
    while len(pts) < mics:
        p = rng.uniform(-aperture / 2, aperture / 2, 2)
        if p @ p <= aperture * aperture / 4 and all(np.hypot(*(p - q)) >= apart for q in pts):
            pts.append(p)
    return np.concatenate([np.array(pts), np.zeros((mics, 1))], axis=1)


def _mics(case):
    if case["array"] == "grid":
        x = (np.arange(case["nx"]) - (case["nx"] - 1) / 2) * 0.01
        y = (np.arange(case["ny"]) - (case["ny"] - 1) / 2) * 0.01
        yy, xx = np.meshgrid(y, x, indexing="ij")
        return np.stack([xx.ravel(), yy.ravel(), np.zeros(xx.size)], axis=1)
    if case["array"] == "hex":
        edge, r = 0.005, case["radius"]
        k = int(math.ceil(r / edge)) * 2 + 4
        pts = [(edge * (i + 0.5 * j), edge * math.sqrt(0.75) * j, 0.0)
               for j in range(-k, k + 1) for i in range(-2 * k, 2 * k + 1)]
        return np.array([p for p in pts if p[0] ** 2 + p[1] ** 2 <= r * r * (1 + 1e-12)])
    return _disc(np.random.default_rng(1000 * case["mics"] + int(1e4 * case["aperture"])), case["mics"],
                 case["aperture"])


def _scan(case):
    if case["scan"] == "voxels":
        def axis(n, lo, hi):
            return lo + (hi - lo) / n * (np.arange(n) + 0.5)
        zz, yy, xx = np.meshgrid(axis(case["n_z"], 1.0, 1.0 + case["n_z"] / 64), axis(case["n_el"], -0.5, 0.5),
                                 axis(case["n_az"], -0.5, 0.5), indexing="ij")
        return np.stack([xx.ravel(), yy.ravel(), zz.ravel()], axis=1)
    az = np.deg2rad(np.linspace(-90, 90, case["n_az"]))
    el = np.deg2rad(np.linspace(-45, 45, case["n_el"]) if case["n_el"] > 1 else np.zeros(1))
    ee, aa = np.meshgrid(el, az, indexing="ij")
    ee, aa = ee.ravel(), aa.ravel()
    return np.stack([np.cos(ee) * np.sin(aa), np.sin(ee), np.cos(ee) * np.cos(aa)], axis=1)


def _fs(case):
    return 192e3 if case["scan"] == "voxels" else 450e3


def _chirp(fs):
    t = np.arange(int(round(1e-3 * fs))) / fs
    return np.sin(2 * np.pi * (25e3 * t + 0.5 * 50e6 * t * t))


# -- recordings -------------------------------------------------------------

def _channels(case, seed):
    """FP64 recordings (M, T) on the GPU. Far field: echoes of the chirp from 20 reflectors at 1/r^2, white
    noise 20 dB below the strongest, matched filtered (raw for "pipeline"). Near field: five band-limited noise
    sources at 0 dB."""
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    rng = np.random.default_rng(seed)
    fs, T = _fs(case), case["samples"]
    mics = _mics(case)
    M = len(mics)
    nfft = 1 << int(math.ceil(math.log2(T + 4096)))
    f = torch.arange(nfft // 2 + 1, device="cuda", dtype=torch.float64) * (fs / nfft)

    def arrivals(spectrum, seconds, amps):
        s = torch.zeros(M, f.numel(), device="cuda", dtype=torch.complex128)
        for k in range(len(amps)):
            tau = torch.from_numpy(seconds[k]).cuda()
            a = torch.from_numpy(np.broadcast_to(amps[k], (M,)).copy()).cuda()
            s += a[:, None] * torch.exp(-2j * math.pi * tau[:, None] * f[None, :]) * spectrum(k)[None, :]
        return s

    if case["scan"] == "voxels":
        src = np.stack([rng.uniform(-0.5, 0.5, 5), rng.uniform(-0.5, 0.5, 5),
                        rng.uniform(1.0, 1.0 + case["n_z"] / 64, 5)], axis=1)
        dist = np.linalg.norm(src[:, None, :] - mics[None], axis=2)
        band = ((f >= 20e3) & (f <= 80e3)).to(torch.float64)

        def noise(_):
            w = torch.randn(nfft, generator=gen, device="cuda", dtype=torch.float64)
            return torch.fft.rfft(w) * band

        x = torch.fft.irfft(arrivals(noise, dist / C, 1.0 / dist), nfft)[:, :T]
        return x + x.std() * torch.randn(M, T, generator=gen, device="cuda", dtype=torch.float64)
    pulse = _chirp(fs)
    P = torch.fft.rfft(torch.from_numpy(pulse).cuda(), nfft)
    r_hi = max(0.35, min(5.0, 0.5 * C * (T - pulse.size - 4) / fs - 0.2))
    r = rng.uniform(0.1 if r_hi < 0.5 else 0.3, r_hi, 20)
    az, el = rng.uniform(-math.pi / 2, math.pi / 2, 20), rng.uniform(-math.pi / 4, math.pi / 4, 20)
    p = r[:, None] * np.stack([np.cos(el) * np.sin(az), np.sin(el), np.cos(el) * np.cos(az)], axis=1)
    path = np.linalg.norm(p, axis=1)[:, None] + np.linalg.norm(p[:, None, :] - mics[None], axis=2)
    raw = torch.fft.irfft(arrivals(lambda _: P, path / C, 1.0 / r ** 2), nfft)[:, :T]
    sigma = float(np.max(1.0 / r ** 2) * np.sqrt(np.mean(pulse ** 2)) / 10)
    raw = raw + sigma * torch.randn(M, T, generator=gen, device="cuda", dtype=torch.float64)
    if case["kind"] == "pipeline":
        return raw.contiguous()
    return torch.fft.irfft(torch.fft.rfft(raw, nfft) * P.conj(), nfft)[:, :T].contiguous()


def _stored(case, seed):
    """The channels in the case's storage type, and the scale that undoes the storage's."""
    x = _channels(case, seed)
    scale = 1.0 if case["dtype"] == "f32" else float(np.float32(x.abs().max().item()))
    return (x / scale).to(TORCH_DTYPE[case["dtype"]]), scale


def _plan(case):
    pipe = case["kind"] == "pipeline"
    return Plan(_mics(case), _scan(case), case["samples"], case["order"], _fs(case), c=C, use_cf=case["cf"],
                nearfield=case["scan"] == "voxels", in_dtype=case["dtype"], linear=case["linear"],
                accumulate=case["accumulate"], env_decimation=case["decimation"],
                mf_pulse=_chirp(_fs(case)) if pipe else None)


def _frames(case, seed):
    """The image cases of a serving burst: arrays, grids, orders and lengths drawn for each frame; the mix
    belongs to the case, the recordings to the seed."""
    rng = np.random.default_rng(case["frames"] + case["max_dirs"])
    out = []
    for _ in range(case["frames"]):
        m = int(rng.choice([k for k in (16, 32, 64) if k <= case["max_mics"]]))
        n = math.sqrt(case["max_dirs"] / float(rng.choice([1, 2, 4])) / 2)
        f = _image("", mics=m, aperture=round(float(rng.uniform(0.06, 0.20)), 3), n_az=int(2 * n), n_el=int(n),
                   samples=int(case["max_samples"] // rng.choice([1, 2])), order=int(rng.choice([3, 5])),
                   decimation=16)
        out.append((f, int(rng.integers(1 << 30)) + seed))
    return out


# -- one pass ---------------------------------------------------------------

def prepare(case, seed):
    if case["kind"] == "serve":
        frames = _frames(case, seed)
        jobs = [(_plan(f), _stored(f, s)[0].cpu().numpy()) for f, s in frames]
        return {"kind": "serve", "jobs": jobs, "server": Server(1 << 30, staging=128 << 20)}
    x, scale = _stored(case, seed)
    return {"kind": case["kind"], "plan": _plan(case), "x": x, "scale": scale, "output": case["output"]}


def run(state):
    if state["kind"] == "serve":
        server = state["server"]
        tickets = [server.submit(plan, x) for plan, x in state["jobs"]]
        images = []
        for t in tickets:
            server.wait(t)
            images.append(server.fetch(t))
            server.release(t)
        return images
    plan, x = state["plan"], state["x"]
    if state["kind"] == "pipeline":
        x = plan.matched_filter(x)
        return {"channels": x, "image": plan.envelope(x)}
    if state["output"] == "envelope":
        return plan.envelope(x, in_scale=state["scale"])
    return plan.beamform(x, in_scale=state["scale"])


# -- what a pass cannot do without --------------------------------------------

def _sizes(case):
    mics = {"disc": case["mics"], "grid": case["nx"] * case["ny"]}.get(case["array"]) or len(_mics(case))
    return mics, case["n_az"] * case["n_el"] * case["n_z"], case["samples"]


def work(case):
    """Channels read and image written once; per microphone and pixel the powers and power sums (and the sums of
    the coherence factor), per pixel Newton-Girard, the factor and the envelope filter."""
    if case["kind"] == "serve":
        every = [work(f) for f, _ in _frames(case, 0)]
        return {k: sum(w[k] for w in every) for k in ("bytes", "flops")}
    M, D, T = _sizes(case)
    n, env = case["order"], case["output"] == "envelope"
    out = -(-T // case["decimation"]) if env else T
    size = 4 if case["dtype"] == "f32" else 2
    per_mic = 1 + (2 * (n - 2) + 1 if n > 1 else 0) + max(0, n // 2 - 1)
    if case["cf"]:
        per_mic += 2 + (1 if n % 2 == 0 else 0)
    if case["linear"]:
        per_mic += 3 + 4
    per_pixel = n * (n + 1) + (6 if case["cf"] else 0)
    flops = D * T * (M * per_mic + per_pixel) + (D * out * 2 * FIR_LEN if env else 0) + 4 * M * T
    moved = M * T * size + D * out * 4
    if case["kind"] == "pipeline":
        taps = _chirp(_fs(case)).size
        flops += 2 * M * T * taps
        moved += M * T * 4
    return {"bytes": moved, "flops": flops}


# -- the same image in 64 bits ------------------------------------------------

def _lowpass(fs):
    """Hamming-windowed sinc of unit gain at DC, as FP32 taps."""
    m = np.arange(FIR_LEN) - (FIR_LEN - 1) / 2
    h = np.sinc(2 * FIR_HZ / fs * m) * np.hamming(FIR_LEN)
    return (h / h.sum()).astype(np.float32).astype(np.float64)


def _delays(mics, points, fs, near):
    """fs * tau of every (point, microphone), one rounding an operation."""
    r, v = mics[None], points[:, None]
    if near:
        q = (v - r) ** 2
        o = points ** 2
        d = np.sqrt(q[..., 0] + q[..., 1] + q[..., 2]) - np.sqrt(o[:, 0] + o[:, 1] + o[:, 2])[:, None]
    else:
        d = -(r[..., 0] * v[..., 0] + r[..., 1] * v[..., 1] + r[..., 2] * v[..., 2])
    return fs * (d / C)


def _exact_image(case, x, scale):
    n, cf, T = case["order"], case["cf"], case["samples"]
    mics, points = _mics(case), _scan(case)
    M, fs, near = len(mics), _fs(case), case["scan"] == "voxels"
    x = x.double()
    h = _lowpass(fs)
    env, dec = case["output"] == "envelope", case["decimation"]
    out = torch.empty(len(points), -(-T // dec) if env else T, device="cuda", dtype=torch.float64)
    rows = max(1, (1 << 24) // T)
    t = torch.arange(T, device="cuda")
    for p0 in range(0, len(points), rows):
        f = _delays(mics, points[p0:p0 + rows], fs, near)
        whole = np.floor(f) if case["linear"] else np.floor(f + 0.5)
        frac = torch.from_numpy(f - whole).cuda()
        whole = torch.from_numpy(whole.astype(np.int64)).cuda()
        pad = int(whole.abs().max()) + 2
        D = whole.shape[0]
        P = torch.zeros(n + 1, D, T, device="cuda", dtype=torch.float64)
        a = torch.zeros(D, T, device="cuda", dtype=torch.float64)
        b = torch.zeros_like(a)
        for i in range(M):
            row = torch.nn.functional.pad(x[i], (pad, pad))
            at = t[None, :] + (whole[:, i, None] + pad)
            v = row[at]
            if case["linear"]:
                v = v + frac[:, i, None] * (row[at + 1] - v)
            s = v.sign() * v.abs() ** (1.0 / n)
            power = s.clone()
            for k in range(1, n + 1):
                P[k] += power
                power *= s
            a += v
            b += v * v
        e = [torch.ones_like(a)]
        for k in range(1, n + 1):
            e.append(sum((1 if i % 2 else -1) * e[k - i] * P[i] for i in range(1, k + 1)) / k)
        y = e[n] * scale
        if cf:
            y = y * a * a / (M * b + CF_EPS)
        if env:
            half = (FIR_LEN - 1) // 2
            m = torch.nn.functional.pad(y.abs(), (half, half))
            y = sum(float(h[k]) * m[:, 2 * half - k:2 * half - k + T] for k in range(FIR_LEN))[:, ::dec]
        out[p0:p0 + D] = y
    return out


def exact(case, seed):
    if case["kind"] == "serve":
        return [_exact_image(f, _stored(f, s)[0], 1.0) for f, s in _frames(case, seed)]
    M, D, T = _sizes(case)
    if M * D * T > 3e10:  # minutes in 64 bits
        return None
    x, scale = _stored(case, seed)
    if case["kind"] == "pipeline":
        raw = x.double()
        pulse = torch.from_numpy(_chirp(_fs(case)).astype(np.float32).astype(np.float64)).cuda()
        m = torch.nn.functional.pad(raw, (0, pulse.numel()))
        x = torch.zeros_like(raw)
        for k in range(pulse.numel()):
            x += pulse[k] * m[:, k:k + T]
        return {"channels": x, "image": _exact_image(case, x, 1.0)}
    return _exact_image(case, x, scale)
