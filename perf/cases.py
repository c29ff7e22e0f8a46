"""Performance cases of the acquisition engine: what its users have it do, at the sizes they do it at.

A case is a dict of plain values.  Three kinds, each through a public entry point of the package:
  search   one record in device memory, Context.acquire_device (precision, sample format, rate and
           options as named), or with host=1 one record in host memory, gnss_acquire
  batch    several different records in device memory, Context.acquire_batch_device
  track    early / prompt / late correlators of records in device memory, Context.track_device

Records are noise with planted satellites, quantised as a front end does (2-bit real IF or int8
complex baseband), made on the GPU from the seed alone.  A program keeps one context per precision
and option set, and one request per buffer it records into: prepare() makes those, run() is the call.

Results: the power grid whole, and of each peak record the whole numbers (PRN, Doppler bin, code
phase, detected) and the powers (peak, second, mean, ratio).  The two refined doubles of a record are
quotients of differences of neighbouring FP32 grid values, doubles by type and single precision by
content; all that they are made of is in the grid.
"""
import math
import random

import numpy as np
import torch

import paper_1309_0052_amd as G

PRECISION = {"fp32": G.GNSS_FP32, "fp16": G.GNSS_FP16, "pfa": G.GNSS_FP16_PFA}
FORMAT = {"i8": G.GNSS_REAL_I8, "ci8": G.GNSS_CPLX_I8, "2bit": G.GNSS_REAL_2BIT_PACKED}
CHIP_RATE = 1023000
L1_HZ = 1575.42e6


def _search(name, fs_khz, fmt, n_prn, bins, step, t_coh, blocks, precision="fp32", **more):
    c = {"kind": "search", "fs_khz": fs_khz, "fmt": fmt, "n_prn": n_prn, "bins": bins, "step": step,
         "t_coh": t_coh, "blocks": blocks, "precision": precision, "host": 0, "code_doppler": 0,
         "doppler_fd": 0, "nav_pairs": 0, "strong": 0}
    c.update(more)
    return dict(c, name=name) if name else c


def listed():
    return [
        # one satellite looked for again a few bins around where it was: the smallest call, all latency
        _search("reacquire-1sat", 4092, "i8", 1, 5, 250.0, 1, 4, strong=1),
        # cold start on 10 ms of a 2-bit front end (the strong-signal workload)
        _search("strong-4MHz", 4092, "i8", 32, 21, 500.0, 1, 10, strong=1),
        # the same record uploaded by a client: host buffers in and out, the grid with it
        _search("strong-4MHz-host", 4092, "i8", 32, 21, 500.0, 1, 10, strong=1, host=1),
        # weak signals, 100 ms at 16.368 MHz (the default workload), in the three precisions
        _search("weak-16MHz", 16368, "ci8", 32, 121, 125.0, 4, 25),
        _search("weak-16MHz-fp16", 16368, "ci8", 32, 121, 125.0, 4, 25, "fp16"),
        _search("weak-16MHz-pfa", 16368, "ci8", 32, 121, 125.0, 4, 25, "pfa"),
        # the same search of a recorder that runs at 10 MHz, no multiple of the chip rate
        _search("weak-10MHz", 10000, "ci8", 32, 121, 125.0, 4, 25),
        # a packed 2-bit recorder at 5 MHz
        _search("if-5MHz-2bit", 5000, "2bit", 32, 41, 250.0, 2, 10),
        # a long integration with code-Doppler compensation, past one group of block sums
        _search("long-8MHz", 8184, "ci8", 12, 41, 250.0, 2, 300, code_doppler=1),
        # records of many clients searched together
        {"name": "batch-24", "kind": "batch", "requests": 24, "precision": "fp32"},
        # correlators of a receiver's channels over stored records, and of one live receiver's last 20 ms
        {"name": "track-32rec", "kind": "track", "records": 32, "channels": 12, "fs_khz": 16368, "fmt": "ci8",
         "epochs": 100, "epoch_ms": 1},
        {"name": "track-live", "kind": "track", "records": 1, "channels": 10, "fs_khz": 4092, "fmt": "ci8",
         "epochs": 20, "epoch_ms": 1},
    ]


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    kind = rng.choices(["search", "batch", "track"], [8, 1, 2])[0]
    if kind == "batch":
        return {"kind": "batch", "requests": rng.randint(2, 24), "precision": rng.choice(["fp32", "pfa", "fp16"])}
    if kind == "track":
        return {"kind": "track", "records": _log_int(rng, 1, 32), "channels": rng.randint(1, 16),
                "fs_khz": rng.choice([2046, 4092, 5000, 8184, 16368]), "fmt": rng.choice(["i8", "ci8", "2bit"]),
                "epochs": _log_int(rng, 1, 80), "epoch_ms": rng.choice([1, 1, 2, 4])}
    general = rng.random() < 0.35
    fs_khz = _log_int(rng, 1500, 16384) if general else 1023 * rng.choice([2, 4, 5, 8, 12, 16])
    precision = "fp32" if general else rng.choice(["fp32", "fp32", "fp16", "pfa"])
    fmt = rng.choice(["i8", "ci8", "2bit"])
    t_coh = rng.choice([1, 1, 2, 4, 5, 10])
    most = 4.0e10 if not general else 1.2e10  # flops: below the largest listed case's by a margin
    while True:
        c = _search("", fs_khz, fmt, _log_int(rng, 1, 32), _log_int(rng, 1, 121), 500.0 / t_coh, t_coh,
                    _log_int(rng, 1, 60), precision, strong=rng.randint(0, 1))
        if work(c)["flops"] <= most and t_coh * c["blocks"] <= 200:
            break
    if not general and rng.random() < 0.2:
        c["code_doppler"] = 1
    elif precision == "pfa" and rng.random() < 0.25 and c["blocks"] >= 2:
        c["nav_pairs"] = 1
        c["blocks"] -= c["blocks"] % 2
    elif precision == "pfa" and rng.random() < 0.4 and fs_khz in (2046, 4092, 8184, 16368) and t_coh in (1, 2, 4):
        c["doppler_fd"] = 1
    if precision == "fp32" and rng.random() < 0.15:
        c["host"] = 1
    return c


def _batch_requests(case):
    """The searches of a batch: the heterogeneous records of the batch workload, shorter."""
    rng = random.Random(1000 + case["requests"])
    out = []
    for _ in range(case["requests"]):
        fs = rng.choice([4092, 8184, 16368])
        half = rng.randint(4, 20)
        out.append(_search("", fs, rng.choice(["i8", "ci8"]), rng.randint(8, 32), 2 * half + 1, 500.0, 1,
                           rng.randint(20, 60), case["precision"], strong=1))
    return out


# --- work ---------------------------------------------------------------------------------------

def _bytes_of(fmt, n):
    return n * 2 if fmt == "ci8" else n if fmt == "i8" else -(-n // 4)


def work(case):
    if case["kind"] == "batch":
        each = [work(c) for c in _batch_requests(case)]
        return {k: sum(e[k] for e in each) for k in ("bytes", "flops")}
    if case["kind"] == "track":
        n = case["fs_khz"] * case["epoch_ms"] * case["epochs"] * case["records"]
        out = case["records"] * case["channels"] * case["epochs"] * 48
        # complex mixing (6) and three complex +-y sums (6) per sample and channel
        return {"bytes": _bytes_of(case["fmt"], n) + out, "flops": 12 * n * case["channels"]}
    N, n = case["fs_khz"], case["fs_khz"] * case["t_coh"] * case["blocks"]
    units = case["bins"] * case["blocks"]
    fft = 5.0 * N * math.log2(N)
    flops = units * fft + units * case["n_prn"] * (fft + 10.0 * N) + 8.0 * n * case["bins"]
    return {"bytes": _bytes_of(case["fmt"], n) + 4 * case["n_prn"] * case["bins"] * N + 48 * case["n_prn"],
            "flops": flops}


# --- records ------------------------------------------------------------------------------------

#: IS-GPS-200 Table 3-Ia, G2 delay in chips of PRN 1..32
G2_DELAY = [5, 6, 7, 8, 17, 18, 139, 140, 141, 251, 252, 254, 255, 256, 257, 258, 469, 470, 471, 472, 473, 474, 509,
            512, 513, 514, 515, 516, 859, 860, 861, 862]


def _ca_code(prn):
    """The C/A code as +-1 (chip 0 -> +1)."""
    g1, g2 = [1] * 10, [1] * 10
    a, b = np.empty(1023, np.int64), np.empty(1023, np.int64)
    for i in range(1023):
        a[i], b[i] = g1[9], g2[9]
        g1 = [g1[2] ^ g1[9]] + g1[:9]
        g2 = [g2[1] ^ g2[2] ^ g2[5] ^ g2[7] ^ g2[8] ^ g2[9]] + g2[:9]
    return 1 - 2 * (a ^ np.roll(b, G2_DELAY[prn - 1]))


_codes = {}


def _chips(prn):
    if prn not in _codes:
        _codes[prn] = torch.from_numpy(_ca_code(prn)).cuda()
    return _codes[prn]


def _record(fs_khz, fmt, n, f_if, planted, seed):
    """Quantised samples on the GPU: planted is a list of (prn, code phase, Doppler, dB-Hz, phase, bits)."""
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    fs = fs_khz * 1000
    cplx = fmt == "ci8"
    re = torch.randn(n, generator=g, device="cuda")
    im = torch.randn(n, generator=g, device="cuda") if cplx else None
    at = torch.arange(n, device="cuda", dtype=torch.int64)
    for prn, phase, doppler, dbhz, theta, bits in planted:
        amp = math.sqrt((2.0 if cplx else 4.0) * 10.0 ** (dbhz / 10.0) / fs)
        w = amp * _chips(prn)[((at - phase) * CHIP_RATE).div(fs, rounding_mode="floor") % 1023].float()
        if bits:
            signs = torch.randint(0, 2, (n // (20 * fs_khz) + 3,), generator=g, device="cuda") * 2 - 1
            w = w * signs[(at - phase).div(20 * fs_khz, rounding_mode="floor") + 1]
        turn = (at.double() * ((f_if + doppler) / fs)) % 1.0
        ang = (2.0 * math.pi) * turn.float() + theta
        re += w * torch.cos(ang)
        if cplx:
            im += w * torch.sin(ang)
    if cplx:
        return torch.stack([re, im], 1).mul_(16.0).round_().clamp_(-127, 127).to(torch.int8).reshape(-1)
    mag = torch.where(re.abs() < re.std(), 1, 3)
    if fmt == "i8":
        return torch.where(re < 0, -mag, mag).to(torch.int8)
    code = (mag // 2 + 2 * (re < 0)).to(torch.uint8)
    code = torch.nn.functional.pad(code, (0, -n % 4)).reshape(-1, 4)
    return code[:, 0] | (code[:, 1] << 2) | (code[:, 2] << 4) | (code[:, 3] << 6)


def _lo(c):
    """The lowest Doppler bin: the window is centred on a multiple of the step."""
    return -(c["bins"] // 2) * c["step"]


def _f_if(c):
    return 0.0 if c["fmt"] == "ci8" else c["fs_khz"] * 250.0


def _search_input(c, seed):
    rng = random.Random(seed * 1009 + 17)
    prns = sorted(rng.sample(range(1, 33), c["n_prn"]))
    half = max(1.0, (c["bins"] // 2) * c["step"])
    planted = []
    for prn in rng.sample(prns, min(len(prns), 4 if c["strong"] else 8)):
        dbhz = 45.0 if c["strong"] else rng.uniform(28.0, 40.0)
        planted.append((prn, rng.randrange(c["fs_khz"]), rng.uniform(-half, half), dbhz, rng.uniform(0, 6.28),
                        not c["strong"]))
    n = c["fs_khz"] * c["t_coh"] * c["blocks"]
    return prns, n, _record(c["fs_khz"], c["fmt"], n, _f_if(c), planted, seed)


def _track_input(case, seed):
    """Records and channels: [(samples, n, [(prn, carrier, phase, code phase, code rate, spacing)])]."""
    rng = random.Random(seed * 1013 + 29)
    fs_khz, n = case["fs_khz"], case["fs_khz"] * case["epoch_ms"] * case["epochs"]
    f_if = _f_if(case)
    out = []
    for i in range(case["records"]):
        planted, channels = [], []
        for prn in rng.sample(range(1, 33), case["channels"]):
            phase, doppler = rng.randrange(fs_khz), rng.uniform(-5000.0, 5000.0)
            planted.append((prn, phase, doppler, 45.0, rng.uniform(0, 6.28), False))
            channels.append((prn, f_if + doppler, rng.random(), (-phase * CHIP_RATE / (fs_khz * 1000.0)) % 1023.0,
                             CHIP_RATE * (1.0 + doppler / L1_HZ), 0.5))
        out.append((_record(fs_khz, case["fmt"], n, f_if, planted[:6], seed * 64 + i), n, channels))
    return out


# --- the calls ----------------------------------------------------------------------------------

_contexts = {}


def _context(precision, **options):
    """The program's context of a precision and an option set."""
    key = (precision,) + tuple(sorted(options.items()))
    if key not in _contexts:
        ctx = G.Context(0, precision=PRECISION[precision])
        for name, value in options.items():
            if value:
                ctx.set(name, value)
        _contexts[key] = ctx
    return _contexts[key]


def _request(c, seed):
    prns, n, x = _search_input(c, seed)
    grid = torch.empty(len(prns), c["bins"], c["fs_khz"], device="cuda")
    peaks = torch.zeros(len(prns), 48, dtype=torch.uint8, device="cuda")
    lo = _lo(c)
    req = G.make_request(x.data_ptr(), FORMAT[c["fmt"]], n, c["fs_khz"] * 1000.0, _f_if(c), prns, lo,
                         lo + (c["bins"] - 1) * c["step"], c["step"], c["t_coh"], c["blocks"], grid.data_ptr(),
                         peaks.data_ptr())
    return req, {"grid": grid, "found": peaks.view(torch.int32)[:, :4], "power": peaks.view(torch.float32)[:, 4:8]}, x


def prepare(case, seed):
    if case["kind"] == "track":
        ctx, reqs, outs, keep = _context("fp32"), [], [], []
        for x, n, channels in _track_input(case, seed):
            out = torch.zeros(len(channels), case["epochs"], 3, 2, dtype=torch.int64, device="cuda")
            reqs.append(G.make_track_request(x.data_ptr(), FORMAT[case["fmt"]], n, case["fs_khz"] * 1000.0, channels,
                                             0, case["fs_khz"] * case["epoch_ms"], case["epochs"], out.data_ptr()))
            outs.append(out)
            keep.append(x)
        return {"call": ctx.track_device, "args": (reqs,), "out": outs, "keep": keep}
    if case["kind"] == "batch":
        made = [_request(c, seed * 64 + i) for i, c in enumerate(_batch_requests(case))]
        return {"call": _context(case["precision"]).acquire_batch_device, "args": ([m[0] for m in made],),
                "out": {"grids": [m[1]["grid"] for m in made], "found": [m[1]["found"] for m in made]}, "keep": made}
    if case["host"]:
        prns, n, x = _search_input(case, seed)
        lo = _lo(case)
        return {"host": (x.cpu().numpy(), FORMAT[case["fmt"]], case["fs_khz"] * 1000.0, _f_if(case), prns, lo,
                         lo + (case["bins"] - 1) * case["step"], case["step"], case["t_coh"], case["blocks"]), "n": n}
    ctx = _context(case["precision"], code_doppler=case["code_doppler"], doppler_fd=case["doppler_fd"],
                   nav_pairs=case["nav_pairs"])
    req, out, x = _request(case, seed)
    return {"call": ctx.acquire_device, "args": (req,), "out": out, "keep": x}


def run(state):
    if "host" in state:
        grid, peaks = G.gnss_acquire(*state["host"], n=state["n"])
        words = peaks.view(np.int32).reshape(len(peaks), 12)
        return {"grid": grid, "found": words[:, :4], "power": words.view(np.float32)[:, 4:8]}
    state["call"](*state["args"], torch.cuda.current_stream())
    return state["out"]


# --- the same results in 64 bits ----------------------------------------------------------------

def _unpacked(x, fmt, n):
    """The record as int64 (re, im)."""
    if fmt == "ci8":
        v = x.reshape(-1, 2)[:n].to(torch.int64)
        return v[:, 0], v[:, 1]
    if fmt == "i8":
        return x[:n].to(torch.int64), None
    two = torch.stack([(x >> (2 * i)) & 3 for i in range(4)], 1).reshape(-1)[:n].to(torch.int64)
    return torch.tensor([1, 3, -1, -3], device=x.device)[two], None


def _grid64(c, prns, n, x):
    """sum_b |R_b[tau]|^2 in FP64: integer NCO and table (or the exact carrier of doppler_fd), the
    folded blocks correlated with the replica by length-N transforms."""
    N, fs, T, B = c["fs_khz"], c["fs_khz"] * 1000, c["t_coh"], c["blocks"]
    xr, xi = _unpacked(x, c["fmt"], n)
    at = torch.arange(n, device="cuda", dtype=torch.int64)
    k = np.arange(1024)
    cos = torch.from_numpy(np.rint(4096 * np.cos(2 * np.pi * k / 1024)).astype(np.int64)).cuda()
    sin = torch.from_numpy(np.rint(4096 * np.sin(2 * np.pi * k / 1024)).astype(np.int64)).cuda()
    m = torch.arange(N, device="cuda", dtype=torch.int64) * CHIP_RATE // fs % 1023
    spectra = torch.fft.fft(torch.stack([_chips(p)[m] for p in prns]).to(torch.complex128)).conj()
    grid = torch.zeros(len(prns), c["bins"], N, dtype=torch.float64, device="cuda")
    group = max(2, (1 << 24) // (N * len(prns)) // 2 * 2)  # blocks at a time
    for kd in range(c["bins"]):
        f = _lo(c) + kd * c["step"]
        if c["doppler_fd"]:
            turn = (at % (T * N)).double() * ((_f_if(c) + f) / fs) % 1.0
            y = torch.complex(xr.double(), xi.double() if xi is not None else torch.zeros_like(xr).double())
            y = (y * torch.polar(torch.ones_like(turn), -2 * math.pi * turn)).reshape(B, T, N).sum(1)
        else:
            step = (_f_if(c) + f) * 2.0 ** 32 / fs
            step = int(math.copysign(math.floor(abs(step) + 0.5), step)) & 0xFFFFFFFF
            e = ((at * step) >> 22) & 1023
            cs, sn = cos[e], sin[e]
            re, im = (xr * cs, -xr * sn) if xi is None else (xr * cs + xi * sn, xi * cs - xr * sn)
            y = torch.complex(re.reshape(B, T, N).sum(1).double(), im.reshape(B, T, N).sum(1).double())
        if c["code_doppler"]:
            for b in range(B):
                s = b * T * N * f / L1_HZ
                y[b] = torch.roll(y[b], int(math.copysign(math.floor(abs(s) + 0.5), s)) % N)
        Y = torch.fft.fft(y)
        for b in range(0, B, group):
            R = torch.fft.ifft(Y[None, b:b + group] * spectra[:, None])
            if c["nav_pairs"]:
                p, q = (R[:, 0::2] + R[:, 1::2]).abs(), (R[:, 0::2] - R[:, 1::2]).abs()
                grid[:, kd] += torch.maximum(p, q).square().sum(1)
            else:
                grid[:, kd] += (R.real.square() + R.imag.square()).sum(1)
    return grid if c["doppler_fd"] else grid * 2.0 ** -24


def _power64(c, grid):
    N = c["fs_khz"]
    Q = grid.max(1).values
    peak, tau = Q.max(1)
    d = (torch.arange(N, device="cuda")[None] - tau[:, None]).abs()
    second = torch.where(torch.minimum(d, N - d) > N * 1000 // CHIP_RATE, Q, 0.0).max(1).values
    return torch.stack([peak, second, grid.mean((1, 2)), peak / second], 1)


def exact(case, seed):
    if case["kind"] == "track":
        return None  # whole numbers: they have no error, and stay equal
    if case["kind"] == "batch":
        # the first requests, so that it stays within seconds
        grids = [_grid64(c, *_search_input(c, seed * 64 + i)) if i < 6 else None
                 for i, c in enumerate(_batch_requests(case))]
        return {"grids": grids, "found": [None] * len(grids)}
    grid = _grid64(case, *_search_input(case, seed))
    return {"grid": grid, "found": None, "power": _power64(case, grid)}
