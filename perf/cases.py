"""What this framework is measured on: batched transforms, matched-filter
compressions, SAR frames, the uneven batch and the autofocus gradient, each
through the Python entry points of the package.

Inputs are made on the GPU from the seed: N(0, 1) rows for the plain
transforms (as the 64 x 4096 and the 20,000-transform workloads use), unit
linear-FM point targets in 20 dB noise for everything that is compressed.
FP8 data is scaled by 1/8, which keeps its spectra below the formats'
saturation.
"""
import math

import numpy as np
import torch

from paper_2605_28451_amd import api
from paper_2605_28451_amd.autofocus import AutofocusPlan, entropy_and_grad

STORAGE = {"fp32": "fp32", "fp16": "fp16", "fp16_fp32": "fp16", "fp16_mul_fp32_acc": "fp16",
           "e4m3": "e4m3", "e5m2": "e5m2"}
FLOAT8 = {"e4m3": torch.float8_e4m3fn, "e5m2": torch.float8_e5m2}
MODES = list(STORAGE)


def listed():
    return [
        # the smallest call in use: a forward transform and its BFP inverse of
        # 64 rows, where latency and launches count
        {"name": "roundtrip 64x4096 fp16", "kind": "roundtrip", "n": 4096, "rows": 64, "mode": "fp16"},
        # the throughput batch of the plain FP16 transform
        {"name": "roundtrip 16384x4096 fp16", "kind": "roundtrip", "n": 4096, "rows": 16384, "mode": "fp16"},
        # the longest transform, an odd number of rows
        {"name": "roundtrip 2047x16384 fp16", "kind": "roundtrip", "n": 16384, "rows": 2047, "mode": "fp16"},
        # short transforms, many to a workgroup, with FP32 arithmetic
        {"name": "roundtrip 65521x256 fp16_fp32", "kind": "roundtrip", "n": 256, "rows": 65521,
         "mode": "fp16_fp32"},
        # fused range compression of one coherent interval in pure FP16
        {"name": "compress 2048x4096 fp16", "kind": "compress", "n": 4096, "rows": 2048, "mode": "fp16"},
        # the same in the mode for deeply weighted apertures, a ragged count of pulses
        {"name": "compress 2045x4096 mul_acc", "kind": "compress", "n": 4096, "rows": 2045,
         "mode": "fp16_mul_fp32_acc"},
        # the same with FP8 storage
        {"name": "compress 1999x4096 e4m3", "kind": "compress", "n": 4096, "rows": 1999, "mode": "e4m3"},
        # FP32 echoes as a receiver delivers them, an odd number of pulses:
        # rounded to FP16, range compressed, corner turned
        {"name": "ingest 1531x4096 fp16_fp32", "kind": "ingest", "n": 4096, "rows": 1531, "mode": "fp16_fp32"},
        # a whole image: range compression, corner turn, azimuth compression
        {"name": "frame 4096x4096 fp16", "kind": "frame", "n": 4096, "rows": 4096, "mode": "fp16"},
        # a whole image with range cell migration correction, in FP32
        {"name": "rcmc frame 2048x2048 fp32", "kind": "rcmc", "n": 2048, "rows": 2048, "mode": "fp32"},
        # 20,000 transforms of mixed length and direction in one launch
        {"name": "uneven 20000 fp16", "kind": "uneven", "count": 20000, "layout": 4, "mode": "fp16"},
        # entropy and its phase gradient, forward and backward, of one image
        {"name": "autofocus 4096x4096 fp32", "kind": "autofocus", "n": 4096, "rows": 4096, "mode": "fp32"},
    ]


def _log(rng, low, high):
    return math.exp(rng.uniform(math.log(low), math.log(high)))


def draw(rng):
    kind = rng.choice(["roundtrip", "roundtrip", "compress", "compress", "ingest", "frame", "rcmc", "uneven",
                       "autofocus"])
    if kind == "uneven":
        return {"kind": kind, "count": int(_log(rng, 50, 20000)), "layout": rng.randint(0, 999),
                "mode": rng.choice(MODES[:4])}
    if kind in ("frame", "rcmc"):  # both axes are transformed
        return {"kind": kind, "n": 1 << rng.randint(10, 12), "rows": 1 << rng.randint(9, 12),
                "mode": rng.choice(["fp16", "fp32", "fp16_fp32"])}
    if kind == "autofocus":
        return {"kind": kind, "n": 1 << rng.randint(9, 12), "rows": int(_log(rng, 200, 4096)), "mode": "fp32"}
    n = 1 << rng.randint(*{"roundtrip": (6, 14), "compress": (9, 14), "ingest": (10, 13)}[kind])
    rows = max(1, int(_log(rng, 1 << 18, 1 << 25) / n))
    return {"kind": kind, "n": n, "rows": rows, "mode": rng.choice(MODES if kind != "ingest" else MODES[:4])}


# ------------------------------------------------------------------ inputs --
def _chirp(length, sign):
    """exp(sign i pi 0.8 (u - L/2)^2 / L), the phase reduced in integers."""
    u = np.arange(length, dtype=np.int64) - length // 2
    return np.exp(sign * 2j * np.pi * ((4 * u * u) % (10 * length)) / (10.0 * length))


def _range_replica(n):
    h = np.zeros(n, dtype=np.complex128)
    h[:n // 4] = _chirp(n // 4, +1)
    return h


def _azimuth_replica(n):
    a = n // 8
    g = np.zeros(n, dtype=np.complex128)
    g[(np.arange(a) - a // 2) % n] = _chirp(a, -1)
    return g


def _gen(seed):
    return torch.Generator(device="cuda").manual_seed(seed)


def _noise(shape, g, snr_db=20.0):
    return torch.randn(tuple(shape) + (2,), generator=g, device="cuda").mul_(
        math.sqrt(0.5 * 10.0 ** (-snr_db / 10.0)))


def _on_gpu(z):
    return torch.view_as_real(torch.from_numpy(np.asarray(z, dtype=np.complex64)).cuda())


def _echo(rows, n, g, rng, azimuth):
    """FP32 echoes [pulse][range] of a few unit point targets: with `azimuth`
    each lights the pulses of its synthetic aperture, else every pulse."""
    x = _noise((rows, n), g)
    h = _chirp(n // 4, +1)
    a = max(rows // 8, 1)
    for _ in range(9 if azimuth else 5):
        d = int(rng.integers(0, n - n // 4 + 1))
        if azimuth:
            m = int(rng.integers(0, rows - a + 1))
            x[m:m + a, d:d + n // 4] += _on_gpu(np.outer(_chirp(a, -1), h))
        else:
            x[:, d:d + n // 4] += _on_gpu(h)
    return x


def _store(x, fmt):
    """FP32 pairs in a storage format, as a host or a producer stores them."""
    if fmt == "fp32":
        return x
    if fmt == "fp16":
        return x.half()
    return (x / 8).to(FLOAT8[fmt]).view(torch.uint8)


def _layout(case):
    """Lengths and directions: what the program's plan is made for."""
    rng = np.random.default_rng(case["layout"])
    log2n = rng.integers(8, 15, size=case["count"]).astype(np.int32)
    return log2n, rng.integers(0, 2, size=case["count"]).astype(np.uint8)


def _data(case, seed):
    """The data a case computes on, in its storage format."""
    g, rng, kind, fmt = _gen(seed), np.random.default_rng(seed), case["kind"], STORAGE[case["mode"]]
    if kind == "uneven":
        total = int((1 << _layout(case)[0].astype(np.int64)).sum())
        return _store(torch.randn((total, 2), generator=g, device="cuda"), fmt)
    rows, n = case["rows"], case["n"]
    if kind == "roundtrip":
        return _store(torch.randn((rows, n, 2), generator=g, device="cuda"), fmt)
    if kind == "autofocus":  # range compressed, [range][pulse]
        x, hist = _noise((rows, n), g), _on_gpu(_chirp(n // 8, -1))
        for r in rng.integers(0, rows, size=9):
            m = int(rng.integers(0, n - n // 8 + 1))
            x[int(r), m:m + n // 8] += hist
        x = torch.view_as_real(torch.view_as_complex(x) * torch.exp(1j * _phase(case, seed)))
        return _store(x, fmt)
    return _store(_echo(rows, n, g, rng, kind != "compress"), "fp32" if kind == "ingest" else fmt)


def _phase(case, seed):
    """A quadratic phase error across the aperture plus pulse-to-pulse noise."""
    n = case["n"]
    m = (torch.arange(n, device="cuda", dtype=torch.float32) - n // 2) / (n // 16)
    return math.pi * m * m + 0.3 * torch.randn(n, generator=_gen(seed + 1000003), device="cuda")


def _shift(case):
    """Range shift per Doppler bin that undoes a parabolic migration."""
    f = torch.fft.fftfreq(case["rows"], device="cuda", dtype=torch.float32)
    return (40.0 * f * f).contiguous()


def prepare(case, seed):
    s = {"kind": case["kind"], "mode": case["mode"], "x": _data(case, seed)}
    if case["kind"] == "uneven":
        s["plan"] = api.UnevenPlan(*_layout(case), case["mode"])
        return s
    n, rows, mode = case["n"], case["rows"], case["mode"]
    if case["kind"] == "autofocus":
        s["plan"] = AutofocusPlan(n, rows, mode)
        s["filter"] = api.filter_tensor(_azimuth_replica(n), n, mode)
        s["phase"] = -0.5 * _phase(case, seed)
        return s
    s["plan"] = api.FFTPlan(n, rows, mode)
    if case["kind"] == "roundtrip":
        return s
    s["filter"] = api.filter_tensor(_range_replica(n), n, mode)
    if case["kind"] in ("frame", "rcmc"):
        s["azimuth"] = api.FFTPlan(rows, n, mode)
        s["azimuth_filter"] = api.filter_tensor(_azimuth_replica(rows), rows, mode)
        s["shift"] = _shift(case)
    return s


def run(s):
    kind, plan, fmt = s["kind"], s["plan"], STORAGE[s["mode"]]
    if kind == "uneven":
        return plan.execute(s["x"])
    if kind == "autofocus":
        entropy, grad, image = entropy_and_grad(plan, s["x"], s["filter"], s["phase"])
        return {"entropy": entropy.float(), "grad": grad, "image": image}
    if kind == "roundtrip":
        spectrum = plan.forward(s["x"])
        out = [spectrum, plan.inverse_bfp(spectrum)]
    elif kind == "compress":
        out = [plan.range_compress(s["x"], s["filter"])]
    elif kind == "ingest":
        x = s["x"] if fmt == "fp32" else api.convert(s["x"], "fp32", fmt)
        out = [api.corner_turn(plan.range_compress(x, s["filter"]), fmt)]
    elif kind == "frame":
        turned = api.corner_turn(plan.range_compress(s["x"], s["filter"]), fmt)
        out = [s["azimuth"].azimuth_compress(turned, s["azimuth_filter"])]
    else:  # migration is corrected between the azimuth transform and its inverse
        doppler = s["azimuth"].forward(api.corner_turn(s["x"], fmt))
        rc = plan.range_compress_rcmc(api.corner_turn(doppler, fmt), s["filter"], s["shift"])
        out = [s["azimuth"].inverse_bfp(api.corner_turn(rc, fmt), s["azimuth_filter"])]
    return [t.view(FLOAT8[fmt]) for t in out] if fmt in FLOAT8 else out


def work(case):
    if case["kind"] == "uneven":
        elements, per = case["count"] * (1 << 15) * 127 / 128 / 7, 8 if case["mode"] == "fp32" else 4
        return {"bytes": 2 * per * elements, "flops": 5 * 13.02 * elements}
    n, rows, b = case["n"], case["rows"], {"fp32": 8, "fp16": 4}.get(STORAGE[case["mode"]], 2)
    across, along, e = 5 * math.log2(n), 5 * math.log2(rows), n * rows
    if case["kind"] == "roundtrip":  # both outputs are written, the spectrum once
        return {"bytes": 3 * b * e, "flops": 2 * across * e}
    if case["kind"] == "compress":
        return {"bytes": 2 * b * e, "flops": 2 * across * e}
    if case["kind"] == "ingest":
        return {"bytes": (8 + b) * e, "flops": 2 * across * e}
    if case["kind"] == "autofocus":  # FP32 in, FP32 image out
        return {"bytes": 2 * b * e, "flops": 4 * across * e}
    return {"bytes": 2 * b * e, "flops": 2 * (across + along) * e}


# ------------------------------------------------- the same in 64 bits --
def _complex(t, fmt):
    if fmt in FLOAT8:
        t = t.view(FLOAT8[fmt]).float()
    return torch.view_as_complex(t.cpu().double().contiguous())


def _filter(replica, mode):
    """The matched filter as the plan stores it (FP32 beside FP8 data)."""
    h = np.fft.fft(replica)
    h = np.conj(h) / np.abs(h).max()
    low = np.float16 if STORAGE[mode] == "fp16" else np.float32
    return torch.complex(torch.from_numpy(h.real.astype(low)).double(), torch.from_numpy(h.imag.astype(low)).double())


def _pairs(z):
    return torch.view_as_real(z.resolve_conj().contiguous())


def exact(case, seed):
    kind, mode = case["kind"], case["mode"]
    fmt = STORAGE[mode]
    x = _complex(_data(case, seed), "fp32" if kind == "ingest" else fmt)
    fft, ifft = torch.fft.fft, torch.fft.ifft
    if kind == "uneven":
        log2n, inverse = _layout(case)
        sizes = 1 << log2n.astype(np.int64)
        starts = np.cumsum(sizes) - sizes
        out = torch.empty_like(x)
        for k in range(8, 15):
            for inv in (0, 1):
                at = starts[(log2n == k) & (inverse == inv)]
                if len(at):
                    rows = torch.stack([x[a:a + (1 << k)] for a in at.tolist()])
                    for a, row in zip(at.tolist(), ifft(rows) if inv else fft(rows)):
                        out[a:a + (1 << k)] = row
        return _pairs(out)
    n, rows = case["n"], case["rows"]
    if kind == "roundtrip":
        return [_pairs(fft(x)), _pairs(x)]
    if kind == "autofocus":
        h = _filter(_azimuth_replica(n), mode)
        phase = -0.5 * _phase(case, seed)
        z = x * torch.exp(1j * phase.cpu().double())
        image = ifft(fft(z) * h)
        power = image.real ** 2 + image.imag ** 2
        total = power.sum()
        log_p = torch.log(power / total)
        entropy = -(power / total * log_p).sum()
        g = ifft(fft((-2.0 / total) * (log_p + entropy) * image) * h.conj())
        return {"entropy": entropy, "grad": (g * z.conj()).imag.sum(0), "image": _pairs(image)}
    h = _filter(_range_replica(n), mode)
    if kind == "compress":
        return [_pairs(ifft(fft(x) * h))]
    if kind == "ingest":
        return [_pairs(ifft(fft(x) * h).T)]
    ha = _filter(_azimuth_replica(rows), mode)
    if kind == "frame":
        return [_pairs(ifft(fft(ifft(fft(x) * h).T) * ha))]
    doppler = fft(x, dim=0)
    ramp = torch.exp(2j * math.pi * torch.fft.fftfreq(n, dtype=torch.float64) * _shift(case).cpu().double()[:, None])
    return [_pairs(ifft(ifft(fft(doppler) * h * ramp).T * ha))]
