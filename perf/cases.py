"""The work that users of the correction have it do, as timed cases.

Every case goes through the public torch entry points of ``paper_2601_01596_amd.ffcz``:
``correct``, ``correct_batched``, ``FFCzCorrect`` (forward and backward), ``encode`` and ``decode``,
``power_spectrum_bounds`` and ``correct_bounds``, ``huffman_compress`` and ``huffman_decompress``.
Inputs are drawn like the package's own workloads (``workloads.py``: Gaussian random fields,
lognormal densities, EEG-like signals, diffraction-like counts, quantised with bin 2E), on the GPU
where the fields are large.

The statistics of a correction (violation counts, rounds) are diagnostics that sit on rounding for
FP32 fields; the outputs compared are the corrected fields, gradients, bound arrays, edit streams
and statuses.
"""

import math

import numpy as np
import torch

from paper_2601_01596_amd import ffcz as F

DEV = "cuda"
DTYPES = {"f32": torch.float32, "f64": torch.float64}


# ------------------------------------------------------------------------------- the cases

def listed():
    return [
        # one sensor channel, as an online pipeline corrects it: a short signal of a length that is
        # no power of two; launches and latency count
        {"name": "signal_6007_f32", "kind": "signal", "n": 6007, "dtype": "f32", "r": 1e-3, "q": 90.0},
        # a small FP64 simulation box (the parity configuration, 64^3)
        {"name": "grf_64x64x64_f64", "kind": "field", "field": "grf", "alpha": 2.0, "shape": "64x64x64",
         "dtype": "f64", "r": 1e-3, "q": 90.0, "cap": 200},
        # a slab of a decomposed domain: extents that differ on every axis
        {"name": "grf_64x256x128_f32", "kind": "field", "field": "grf", "alpha": 5.0 / 3.0, "shape": "64x256x128",
         "dtype": "f32", "r": 1e-4, "q": 99.0, "cap": 500},
        # the benchmark field (512^3 lognormal density) in both precisions
        {"name": "lognormal_512x512x512_f32", "kind": "field", "field": "lognormal", "alpha": 2.5,
         "shape": "512x512x512", "dtype": "f32", "r": 1e-4, "q": 95.0, "cap": 500},
        {"name": "lognormal_512x512x512_f64", "kind": "field", "field": "lognormal", "alpha": 2.5,
         "shape": "512x512x512", "dtype": "f64", "r": 1e-4, "q": 95.0, "cap": 500},
        # one diffraction frame as it leaves the detector
        {"name": "diffraction_2048x2048_f32", "kind": "field", "field": "diffraction", "alpha": 0.0,
         "shape": "2048x2048", "dtype": "f32", "r": 1e-3, "q": 90.0, "cap": 200},
        # a recording session: many channels of uneven lengths in one call
        {"name": "batch_eeg128_f32", "kind": "batch", "signals": 128, "fields": 0, "edge": 0, "lo": 4096, "hi": 262144,
         "dtype": "f32", "r": 1e-3, "q": 90.0},
        # channels and detector frames together
        {"name": "batch_eeg64_frames16x2048_f32", "kind": "batch", "signals": 64, "fields": 16, "edge": 2048,
         "lo": 4096, "hi": 262144, "dtype": "f32", "r": 1e-3, "q": 90.0},
        # differentiable correction: 50 fixed rounds forward, masks recorded, and the adjoint
        {"name": "grad_256x256x256_f32", "kind": "grad", "field": "grf", "alpha": 2.0, "shape": "256x256x256",
         "dtype": "f32", "r": 1e-3, "q": 90.0, "rounds": 50},
        # the edits as a compressor stores them, and their application by a reader
        {"name": "codec_256x256x256_f32", "kind": "codec", "field": "lognormal", "alpha": 2.5,
         "shape": "256x256x256", "dtype": "f32", "r": 1e-4, "q": 95.0, "cap": 500},
        # relative power-spectrum bounds: the bound array, then the correction against it
        {"name": "spectrum_256x256x256_f32", "kind": "spectrum", "field": "lognormal", "alpha": 2.5,
         "shape": "256x256x256", "dtype": "f32", "r": 1e-4, "rho": 1e-3, "disk": False, "cap": 500},
        # lossless coding of a flag stream and a code stream, and back
        {"name": "huffman_16M_flags_1M_codes", "kind": "huffman", "flags": 16777216, "codes": 1048576,
         "density": 0.02, "spread": 300.0},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _shape(rng, dtype, lg_lo, lg_hi, dims):
    """Power-of-two extents (the multidimensional passes take these) of 2^lg_lo to 2^lg_hi points."""
    most = 11 if dtype == "f32" else 10
    while True:
        nd = rng.choice(dims)
        e = [rng.randint(3, most) for _ in range(nd - 1)] + [rng.randint(4, 12)]
        if lg_lo <= sum(e) <= lg_hi:
            return "x".join(str(1 << k) for k in e)


def draw(rng):
    kind = rng.choice(["signal", "field", "field", "field", "batch", "grad", "codec", "spectrum", "huffman"])
    dtype = rng.choice(["f32", "f32", "f64"])
    r = math.exp(rng.uniform(math.log(1e-4), math.log(1e-3)))
    q = rng.uniform(90.0, 99.0)
    if kind == "signal":
        return {"kind": kind, "n": _log_int(rng, 500, 200000), "dtype": dtype, "r": r, "q": q}
    if kind == "field":
        field = rng.choice(["grf", "lognormal"])
        return {"kind": kind, "field": field, "alpha": rng.uniform(1.6, 2.5),
                "shape": _shape(rng, dtype, 13, 26, [2, 3, 3]), "dtype": dtype, "r": r, "q": q, "cap": 500}
    if kind == "batch":
        fields = rng.randint(0, 8)
        return {"kind": kind, "signals": rng.randint(8, 96), "fields": fields,
                "edge": rng.choice([512, 1024, 2048]) if fields else 0, "lo": 4096, "hi": 262144, "dtype": "f32",
                "r": r, "q": q}
    if kind == "grad":
        return {"kind": kind, "field": "grf", "alpha": rng.uniform(1.6, 2.5), "shape": _shape(rng, "f32", 15, 24, [3]),
                "dtype": "f32", "r": r, "q": q, "rounds": rng.randint(5, 50)}
    if kind == "codec":
        return {"kind": kind, "field": rng.choice(["grf", "lognormal"]), "alpha": rng.uniform(1.6, 2.5),
                "shape": _shape(rng, dtype, 15, 24, [2, 3]), "dtype": dtype, "r": r, "q": q, "cap": 500}
    if kind == "spectrum":
        return {"kind": kind, "field": "lognormal", "alpha": rng.uniform(1.6, 2.5),
                "shape": _shape(rng, dtype, 15, 24, [2, 3]), "dtype": dtype, "r": r, "rho": 1e-3,
                "disk": rng.random() < 0.5, "cap": 500}
    return {"kind": kind, "flags": _log_int(rng, 30000, 16777216), "codes": _log_int(rng, 3000, 1048576),
            "density": rng.uniform(0.005, 0.2), "spread": rng.uniform(10.0, 2000.0)}


# ------------------------------------------------------------------------------- inputs

def _dims(case):
    return tuple(int(v) for v in case["shape"].split("x"))


def _generator(seed, device=DEV):
    g = torch.Generator(device=device)
    g.manual_seed(int(seed) % (1 << 62))
    return g


def _kmag(shape):
    k2 = 0.0
    for i, n in enumerate(shape):
        if i == len(shape) - 1:
            f = torch.arange(n // 2 + 1, dtype=torch.float64, device=DEV)
        else:
            f = torch.fft.fftfreq(n, 1.0 / n, dtype=torch.float64, device=DEV)
        k2 = k2 + (f * f).reshape([-1 if j == i else 1 for j in range(len(shape))])
    return k2.sqrt()


def _field(case, seed, shape=None):
    """The original field, FP64: a Gaussian random field of spectrum k^-alpha, its exponential (a
    density), or the Poisson counts of a far-field intensity."""
    shape = shape or _dims(case)
    g = _generator(seed)
    if case.get("field", "diffraction") == "diffraction":
        n = shape[0]
        rad = n / 16.0 + (n / 4.0 - n / 16.0) * float(torch.rand((), generator=g, device=DEV, dtype=torch.float64))
        c = torch.arange(n, device=DEV, dtype=torch.float64) - n / 2
        disk = (c[:, None] ** 2 + c[None, :] ** 2) <= rad * rad
        amp = torch.rand(shape, generator=g, device=DEV, dtype=torch.float64)
        ph = 2.0 * math.pi * torch.rand(shape, generator=g, device=DEV, dtype=torch.float64)
        obj = torch.where(disk, torch.polar(amp, ph), torch.zeros((), dtype=torch.complex128, device=DEV))
        inten = torch.fft.fftshift(torch.fft.fft2(obj)).abs().square()
        return torch.poisson(inten * (1e4 / inten.max()), generator=g)
    w = torch.fft.rfftn(torch.randn(shape, generator=g, device=DEV, dtype=torch.float64))
    k = _kmag(shape)
    w *= torch.where(k > 0, k.clamp_min(1.0).pow(-case["alpha"] / 2.0), torch.zeros_like(k))
    f = torch.fft.irfftn(w, s=shape)
    f = (f - f.mean()) / f.std()
    return f.exp() if case["field"] == "lognormal" else f


def _eeg(n, rng):
    """Pink noise of unit deviation plus one to three tones of the alpha band at 256 Hz."""
    w = np.fft.rfft(rng.standard_normal(n))
    f = np.arange(w.size, dtype=np.float64)
    p = np.fft.irfft(w * np.where(f > 0, 1.0 / np.sqrt(np.maximum(f, 1.0)), 0.0), n=n)
    p /= p.std()
    t = np.arange(n) / 256.0
    for _ in range(int(rng.integers(1, 4))):
        p += rng.uniform(0.5, 2.0) * np.sin(2.0 * math.pi * (rng.uniform(8.0, 13.0) * t + rng.uniform()))
    return p


def _quantized(x, r):
    """Bound E = r x range and the base reconstruction: a uniform quantiser of bin 2E."""
    x64 = x.double()
    E = r * float(x64.max() - x64.min())
    return E, (2.0 * E * torch.round(x64 / (2.0 * E))).to(x.dtype)


def _spectral_bound(m, q):
    """Halfway between the q-th percentile of the values m and the next larger one."""
    m = m.reshape(-1)
    k = min(m.numel() - 1, max(1, int(math.ceil(q / 100.0 * m.numel()))))
    a = float(torch.kthvalue(m, k).values)
    above = m[m > a]
    return 0.5 * (a + float(above.min())) if above.numel() else a


def _problem(case, seed, shape=None):
    """x, x_hat, E and Delta of one field."""
    x = _field(case, seed, shape).to(DTYPES[case["dtype"]])
    E, xb = _quantized(x, case["r"])
    if "q" not in case:
        return x, xb, E, 0.0
    d = torch.fft.rfftn(xb.double() - x.double())
    return x, xb, E, _spectral_bound(torch.maximum(d.real.abs(), d.imag.abs()), case["q"])


def _signal_problem(case, n, rng):
    """x, x_hat (host), E and Delta of one signal."""
    x = torch.from_numpy(_eeg(n, rng)).to(DTYPES[case["dtype"]])
    E, xb = _quantized(x, case["r"])
    d = np.fft.rfft((xb.double() - x.double()).numpy())
    return x, xb, E, _spectral_bound(torch.from_numpy(np.maximum(np.abs(d.real), np.abs(d.imag))), case["q"])


def _members(case, seed):
    """(x, x_hat, E, Delta) of every member of a batch; signals on the host."""
    rng = np.random.default_rng(seed)
    out = []
    for _ in range(case["signals"]):
        n = int(np.rint(math.exp(rng.uniform(math.log(case["lo"]), math.log(case["hi"])))))
        out.append(_signal_problem(case, n, rng))
    for j in range(case["fields"]):
        out.append(_problem(case, seed * 1000 + 17 + j, (case["edge"], case["edge"])))
    return out


def _symbols(case, seed):
    g = _generator(seed)
    bits = torch.rand((case["flags"], 8), generator=g, device=DEV) < case["density"]
    flags = (bits.to(torch.int32) << torch.arange(8, device=DEV, dtype=torch.int32)).sum(1).to(torch.uint8)
    u = torch.rand(case["codes"], generator=g, device=DEV, dtype=torch.float64) - 0.5
    codes = torch.round(-case["spread"] * u.sign() * torch.log1p(-2.0 * u.abs().clamp(max=0.4999999)))
    return flags, codes.to(torch.int32)


def _side_by_side(fields, case, dtype=None):
    """A zeroed buffer of one size for every seed, and a view of it per member (at whole 256 elements)."""
    room = case["signals"] * (case["hi"] + 256) + case["fields"] * case["edge"] ** 2
    buf = torch.zeros(room, dtype=dtype or fields[0].dtype, device=DEV)
    views, at = [], 0
    for x in fields:
        views.append(buf[at:at + x.numel()].view(x.shape))
        at += (x.numel() + 255) // 256 * 256
    return buf, views


def prepare(case, seed):
    kind = case["kind"]
    st = {"kind": kind, "case": case}
    if kind == "huffman":
        st["flags"], st["codes"] = _symbols(case, seed)
        # where the streams go: one buffer per stream, larger than any stream of these sizes
        st["out"] = [torch.zeros(2 * b + (1 << 20), dtype=torch.uint8, device=DEV)
                     for b in (case["flags"], 4 * case["codes"])]
        return st
    if kind == "signal":
        x, xb, st["E"], st["D"] = _signal_problem(case, case["n"], np.random.default_rng(seed))
        st["x"], st["xb"], st["cap"] = x.to(DEV), xb.to(DEV), 200
        return st
    if kind == "batch":
        st["members"] = [(x.to(DEV), xb.to(DEV), E, D) for x, xb, E, D in _members(case, seed)]
        st["ws"] = F.batched_workspace(st["members"], 200)
        # the outputs side by side in one buffer
        st["y"], st["outs"] = _side_by_side([m[0] for m in st["members"]], case)
        return st
    st["x"], st["xb"], st["E"], st["D"] = _problem(case, seed)
    st["cap"] = case.get("cap", 0)
    code = F.F32 if case["dtype"] == "f32" else F.F64
    if kind == "field":
        st["ws"] = F.workspace(code, st["x"].shape, st["cap"], st["x"].device)
    elif kind == "grad":
        st["g"] = torch.randn(_dims(case), generator=_generator(seed + 1), device=DEV, dtype=st["x"].dtype)
    elif kind == "codec":
        n = F.ffcz_encode_workspace_bytes(code, _dims(case), st["cap"])
        st["ws"] = torch.empty(n, dtype=torch.uint8, device=DEV)
        # where the code streams go: their longest forms
        st["out"] = [torch.zeros(k, dtype=torch.int32, device=DEV) for k in F.edit_coords(_dims(case))]
    return st


def _store(buf, stream):
    """A stream into its place, whose size does not depend on the data; its length."""
    buf[:stream.numel()].copy_(stream)
    return stream.numel()


# ------------------------------------------------------------------------------- one pass

def run(state):
    s, kind = state, state["kind"]
    if kind in ("signal", "field"):
        r = F.correct(s["x"], s["xb"], s["E"], s["D"], s["cap"], ws=s.get("ws"))
        return {"y": r.y, "status": r.status}
    if kind == "batch":
        _, status, _ = F.correct_batched(s["members"], 200, ws=s["ws"], outs=s["outs"])
        return {"y": s["y"], "status": status}
    if kind == "grad":
        xb = s["xb"].detach().requires_grad_(True)
        y = F.FFCzCorrect.apply(xb, s["x"], s["E"], s["D"], s["case"]["rounds"])
        (g,) = torch.autograd.grad(y, xb, s["g"])
        return {"y": y.detach(), "grad": g}
    if kind == "codec":
        e = F.encode(s["x"], s["xb"], s["E"], s["D"], s["cap"], ws=s["ws"])
        y = F.decode(s["xb"], e, ws=s["ws"])
        sn, fn = _store(s["out"][0], e.spat_codes), _store(s["out"][1], e.freq_codes)
        return {"spat_flags": e.spat_flags, "spat_codes": s["out"][0], "spat_count": sn, "freq_flags": e.freq_flags,
                "freq_codes": s["out"][1], "freq_count": fn, "status": e.status, "y": y}
    if kind == "spectrum":
        c = s["case"]
        D = F.power_spectrum_bounds(s["x"], c["rho"], disk=c["disk"])
        r = F.correct_bounds(s["x"], s["xb"], s["cap"], eps_s=s["E"], D_re=D, D_im=D, disk=c["disk"])
        return {"bound": D, "y": r.y, "status": r.status}
    flags, codes = s["flags"], s["codes"]
    fs, fz = F.huffman_compress(flags)
    cs, cz = F.huffman_compress(codes)
    fn, cn = _store(s["out"][0], fs), _store(s["out"][1], cs)
    return {"flag_stream": s["out"][0], "flag_bytes": fn, "code_stream": s["out"][1], "code_bytes": cn,
            "flags": F.huffman_decompress(fs, flags.numel(), torch.uint8, int(fz.nalpha)),
            "codes": F.huffman_decompress(cs, codes.numel(), torch.int32, int(cz.nalpha))}


def work(case):
    """Inputs read once, outputs written once; transforms of the first check, one round and the
    closing verification (2.5 N log2 N operations each)."""
    kind = case["kind"]
    if kind == "huffman":
        n = case["flags"] + 4 * case["codes"]
        return {"bytes": 2 * n + 2 * 0.6 * n, "flops": 0}
    s = 4 if case["dtype"] == "f32" else 8

    def fft(n):
        return 2.5 * n * math.log2(n)

    if kind == "signal":
        return {"bytes": 3 * s * case["n"], "flops": 3 * fft(case["n"])}
    if kind == "batch":
        mean = (case["hi"] - case["lo"]) / math.log(case["hi"] / case["lo"])
        n1, n2 = case["signals"] * mean, case["fields"] * case["edge"] ** 2
        return {"bytes": 3 * s * (n1 + n2), "flops": 3 * (n1 * 2.5 * math.log2(mean) + case["fields"]
                                                          * fft(max(2, case["edge"] ** 2)))}
    n = math.prod(_dims(case))
    if kind == "grad":
        # the fields, the gradients, and a clip mask of about two bits a point and round, both ways
        return {"bytes": 5 * s * n + 2 * case["rounds"] * n * 3 / 8, "flops": 4 * case["rounds"] * fft(n)}
    if kind == "codec":
        # x and x_hat, the flags written and read, x_hat again and y
        return {"bytes": 4 * s * n + 2 * 2 * n / 8, "flops": 4 * fft(n)}
    if kind == "spectrum":
        return {"bytes": 3 * s * n + s * n / 2, "flops": 4 * fft(n)}
    return {"bytes": 3 * s * n, "flops": 3 * fft(n)}


# ------------------------------------------------------------------------------- in 64 bits

def _ulp2_mean(x):
    """Mean squared spacing of the FP32 grid at the values of x."""
    a = x.abs()
    return float((torch.nextafter(a, torch.full_like(a, math.inf)).double() - a.double()).square().mean())


def _margin(x, D, disk=False):
    """The relative shrink: 2^-16, or for FP32 outputs eight deviations of their rounding."""
    if x.dtype == torch.float64:
        return 2.0 ** -16
    m = 8.0 * math.sqrt(_ulp2_mean(x) / 12.0) * math.sqrt(x.numel() / 2.0) / D if D > 0 else 0.5
    return min(0.5, max(2.0 ** -16, m * (math.sqrt(2.0) if disk else 1.0)))


def _fft(e):
    if e.dim() == 1 and not e.is_cuda:
        return torch.from_numpy(np.fft.rfft(e.numpy()))
    return torch.fft.rfftn(e)


def _ifft(d, shape):
    if len(shape) == 1 and not d.is_cuda:
        return torch.from_numpy(np.fft.irfft(d.numpy(), n=shape[0]))
    return torch.fft.irfftn(d, s=shape)


def _clip_box(d, br, bi):
    return torch.complex(torch.clamp(d.real, -br, br), torch.clamp(d.imag, -bi, bi))


def _tensor(v, like):
    return torch.as_tensor(v, dtype=torch.float64, device=like.device)


def _project(x, xb, Ep, Dc, Dp, cap, fixed=False, disk=False, edits=False, masks=None):
    """The alternating projection in 64 bits: the final error, and the summed edits."""
    x64 = x.double()
    e0 = xb.double() - x64
    Ep, Dc, Dp = _tensor(Ep, x64), _tensor(Dc, x64), _tensor(Dp, x64)
    eps = torch.clamp(e0, -Ep, Ep)
    if masks is not None:
        masks.append(e0.abs() <= Ep)
    s = eps - e0 if edits else None
    f = 0.0
    k = 0
    while True:
        d = _fft(eps)
        bad = d.abs() > Dc if disk else (d.real.abs() > Dc) | (d.imag.abs() > Dc)
        if k == cap or (not fixed and not bool(bad.any())):
            break
        if disk:
            m = d.abs()
            c = torch.where(m > Dp, d * (Dp / m.clamp_min(1e-300)), d)
        else:
            c = _clip_box(d, Dp, Dp)
        if edits:
            f = f + (c - d)
        if masks is not None:
            masks.append((d.real.abs() <= Dp, d.imag.abs() <= Dp))
        e = _ifft(c, x.shape)
        eps = torch.clamp(e, -Ep, Ep)
        if masks is not None:
            masks.append(e.abs() <= Ep)
        if edits:
            s = s + (eps - e)
        k += 1
    return (eps, s, f) if edits else eps


def _scalar(x, xb, E, D, cap, fixed=False, masks=None):
    mu = _margin(x, D)
    rho = 0.0 if x.dtype == torch.float64 else mu
    return x.double() + _project(x, xb, E * (1 - mu), D * (1 - rho), D * (1 - rho - mu), cap, fixed, masks=masks)


def _shell_bounds(x, rho, disk):
    X = torch.fft.rfftn(x.double()).abs()
    b = _kmag(x.shape).round().long().reshape(-1)
    w = torch.full_like(X, 2.0)
    w[..., 0] = 1.0
    w[..., -1] = 1.0
    nb = int(b.max()) + 1

    def total(v):
        return torch.zeros(nb, dtype=torch.float64, device=DEV).index_add_(0, b, v.reshape(-1))

    P, S, W = total(w * X * X), total(w * X), total(w)
    c = 1.0 if disk else 2.0
    den = torch.sqrt(c * S * S + c * W * rho * P) + math.sqrt(c) * S
    return torch.where(den > 0, rho * P / den, torch.zeros_like(den))[b].reshape(X.shape)


def exact(case, seed):
    kind = case["kind"]
    if kind == "huffman":
        return None  # bytes and whole numbers
    if kind == "signal":
        x, xb, E, D = _signal_problem(case, case["n"], np.random.default_rng(seed))
        return {"y": _scalar(x, xb, E, D, 200)}
    if kind == "batch":
        ms = _members(case, seed)
        buf, views = _side_by_side([m[0] for m in ms], case, torch.float64)
        for v, (x, xb, E, D) in zip(views, ms):
            v.copy_(_scalar(x, xb, E, D, 200))
        return {"y": buf}
    x, xb, E, D = _problem(case, seed)
    if kind == "field":
        return {"y": _scalar(x, xb, E, D, case["cap"])}
    if kind == "grad":
        masks = []
        y = _scalar(x, xb, E, D, case["rounds"], fixed=True, masks=masks)
        g = torch.randn(_dims(case), generator=_generator(seed + 1), device=DEV, dtype=x.dtype).double()
        g = torch.where(masks.pop(), g, 0.0)
        while masks:
            mr, mi = masks.pop()
            d = torch.fft.rfftn(g)
            g = torch.fft.irfftn(torch.complex(torch.where(mr, d.real, 0.0), torch.where(mi, d.imag, 0.0)), s=g.shape)
            g = torch.where(masks.pop(), g, 0.0)
        return {"y": y, "grad": g}
    if kind == "codec":
        # the encoder's shrinks and its 16-bit steps; the streams themselves are whole numbers
        q = 4.0 * 2.0 ** -16
        top = (x.abs().max().double() + E).to(x.dtype)
        u = float(torch.nextafter(top, torch.full_like(top, math.inf)).double() - top.double())
        mf = min(0.25, max(_margin(x, D), q))
        ms = min(0.5, q + u / E)
        _, s, f = _project(x, xb, E * (1 - ms), D * (1 - mf), D * (1 - 2 * mf), case["cap"], edits=True)
        y = xb.double() + s if isinstance(f, float) else xb.double() + s + torch.fft.irfftn(f, s=x.shape)
        return {"y": y}
    B = _shell_bounds(x, case["rho"], case["disk"])
    mu = _margin(x, float(B.min()), case["disk"])
    rho = 0.0 if x.dtype == torch.float64 else mu
    eps = _project(x, xb, E * (1 - mu), B * (1 - rho), B * (1 - rho - mu), case["cap"], disk=case["disk"])
    return {"bound": B, "y": x.double() + eps}
