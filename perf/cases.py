"""What a user of the spectrometer library has it do: the workloads by which its speed is followed.

A case is a dict of plain values.  ``listed()`` names the fixed ones, ``draw(rng)`` gives another of the same
ranges; ``prepare(case, seed)`` makes on the GPU what a program holds before the call (packed sampler codes, a
bound plan, calibration tables, output buffers), ``run(state)`` is one pass through the public entry points,
``work(case)`` counts the bytes and operations the pass cannot do without, and ``exact(case, seed)`` gives its
results in 64 bits with plain torch.

The kinds of case:

* ``spectra``: one integration of one stream set, reset -> accumulate_stokes (packed codes to calibrated
  I, Q, U, V), as a streaming spectrometer calls it once per output period;
* ``power``: the same with level histograms counted (total-power observing) and read out;
* ``train``: one step of calibration by gradient: differentiable Stokes of one integration and the gradients of
  gains, leakage and window taps;
* ``batch``: several stream sets of uneven frame lengths and formats in one plan;
* ``reduce``: the reductions of a series of integrated spectra (smoothed bandpass, bandpass variation, channel
  averages with flags, band moments, spectral Allan variance);
* ``tav``: time-based Allan variances of every channel of a run of integrations.
"""
from __future__ import annotations

import math

import torch

import paper_1412_1256_amd as ps
from paper_1412_1256_amd import autograd

PAIRS = {2: ((0, 1),), 4: ((0, 2), (1, 3))}  # X, Y; or Table 1's X0, X1, Y0, Y1


def _spectra(name, log2n, frames, bits, streams=2, window="rect", hop=1, precision="fp32", cal=False,
             feed="linear"):
    """frames: frame lengths of data in the buffer; hop: frames start every fft_len / hop samples."""
    return dict(name=name, kind="spectra", log2n=log2n, frames=frames, bits=bits, streams=streams, window=window,
                hop=hop, precision=precision, cal=cal, feed=feed)


def listed():
    return [
        # the smallest integration a user runs (the smoke check's size): launches and latency count
        _spectra("tiny-2^10", 10, 64, 2, window="hann"),
        # coarse channels, many short frames, gains and leakage applied
        _spectra("short-2^12", 12, 4096, 8, cal=True),
        # one second of one 16-Msps pair at the paper's 61-Hz channels
        _spectra("paper-2^18", 18, 61, 8),
        # Table 1's 8 MHz mode: four 4-bit IFs, two pairs, calibrated
        _spectra("mode-8MHz", 18, 61, 4, streams=4, cal=True),
        # the same second with apodised, half-overlapped frames
        _spectra("overlap-2^18", 18, 61, 8, window="hamming", hop=2),
        # finer channels than the paper's, 2-bit samplers, circular feeds
        _spectra("long-2^20", 20, 32, 2, feed="circular"),
        # ten seconds of four int8 IFs in 16-bit transform passes with compensated sums
        _spectra("precision-2^18", 18, 610, 8, streams=4, precision="fp16"),
        # one second with the level histograms of total-power observing
        dict(name="power-2^18", kind="power", log2n=18, frames=61, bits=8),
        # one step of the learned calibration: forward and backward
        dict(name="train-2^16", kind="train", log2n=16, frames=128, bits=8, taps=64),
        # 16 uneven stream sets in one plan
        dict(name="batch-16", kind="batch", sets=16, lo=12, hi=20, fmin=8, fmax=128, shapes=4),
        # half a minute of 1-s spectra against their smoothed bandpass
        dict(name="reduce-30x131072", kind="reduce", spectra=30, channels=1 << 17, factor=256, knots=128),
        # half an hour of 1-s spectra, every channel, eight lags
        dict(name="tav-1800x131072", kind="tav", points=1800, series=1 << 17, lags="1,2,4,8,16,64,256,512"),
    ]


def _unnamed(case):
    return {k: v for k, v in case.items() if k != "name"}


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["spectra"] * 6 + ["power", "train", "batch", "reduce", "tav", "precision"])
    if kind == "precision":
        log2n = rng.randint(16, 18)
        streams = rng.choice([2, 4])
        frames = max(2, _log_int(rng, 1 << 20, 1 << 26) >> log2n)
        return _unnamed(_spectra("", log2n, frames, 8, streams, window=rng.choice(["rect", "rect", "hann"]),
                             precision=rng.choice(["fp16", "bf16"]), cal=rng.random() < 0.5))
    if kind == "spectra":
        log2n = rng.randint(8, 22)
        streams = rng.choice([2, 2, 4])
        frames = max(2, (_log_int(rng, 1 << 16, 1 << 25) >> log2n) - rng.randint(0, 1))
        return _unnamed(_spectra("", log2n, frames, rng.choice([2, 4, 8]), streams,
                             window=rng.choice(["rect", "rect", "hann", "hamming", "blackman"]),
                             hop=rng.choice([1, 1, 1, 2]), cal=rng.random() < 0.5,
                             feed=rng.choice(["linear", "circular"])))
    if kind == "power":
        log2n = rng.randint(12, 19)
        return dict(kind="power", log2n=log2n, frames=max(2, _log_int(rng, 1 << 18, 1 << 24) >> log2n),
                    bits=rng.choice([2, 4, 8]))
    if kind == "train":
        log2n = rng.randint(12, 18)
        return dict(kind="train", log2n=log2n, frames=max(2, _log_int(rng, 1 << 18, 1 << 23) >> log2n),
                    bits=rng.choice([2, 8]), taps=rng.choice([16, 33, 64]))
    if kind == "batch":
        return dict(kind="batch", sets=rng.randint(3, 16), lo=rng.randint(9, 13), hi=rng.randint(16, 19),
                    fmin=rng.randint(3, 16), fmax=rng.randint(33, 128), shapes=rng.randint(5, 10 ** 6))
    if kind == "reduce":
        channels = 1 << rng.randint(13, 17)
        return dict(kind="reduce", spectra=rng.randint(2, 40), channels=channels,
                    factor=1 << rng.randint(3, 9), knots=rng.choice([64, 96, 128, 200]))
    points = _log_int(rng, 100, 1800)
    lags = sorted({_log_int(rng, 1, min(512, points // 3)) for _ in range(rng.randint(3, 8))})
    return dict(kind="tav", points=points, series=_log_int(rng, 1000, 1 << 17),
                lags=",".join(map(str, lags)))


# ------------------------------------------------------------------------------------------------
# inputs

def _gen(seed):
    return torch.Generator(device="cuda").manual_seed(seed)


def _codes(gen, samples, streams, bits, rho=0.3):
    """Packed codes of pairs of correlated Gaussian streams with a weak common tone, through the samplers'
    quantisers (2-bit thresholds at 0 and 1 sigma, 4-bit steps of sigma / 2, int8 with sigma = 16 LSB)."""
    codes = torch.empty((samples, streams), dtype=torch.uint8, device="cuda")
    step = 1 << 24
    for p in range(streams // 2):
        for t0 in range(0, samples, step):
            n = min(step, samples - t0)
            c = torch.randn(n, device="cuda", generator=gen) * math.sqrt(rho)
            c += 0.05 * torch.sin(torch.arange(n, device="cuda") * (2 * math.pi * 0.1171875))
            for s in PAIRS[streams][p]:
                v = torch.randn(n, device="cuda", generator=gen) * math.sqrt(1 - rho) + c
                if bits == 2:
                    q = (v >= -1).to(torch.uint8) + (v >= 0).to(torch.uint8) + (v >= 1).to(torch.uint8)
                elif bits == 4:
                    q = (torch.floor(v * 2) + 8).clamp(0, 15).to(torch.uint8)
                else:
                    q = torch.round(v * 16).clamp(-128, 127).to(torch.int8).view(torch.uint8)
                codes[t0:t0 + n, s] = q
    flat = codes.view(-1)
    if bits == 8:
        return flat
    per = 8 // bits
    g = flat.view(-1, per)
    out = g[:, 0].clone()
    for i in range(1, per):
        out |= g[:, i] << (i * bits)
    return out


def _complex(gen, shape, sd):
    return sd * torch.view_as_complex(torch.randn((*shape, 2), device="cuda", generator=gen))


def _calibration(gen, pairs, channels):
    """Complex gains near 1 per channel, leakage terms of a few per cent per pair, a parallactic angle."""
    return dict(gain_x=1 + _complex(gen, (pairs, channels), 0.05), gain_y=1 + _complex(gen, (pairs, channels), 0.05),
                dterms=_complex(gen, (pairs, 2), 0.02), psi=0.3)


def _stream_sets(case):
    """(log2 frame length, frames, bits) of each stream set of a batch case."""
    g = torch.Generator().manual_seed(case["shapes"])
    pick = lambda lo, hi: int(torch.randint(lo, hi + 1, (1,), generator=g))
    return [(pick(case["lo"], case["hi"]), pick(case["fmin"], case["fmax"]), (2, 8)[pick(0, 1)])
            for _ in range(case["sets"])]


def _inputs(case, seed):
    gen = _gen(seed)
    kind = case["kind"]
    if kind in ("spectra", "power", "train"):
        n, streams = 1 << case["log2n"], case.get("streams", 2)
        pairs = PAIRS[streams]
        d = dict(packed=_codes(gen, n * case["frames"], streams, case["bits"]))
        if case.get("cal") or kind == "train":
            d["cal"] = _calibration(gen, len(pairs), n // 2)
        if kind == "train":
            d["taps"] = 1 + 0.1 * torch.randn(case["taps"], device="cuda", generator=gen)
            d["upstream"] = torch.randn((len(pairs), 4, n // 2), device="cuda", generator=gen) / n
        return d
    if kind == "batch":
        return dict(packed=[_codes(gen, f << e, 2, b) for e, f, b in _stream_sets(case)])
    if kind == "reduce":
        n, c = case["spectra"], case["channels"]
        k = torch.arange(c, device="cuda") / c
        shape = 1 + 0.2 * torch.sin(40 * k) - 0.3 * (2 * k - 1) ** 8
        gain = 1 + 0.01 * torch.randn(n, device="cuda", generator=gen, dtype=torch.float64)
        noise = torch.randn((n, c), device="cuda", generator=gen)
        hk = (gain[:, None] * shape * (1 + 0.05 * noise)).float()
        h = (shape * (1 + 0.005 * torch.randn(c, device="cuda", generator=gen))).float()
        flags = torch.zeros(c, dtype=torch.uint8, device="cuda")
        flags[c // 2] = 1  # the spurious channel at the band centre
        hk[:, c // 2] *= 1.5
        return dict(h=h, hk=hk, gain=gain, flags=flags)
    x = torch.randn((case["points"], case["series"]), device="cuda", generator=gen)
    x.mul_(0.008).add_(1)
    x *= 1 + 1e-3 * torch.cumsum(torch.randn(case["points"], device="cuda", generator=gen), 0)[:, None] / 30
    return dict(x=x)


# ------------------------------------------------------------------------------------------------
# the measured pass

def _instance(case, **over):
    streams = case.get("streams", 2)
    n = 1 << case["log2n"]
    kw = dict(fft_len=n, bits=case["bits"], n_streams=streams, pairs=PAIRS[streams],
              window=case.get("window", "rect"), hop=n // case.get("hop", 1))
    if case.get("precision", "fp32") != "fp32":
        kw.update(precision=case["precision"], accum="kahan32")
    kw.update(over)
    return ps.Instance(**kw)


def _out(inst):
    return torch.empty((inst.n_pairs, 4, inst.channels), dtype=torch.float32, device="cuda")


def prepare(case, seed):
    d = _inputs(case, seed)
    d["case"] = case
    kind = case["kind"]
    if kind in ("spectra", "power"):
        inst = _instance(case)
        d["plan"], d["out"] = ps.Plan([inst], device="cuda"), _out(inst)
        if kind == "power":
            d["plan"].set_histograms(True)
    elif kind == "train":
        d["plan"] = ps.Plan([_instance(case, window="taps", n_taps=case["taps"])], device="cuda")
        cal = d["cal"]
        d["params"] = [t.clone().requires_grad_(True) for t in (cal["gain_x"], cal["gain_y"], cal["dterms"], d["taps"])]
    elif kind == "batch":
        insts = [ps.Instance(fft_len=1 << e, bits=b) for e, _, b in _stream_sets(case)]
        d["plan"], d["outs"] = ps.Plan(insts, device="cuda"), [_out(i) for i in insts]
    elif kind == "tav":
        d["lags"] = [int(v) for v in case["lags"].split(",")]
    return d


SAV_LAGS = [1, 2, 4, 8, 16, 64, 256, 512]
SAV_SPACING = 16e6 / 2 ** 18  # channel width in Hz


def run(state):
    case = state["case"]
    kind = case["kind"]
    if kind == "spectra":
        plan = state["plan"]
        plan.reset()
        plan.accumulate_stokes(state["packed"], out=state["out"], feed=case["feed"], **state.get("cal", {}))
        return state["out"]
    if kind == "power":
        plan = state["plan"]
        plan.reset()
        plan.accumulate_stokes(state["packed"], out=state["out"])
        counts, power, _ = plan.histograms()
        return state["out"], counts, power
    if kind == "train":
        params = state["params"]
        iquv = autograd.stokes(state["plan"], state["packed"], *params, psi=state["cal"]["psi"])
        return (iquv.detach(), *torch.autograd.grad(iquv, params, state["upstream"]))
    if kind == "batch":
        plan = state["plan"]
        plan.reset()
        return plan.accumulate_stokes(state["packed"], outs=state["outs"])
    if kind == "reduce":
        smooth = ps.bandpass_fit(state["h"], case["knots"], 0.06)
        hat = ps.bandpass_correct(state["hk"], smooth, state["gain"])
        mean, count = ps.channel_average(hat, case["factor"], state["flags"])
        return smooth, hat, mean, count, ps.band_stats(mean), ps.allan(hat, SAV_LAGS, SAV_SPACING)
    return ps.allan(state["x"], state["lags"], 1.0, normalize=True, axis=0)


# ------------------------------------------------------------------------------------------------
# what a pass cannot do without

def _integration_work(log2n, samples, streams, bits, hop=1):
    n = 1 << log2n
    frames = (samples - n) * hop // n + 1
    pairs = len(PAIRS[streams])
    # real transforms (5/2 N log2 N), products and sums (14 per pair and channel)
    flops = frames * (streams * 2.5 * n * log2n + pairs * 14 * n / 2)
    return samples * streams * bits / 8 + pairs * n / 2 * 16, flops


def work(case):
    kind = case["kind"]
    if kind in ("spectra", "power", "train"):
        n, streams = 1 << case["log2n"], case.get("streams", 2)
        pairs = len(PAIRS[streams])
        b, f = _integration_work(case["log2n"], n * case["frames"], streams, case["bits"], case.get("hop", 1))
        if case.get("cal"):
            b += pairs * n / 2 * 16
        if kind == "power":
            b += 2 * (8 << case["bits"])
        if kind == "train":  # gains in and out, the upstream gradient; the adjoint transforms
            b += pairs * n / 2 * (16 + 16 + 16)
            f *= 2
        return dict(bytes=b, flops=f)
    if kind == "batch":
        parts = [_integration_work(e, f << e, 2, b) for e, f, b in _stream_sets(case)]
        return dict(bytes=sum(p[0] for p in parts), flops=sum(p[1] for p in parts))
    if kind == "reduce":
        n, c = case["spectra"], case["channels"]
        # h, hk, flags in; smooth, the variation, bins and counts, moments and Allan variances out
        return dict(bytes=4 * c + 4 * n * c + c + 4 * c + 4 * n * c + 8 * n * c / case["factor"] + 16 * n
                    + 8 * n * len(SAV_LAGS),
                    flops=c * 40 + n * c * (3 + 2 + 4 * len(SAV_LAGS)))
    lags = len(case["lags"].split(","))
    return dict(bytes=4 * case["points"] * case["series"] + 8 * lags * case["series"],
                flops=case["points"] * case["series"] * (1 + 4 * lags))


# ------------------------------------------------------------------------------------------------
# the results in 64 bits

def _levels(packed, samples, streams, bits):
    """[samples][streams] float64 levels of packed codes."""
    if bits == 8:
        return packed.view(torch.int8).view(samples, streams).double()
    mask = (1 << bits) - 1
    parts = [(packed >> (i * bits)) & mask for i in range(8 // bits)]
    return (2 * torch.stack(parts, 1).view(samples, streams).double() - mask)


def _window64(kind, n):
    if kind == "rect":
        return torch.ones(n, dtype=torch.float64, device="cuda")
    a0, a1, a2 = {"hann": (0.5, 0.5, 0.0), "hamming": (0.54, 0.46, 0.0), "blackman": (0.42, 0.5, 0.08)}[kind]
    ph = 2 * math.pi * torch.arange(n, dtype=torch.float64, device="cuda") / n
    return a0 - a1 * torch.cos(ph) + a2 * torch.cos(2 * ph)


def _coherency64(packed, log2n, samples, streams, bits, window, hop=1):
    """Normalised XX*, YY*, XY* [pairs][channels] of an integration, frames in chunks of about 2^23 samples."""
    n = 1 << log2n
    step = n // hop
    frames = (samples - n) // step + 1
    chunk = max(1, (1 << 23) // n)
    pairs = PAIRS[streams]
    c = n // 2
    xx = torch.zeros((len(pairs), c), dtype=torch.float64, device="cuda")
    yy, xy = torch.zeros_like(xx), torch.zeros((len(pairs), c), dtype=torch.complex128, device="cuda")
    per_sample = streams * bits
    for f0 in range(0, frames, chunk):
        nf = min(chunk, frames - f0)
        t0, t1 = f0 * step, (f0 + nf - 1) * step + n
        v = _levels(packed[t0 * per_sample // 8:t1 * per_sample // 8], t1 - t0, streams, bits)
        for p, (x, y) in enumerate(pairs):
            sx = torch.fft.rfft(v[:, x].contiguous().unfold(0, n, step) * window)[:, :c]
            sy = torch.fft.rfft(v[:, y].contiguous().unfold(0, n, step) * window)[:, :c]
            xx[p] += sx.abs().square().sum(0)
            yy[p] += sy.abs().square().sum(0)
            xy[p] += (sx * sy.conj()).sum(0)
    scale = 1 / (frames * window.square().sum())
    return xx * scale, yy * scale, xy * scale


def _stokes64(xx, yy, xy, cal=None, feed="linear"):
    psi = 0.0
    if cal:
        psi = cal["psi"]
        gx, gy = cal["gain_x"].to(torch.complex128), cal["gain_y"].to(torch.complex128)
        d = cal["dterms"].to(torch.complex128)
        dx, dy = d[:, :1], d[:, 1:]
        # C = (G J)^-1 M (G J)^-H with J = [[1, dx], [dy, 1]]
        det = gx * gy * (1 - dx * dy)
        a, b, e, f = gy / det, -gx * dx / det, -gy * dy / det, gx / det
        yx = xy.conj()
        t00, t01, t10, t11 = a * xx + b * yx, a * xy + b * yy, e * xx + f * yx, e * xy + f * yy
        xx, yy = (t00 * a.conj() + t01 * b.conj()).real, (t10 * e.conj() + t11 * f.conj()).real
        xy = t00 * e.conj() + t01 * f.conj()
    c2, s2 = math.cos(2 * psi), math.sin(2 * psi)
    total, diff = (xx + yy) / 2, (xx - yy) / 2
    if feed == "circular":
        return torch.stack([total, c2 * xy.real - s2 * xy.imag, s2 * xy.real + c2 * xy.imag, diff], 1)
    return torch.stack([total, c2 * diff - s2 * xy.real, s2 * diff + c2 * xy.real, xy.imag], 1)


def _histograms64(packed, samples, bits):
    """Counts [1][2][2^bits] in level order and the power estimates [1][2][2]."""
    lv = _levels(packed, samples, 2, bits)
    bins = ((lv + 128) if bits == 8 else (lv + (1 << bits) - 1) / 2).to(torch.int64)
    counts = torch.stack([torch.bincount(bins[:, s], minlength=1 << bits) for s in (0, 1)])[None]
    mean = lv.square().mean(0)
    ratio = torch.full_like(mean, math.nan)
    if bits == 2:
        inner = counts[0, :, 1:3].sum(1).double() / samples
        ratio = 1 / (math.sqrt(2) * torch.erfinv(inner))
    return counts, torch.stack([mean, ratio], 1)[None]


def _window_taps64(taps, n):
    u = torch.arange(n, dtype=torch.float64, device="cuda") * (len(taps) - 1) / (n - 1)
    j = u.floor().clamp(max=len(taps) - 2).long()
    return (1 - (u - j)) * taps[j] + (u - j) * taps[j + 1]


def _train64(case, d):
    n, frames = 1 << case["log2n"], case["frames"]
    with torch.enable_grad():
        cal = d["cal"]
        params = [t.detach().to(torch.complex128 if t.is_complex() else torch.float64).requires_grad_(True)
                  for t in (cal["gain_x"], cal["gain_y"], cal["dterms"], d["taps"])]
        window = _window_taps64(params[3], n)
        chunk = max(1, (1 << 23) // n)
        sums = [0, 0, 0]
        for f0 in range(0, frames, chunk):
            nf = min(chunk, frames - f0)
            per = 2 * case["bits"] * n // 8
            v = _levels(d["packed"][f0 * per:(f0 + nf) * per], nf * n, 2, case["bits"]).view(nf, n, 2)
            sx = torch.fft.rfft(v[:, :, 0] * window)[:, :n // 2]
            sy = torch.fft.rfft(v[:, :, 1] * window)[:, :n // 2]
            parts = (sx.real.square() + sx.imag.square(), sy.real.square() + sy.imag.square(), sx * sy.conj())
            sums = [s + q.sum(0) for s, q in zip(sums, parts)]
        scale = 1 / (frames * window.square().sum())
        xx, yy, xy = (s[None] * scale for s in sums)
        iquv = _stokes64(xx, yy, xy, dict(gain_x=params[0], gain_y=params[1], dterms=params[2], psi=cal["psi"]))
        return (iquv.detach(), *torch.autograd.grad(iquv, params, d["upstream"].double()))


def _spline64(h, knots, edge):
    """Least-squares cubic B-spline of h with uniform knots, edge of the band left out (NaN) at each end."""
    n = h.numel()
    c0 = math.floor(edge * n)
    c1 = n - c0
    n_int = -(-(c1 - c0) // knots)
    s = torch.arange(c1 - c0, dtype=torch.float64, device="cuda") / knots
    j = s.floor().long()
    u = s - j
    basis = torch.stack([(1 - u) ** 3 / 6, (3 * u ** 3 - 6 * u ** 2 + 4) / 6,
                         (-3 * u ** 3 + 3 * u ** 2 + 3 * u + 1) / 6, u ** 3 / 6], 1)
    at = j[:, None] + torch.arange(4, device="cuda")
    nb = n_int + 3
    a = torch.zeros(nb * nb, dtype=torch.float64, device="cuda")
    a.index_add_(0, (at[:, :, None] * nb + at[:, None, :]).reshape(-1), (basis[:, :, None] * basis[:, None, :]).reshape(-1))
    r = torch.zeros(nb, dtype=torch.float64, device="cuda")
    r.index_add_(0, at.reshape(-1), (basis * h[c0:c1].double()[:, None]).reshape(-1))
    coef = torch.linalg.solve(a.view(nb, nb).cpu(), r.cpu()).cuda()
    out = torch.full((n,), math.nan, dtype=torch.float64, device="cuda")
    out[c0:c1] = (basis * coef[at]).sum(1)
    return out


def _allan64(x, lags, spacing, normalize):
    """Second-difference Allan variances along the last axis, non-finite triples left out."""
    if normalize:
        x = x / x.nanmean(-1, keepdim=True)
    out = []
    for lag in lags:
        d = x[:, 2 * lag:] - 2 * x[:, lag:-lag] + x[:, :-2 * lag]
        out.append(d.square().nanmean(-1) / (2 * (lag * spacing) ** 2))
    return torch.stack(out, 1)


def exact(case, seed):
    d = _inputs(case, seed)
    kind = case["kind"]
    if kind in ("spectra", "power"):
        n, streams = 1 << case["log2n"], case.get("streams", 2)
        m = _coherency64(d["packed"], case["log2n"], n * case["frames"], streams, case["bits"],
                         _window64(case.get("window", "rect"), n), case.get("hop", 1))
        iquv = _stokes64(*m, d.get("cal"), case.get("feed", "linear"))
        return iquv if kind == "spectra" else (iquv, *_histograms64(d["packed"], n * case["frames"], case["bits"]))
    if kind == "train":
        return _train64(case, d)
    if kind == "batch":
        return [_stokes64(*_coherency64(p, e, f << e, 2, b, _window64("rect", 1 << e)))
                for p, (e, f, b) in zip(d["packed"], _stream_sets(case))]
    if kind == "reduce":
        smooth = _spline64(d["h"], case["knots"], 0.06)
        hat = d["hk"].double() / (d["gain"][:, None] * smooth)
        bins = hat.view(hat.shape[0], -1, case["factor"])
        use = bins.isfinite() & (d["flags"] == 0).view(-1, case["factor"])
        count = use.sum(-1)
        mean = torch.where(use, bins, 0.0).sum(-1) / count
        moments = torch.stack([mean.nanmean(-1), (mean - mean.nanmean(-1, keepdim=True)).square().nanmean(-1).sqrt()], 1)
        return smooth, hat, mean, count.to(torch.int32), moments, _allan64(hat, SAV_LAGS, SAV_SPACING, False)
    lags = [int(v) for v in case["lags"].split(",")]
    x = d["x"]
    return torch.cat([_allan64(x[:, s:s + 4096].double().t().contiguous(), lags, 1.0, True)
                      for s in range(0, x.shape[1], 4096)])
