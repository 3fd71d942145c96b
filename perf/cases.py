"""Performance cases: what a user of the library has it do, through its public entry points.

The library's work is period detection in batches of sampled traces.  A program
holds the traces in GPU memory and a call site with its buffers (Detector,
RollingDetector, SpectralDetector), and calls it for every batch; the finalist
re-scorers (similarity, score_centred) are plain calls.  The cases cover each
entry point, each of the three score methods, one channel and several, windows
of their own and overlapping ones, lengths that are powers of two and lengths
that are not, and sizes from one short trace to a gigabyte of samples.

  listed()  draw(rng)            the cases, and one more of the same ranges
  prepare(case, seed)            inputs made on the GPU from the seed, and the call site
  run(state)                     one pass
  work(case)  tolerance(case)    bytes and operations of a pass; how exact its results are
  exact(case, seed)              the results in 64 bits, in plain torch
"""
from __future__ import annotations

import math

import numpy as np
import torch

import paper_2201_01684_amd as pd

DEVICE = "cuda"
METHODS = {"direct": 0, "fft": pd.FFT_SCORES, "mfma": pd.MFMA_SCORES}
C_LAG, ERR_MAX = pd.DEFAULT_C_LAG, pd.DEFAULT_ERR_MAX
C_PEAK = 0.65
STEP, C_EVAL, C_MEASURE, DIFF_THRESHOLD = 0.5, 6.5, 2.0, 0.05
FINALISTS = 5


def _detect(name, windows, n, tmin, tmax, method="direct", channels=1, stride=0, pmin=0, pmax=0,
            jitter=False, spikes=False):
    return {"name": name, "kind": "detect", "windows": windows, "channels": channels, "n": n,
            "stride": stride, "tmin": tmin, "tmax": tmax, "method": method,
            "pmin": pmin or max(8, tmax // 100), "pmax": pmax or max(16, (3 * tmax) // 5),
            "jitter": jitter, "spikes": spikes}


def _finalists(name, kind, windows, n, pmin, pmax, groups=3, channels=1):
    return {"name": name, "kind": kind, "windows": windows, "channels": channels, "n": n,
            "tmin": 2, "tmax": 2 * pmax + 2, "pmin": pmin, "pmax": pmax, "groups": groups,
            "jitter": False, "spikes": True}


def listed():
    return [
        # One short power trace re-detected as it grows (the online loop of Algorithm 3): latency.
        _detect("online", 1, 4096, 2, 1024, pmin=137, pmax=137),
        # A node's worth of jobs, each trace with its period's length wandering by 2%.
        _detect("batch", 64, 65536, 2, 8192, pmin=50, pmax=5000, jitter=True),
        # One long recording cut into overlapping windows, to find where its period changes.
        _detect("sliding", 4089, 16384, 2, 4096, stride=2048, pmin=900, pmax=1430),
        # A cluster's recordings with sampling spikes, all lags by the direct sums.
        _detect("large", 1024, 262144, 2, 32768, pmin=100, pmax=20000, spikes=True),
        # A batch of an odd length, not aligned to anything, scored through the FFT.
        _detect("batch_fft", 96, 100003, 7, 12345, method="fft"),
        # The cluster's recordings through the FFT.
        _detect("large_fft", 1024, 262144, 2, 32768, method="fft", pmin=100, pmax=20000,
                spikes=True),
        # Composite detection features: eight normalised counters a job, scores summed.
        _detect("channels_fft", 256, 131072, 2, 16384, method="fft", channels=8, pmin=200,
                pmax=8000),
        # The same kind of feature on the matrix cores, at an odd length.
        _detect("channels_mfma", 24, 65537, 3, 8192, method="mfma", channels=8),
        # Rolling detection (Algorithm 3): the suffixes of every trace, and whether it is stable.
        {"name": "rolling_fft", "kind": "rolling", "windows": 128, "channels": 1, "n": 100001,
         "tmin": 2, "tmax": 16384, "method": "fft", "pmin": 100, "pmax": 10000, "jitter": False,
         "spikes": True},
        # Finalist periods of a batch by Algorithm 2's grouped similarity.
        _finalists("similarity", "similarity", 256, 131072, 100, 20000),
        # The same finalists by the mean-removed score, at an odd length.
        _finalists("centred", "centred", 500, 200003, 100, 20000),
        # Algorithm 1's front end: the amplitude-spectrum peaks of two-channel traces.
        {"name": "spectral", "kind": "spectral", "windows": 300, "channels": 2, "n": 150001,
         "tmin": 2, "tmax": 32768, "pmin": 100, "pmax": 20000, "jitter": False, "spikes": True},
    ]


def _log(rng, lo, hi):
    """A whole number spread over [lo, hi] on the logarithm; odd as often as not."""
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(("online", "batch", "sliding", "fft", "mfma", "rolling", "similarity",
                       "centred", "spectral"))
    if kind == "online":
        n = _log(rng, 512, 16384)
        case = _detect("", rng.randint(1, 8), n, rng.randint(1, 8), min(n // 2, 6000, _log(rng, n // 8, n // 2)))
    elif kind == "batch":
        n = _log(rng, 12000, 200000)
        tmax = _log(rng, n // 32, n // 4)
        windows = max(1, min(_log(rng, 4, 400), int(1e12 / (n * tmax))))
        case = _detect("", windows, n, rng.randint(1, 9), tmax, channels=rng.choice((1, 1, 3)),
                       jitter=rng.random() < 0.5, spikes=rng.random() < 0.5)
    elif kind == "sliding":
        stride = 1024 * rng.randint(1, 3)
        n = stride * rng.choice((4, 6, 8)) if rng.random() < 0.6 else _log(rng, 6000, 20000)
        case = _detect("", _log(rng, 200, 3000), n, rng.randint(2, 5), _log(rng, n // 16, n // 4),
                       stride=stride)
    elif kind == "fft":
        n = _log(rng, 3000, 300000)
        channels = rng.choice((1, 1, 2, 5, 8))
        windows = max(1, min(_log(rng, 8, 2000), (1 << 26) // (n * channels)))
        case = _detect("", windows, n, rng.randint(1, 9), _log(rng, n // 64, n // 3), method="fft",
                       channels=channels, jitter=rng.random() < 0.5, spikes=rng.random() < 0.5)
    elif kind == "mfma":
        n = _log(rng, 6000, 200000)
        tmax = _log(rng, n // 64, n // 4)
        channels = rng.choice((1, 3, 8))
        windows = max(1, min(_log(rng, 4, 400), int(1.5e12 / (n * tmax * channels))))
        case = _detect("", windows, n, rng.randint(1, 9), tmax, method="mfma", channels=channels)
    elif kind == "rolling":
        n = _log(rng, 8000, 200000)
        tmax = _log(rng, n // 32, n // 5)
        windows = max(1, min(_log(rng, 8, 256), (1 << 24) // n))
        case = {"kind": "rolling", "windows": windows, "channels": 1, "n": n,
                "tmin": rng.randint(1, 5), "tmax": tmax, "method": rng.choice(("fft", "fft", "mfma")),
                "pmin": max(8, tmax // 100), "pmax": max(16, tmax // 2), "jitter": False,
                "spikes": rng.random() < 0.5}
    elif kind in ("similarity", "centred"):
        n = _log(rng, 6000, 250000)
        most = 1 << (24 if kind == "similarity" else 26)
        pmax = _log(rng, n // 40, n // 6)
        case = _finalists("", kind, max(1, min(_log(rng, 16, 1000), most // n)), n,
                          max(8, pmax // 100), pmax, groups=rng.randint(2, 4))
    else:
        n = _log(rng, 1500, 300000)
        channels = rng.choice((1, 2, 4))
        tmax = _log(rng, n // 32, n // 3)
        case = {"kind": "spectral", "windows": max(1, min(_log(rng, 8, 2000), (1 << 26) // (n * channels))),
                "channels": channels, "n": n, "tmin": rng.randint(1, 5), "tmax": tmax,
                "pmin": max(8, tmax // 100), "pmax": max(16, tmax // 2), "jitter": False,
                "spikes": rng.random() < 0.5}
    case.pop("name", None)
    return case


# ---------------------------------------------------------------------------
# Inputs: a template of piecewise-constant levels a trace, tiled with its
# period, plus noise (and one-sample spikes, or repeats of varying length).
# One channel is sampled power in W; several are normalised counters.
# ---------------------------------------------------------------------------

def _levels_at(phase, period, cuts, levels):
    """levels[b, c, k] where cuts[b, k - 1] <= phase / period < cuts[b, k]."""
    idx = torch.searchsorted(cuts, phase / period, right=True)
    return torch.gather(levels, 2, idx[:, None, :].expand(-1, levels.shape[1], -1))


def _traces(case, rows, n, seed):
    """[rows, channels, n] float32 samples and the planted periods [rows]."""
    g = torch.Generator(device=DEVICE).manual_seed(1009 * seed + 7)
    u = lambda *s: torch.rand(*s, generator=g, device=DEVICE, dtype=torch.float32)
    c = case["channels"]
    lo, hi = math.log(case["pmin"]), math.log(case["pmax"])
    period = torch.exp(lo + (hi - lo) * u(rows).double()).round()
    kmax = 24
    cuts = u(rows, kmax - 1)
    keep = torch.arange(kmax - 1, device=DEVICE)[None, :] < 3 + (u(rows, 1) * (kmax - 4)).floor()
    cuts = torch.where(keep, cuts, torch.full_like(cuts, 2.0)).sort(dim=1).values
    levels = 80.0 + 320.0 * u(rows, c, kmax)
    x = torch.empty((rows, c, n), dtype=torch.float32, device=DEVICE)
    i = torch.arange(n, device=DEVICE, dtype=torch.float64)
    step = max(1, (1 << 23) // n)
    for b in range(0, rows, step):
        s = slice(b, min(rows, b + step))
        p = period[s, None]
        if case["jitter"]:
            reps = int(n / (0.97 * case["pmin"])) + 2
            ends = torch.cumsum((p * (0.98 + 0.04 * u(p.shape[0], reps))).round(), 1)
            at = i.expand(p.shape[0], -1).contiguous()
            rep = torch.searchsorted(ends, at, right=True)
            edges = torch.cat((torch.zeros_like(ends[:, :1]), ends), 1)
            start, end = torch.gather(edges, 1, rep), torch.gather(edges, 1, rep + 1)
            phase, length = at - start, end - start
        else:
            phase, length = i[None, :] % p, p
        y = _levels_at(phase.float(), length.float(), cuts[s], levels[s])
        if c > 1:
            y = (y - y.mean(2, keepdim=True)) / y.std(2, keepdim=True)
            y += 0.05 * torch.randn(y.shape, generator=g, device=DEVICE)
        else:
            if case["spikes"]:
                y += 50.0 * (u(*y.shape) < 0.05)
            y += 4.0 * torch.randn(y.shape, generator=g, device=DEVICE)
        x[s] = y
    return x, period.to(torch.int64)


def _overlapping(case, seed):
    """One recording whose period changes in the middle, cut into overlapping windows."""
    total = (case["windows"] - 1) * case["stride"] + case["n"]
    one, two = dict(case, pmax=case["pmin"]), dict(case, pmin=case["pmax"])
    h = total // 2
    return torch.cat((_traces(one, 1, h, seed)[0].reshape(-1),
                      _traces(two, 1, total - h, seed + 500000)[0].reshape(-1)))


def _inputs(case, seed):
    if case.get("stride"):
        return _overlapping(case, seed), None
    return _traces(case, case["windows"], case["n"], seed)


def _weights(case):
    c = case["channels"]
    return None if c == 1 else [0.5 + 0.25 * k for k in range(c)]


def _queries(case, period):
    """Finalists of each window: its period, the neighbours, the double and one that is none."""
    p = period[:, None]
    lags = torch.cat((p - 1, p, p + 1, 2 * p, (3 * p) // 2), 1)
    lags = lags.clamp(1, case["n"] // 2).to(torch.int32).reshape(-1).contiguous()
    windows = torch.arange(case["windows"], device=DEVICE, dtype=torch.int32)
    return windows.repeat_interleave(FINALISTS).contiguous(), lags


def prepare(case, seed):
    x, period = _inputs(case, seed)
    n, c = case["n"], case["channels"]
    flags = METHODS[case.get("method", "direct")]
    desc, w = pd.make_desc(case["windows"], c, n, case.get("stride") or n * c, n, case["tmin"],
                           min(case["tmax"], n // 2), weights=_weights(case), flags=flags)
    state = {"kind": case["kind"], "case": case, "x": x, "desc": desc, "w": w}
    if case["kind"] == "detect":
        state["det"] = pd.Detector(x, desc, w)
    elif case["kind"] == "rolling":
        state["det"] = pd.RollingDetector(x, desc, pd.rolling_params(), w)
    elif case["kind"] == "spectral":
        state["det"] = pd.SpectralDetector(x, desc, pd.spectral_params(C_PEAK), w)
    else:
        state["windows"], state["lags"] = _queries(case, period)
    return state


# Result records are int32 tensors; their fields are views of them.  Left out:
# how many scores a call recomputed, and whether it did (counts of its own work).

def _detect_fields(r):
    return {"period": r[:, 0], "verdict": r[:, 1], "err": r.view(torch.float32)[:, 2],
            "n_candidates": r[:, 3], "t_cand": r[:, 4], "t_low": r[:, 5], "t_up": r[:, 6]}


def _rolling_fields(r):
    f32, f64, i64 = r.view(torch.float32), r.view(torch.float64), r.view(torch.int64)
    return {"period": r[:, 0], "verdict": r[:, 1], "stable": r[:, 2], "n_windows": r[:, 3],
            "t_init": r[:, 4], "best": r[:, 5], "smpdur_next": f64[:, 3], "diff": f32[:, 8],
            "err": f32[:, 9], "flags": r[:, 10], "periods": r[:, 12:28], "starts": i64[:, 14:30]}


def _spectral_fields(r):
    f64 = r.view(torch.float64)
    return {"count": r[:, 0], "n_peaks": r[:, 2], "max_peak": f64[:, 2], "periods": r[:, 6:22],
            "bins": r[:, 22:38], "amplitudes": f64[:, 19:35]}


def run(state):
    kind = state["kind"]
    if kind == "similarity":
        return pd.similarity(state["x"], state["desc"], state["windows"], state["lags"],
                             num_groups=state["case"]["groups"])
    if kind == "centred":
        return pd.score_centred(state["x"], state["desc"], state["windows"], state["lags"])
    det = state["det"]
    det.run()
    if kind == "detect":
        return dict(_detect_fields(det.results), scores=det.scores)
    return _rolling_fields(det.results) if kind == "rolling" else _spectral_fields(det.results)


def work(case):
    """Samples read once, results written once.  Operations: by the direct sums and on the matrix
    cores three a pair of samples (for overlapping windows each pair of the recording once), by the
    FFT a real transform of N + Tmax points there and back, and what the finalist scores' definitions
    take (grouped similarity: 20 fitting steps of G components at 13 a sample)."""
    b, c, n, kind = case["windows"], case["channels"], case["n"], case["kind"]
    tmin, tmax = case["tmin"], min(case["tmax"], n // 2)
    lags = tmax - tmin + 1
    samples = b * c * n
    if case.get("stride") and case["stride"] < n:
        samples = (b - 1) * case["stride"] + n
    out = b * {"detect": 4 * lags + 36, "rolling": 240, "spectral": 280}.get(kind, 8 * FINALISTS)
    mean = n - (tmin + tmax) / 2
    fft = lambda points: 2.5 * points * math.log2(points)
    if kind == "detect" and case["method"] != "fft":
        flops = 3.0 * lags * (b * c * mean if not case["stride"] else min(b * mean, samples))
    elif kind == "detect":
        flops = b * c * 2 * fft(n + tmax)
    elif kind == "rolling":   # the whole trace, then its suffixes (7 of 5.25 .. 2.25 periods)
        p = math.sqrt(case["pmin"] * case["pmax"])
        spans = [min(n, (2.25 + 0.5 * k) * p) for k in range(7)]
        flops = b * c * (2 * fft(n + tmax) + sum(2 * fft(1.5 * s) for s in spans))
    elif kind == "spectral":
        flops = b * c * fft(n)
    elif kind == "similarity":
        flops = float(FINALISTS) * samples * 20 * 13 * case["groups"]
    else:
        flops = float(FINALISTS) * samples * 4
    return {"bytes": 4.0 * samples + out, "flops": flops}


def tolerance(case):
    kind = case["kind"]
    if kind in ("detect", "rolling"):
        # fp32 runs of at most 256 terms, or the rounding to fp32: up to 1.5e-7 off the exact
        # scores.  Periods and bounds are decided exactly, whatever the rounding of the scores.
        return {"rel": 1e-6, "max": 1e-5, "differ": 0.0}
    # fp64 throughout, 1e-15 off or less.  A fit's rounding reaches the grouped similarity only
    # through a label that it flips, and a spectrum's only through its own last bits.
    if kind == "similarity":
        return {"rel": 1e-11, "max": 1e-9}
    return {"rel": 1e-14, "max": 1e-12, "differ": 0.0}


# ---------------------------------------------------------------------------
# The same in 64 bits and plain torch.
# ---------------------------------------------------------------------------

def _scores64(y, tmin, tmax, w):
    """S(T) of [rows, channels, n] float64 windows, tmin <= T <= tmax, through torch's FFT."""
    n = y.shape[2]
    y = y - y.mean(2, keepdim=True)
    spec = torch.fft.rfft(y, n=1 << (n + tmax - 1).bit_length())
    power = spec.real.square() + spec.imag.square()
    r = torch.fft.irfft(torch.complex(power, torch.zeros_like(power)),
                        n=1 << (n + tmax - 1).bit_length())[..., tmin:tmax + 1]
    e = torch.cumsum(y.square(), 2)
    t = torch.arange(tmin, tmax + 1, device=y.device)
    d = e[..., n - t - 1] + (e[..., -1:] - e[..., t - 1]) - 2.0 * r
    s = d / (n - t).double()
    return (s * w[None, :, None]).sum(1)


def _select64(s, r, n, tmin):
    """Algorithm 1's rule on scores s [rows, lags] with references r [rows]."""
    rows, lags = s.shape
    t = torch.arange(tmin, tmin + lags, device=s.device)
    big = torch.full_like(s, math.inf)
    peak = torch.zeros_like(s, dtype=torch.bool)
    peak[:, 1:-1] = (s[:, 1:-1] < s[:, :-2]) & (s[:, 1:-1] <= s[:, 2:])
    s_pk = torch.where(peak, s, big).amin(1)
    thr = r - C_LAG * (r - s_pk)
    cand = peak & (s < thr[:, None])
    found = cand.any(1)
    tc = torch.where(found, t[cand.to(torch.int8).argmax(1)], torch.ones_like(t[:1]))
    d = n - 1
    lo = ((tc * d + (d + tc) - 1) // (d + tc)).clamp(min=tmin)
    hi = ((tc * d) // (d - tc)).clamp(max=tmin + lags - 1)
    near = torch.where((t >= lo[:, None]) & (t <= hi[:, None]), s, big)
    best = near.argmin(1)
    err = s.gather(1, best[:, None])[:, 0] / r
    z = lambda v: torch.where(found, v, torch.zeros_like(v)).to(torch.int32)
    aperiodic = ~found | (err >= ERR_MAX)
    return {"period": z(t[best]), "verdict": aperiodic.to(torch.int32),
            "err": torch.where(found, err, torch.zeros_like(err)),
            "n_candidates": cand.sum(1).to(torch.int32), "t_cand": z(tc), "t_low": z(lo),
            "t_up": z(hi)}


def _detect64(windows, tmin, tmax, w, step):
    """Scores and selections of windows [rows, channels, n], a few rows at a time."""
    parts, scores = [], []
    for b in range(0, windows.shape[0], step):
        y = windows[b:b + step].double()
        s = _scores64(y, tmin, tmax, w)
        r = 2.0 * (y.var(2, unbiased=False) * w[None, :]).sum(1)
        parts.append(_select64(s, r, y.shape[2], tmin))
        scores.append(s)
    return {k: torch.cat([p[k] for p in parts]) for k in parts[0]}, torch.cat(scores)


def _similarity64(x, t, groups, iters=20):
    """Algorithm 2's Err of one window x [n] and period t."""
    k = x.shape[0] // t
    if k < 2:
        return torch.full((), -1.0, dtype=torch.float64, device=x.device)
    a = x[:k * t].reshape(k, t)
    prev, back = a[:-1], a[1:]
    lo, hi = prev.amin(1, keepdim=True), prev.amax(1, keepdim=True)
    width = (hi - lo) / groups
    mu = lo + (torch.arange(groups, device=x.device) + 0.5) * width
    var, pi = (width * width).expand_as(mu), torch.full_like(mu, 1.0 / groups)
    floor = 1e-6 * width * width

    def density():
        d = prev[:, :, None] - mu[:, None, :]
        return (pi.log() - 0.5 * (2.0 * math.pi * var).log())[:, None, :] - d * d / (2.0 * var)[:, None, :]

    for _ in range(iters):
        r = torch.softmax(density(), 2)
        nk = r.sum(1)
        mu = (r * prev[:, :, None]).sum(1) / nk
        var = torch.maximum((r * (prev[:, :, None] - mu[:, None, :]).square()).sum(1) / nk, floor)
        pi = nk / t
    hard = torch.nn.functional.one_hot(density().argmax(2), groups).double()
    cnt = hard.sum(1)
    div = cnt.clamp(min=1.0)
    ma = (hard * prev[:, :, None]).sum(1) / div - prev.mean(1, keepdim=True)
    mb = (hard * back[:, :, None]).sum(1) / div - back.mean(1, keepdim=True)
    den = (ma.abs() + mb.abs()) / 2.0
    smape = torch.where(den > 0, (ma - mb).abs() / den, torch.zeros_like(den))
    return ((cnt * smape).sum(1) / t).mean()


def _centred64(x, t):
    k = x.shape[0] // t
    if k < 2:
        return torch.full((), -1.0, dtype=torch.float64, device=x.device)
    a = x[:k * t].reshape(k, t)
    a = a - a.mean(1, keepdim=True)
    return (a[1:] - a[:-1]).square().sum() / ((k - 1) * t)


def _rolling64(x, case):
    """Algorithm 3 on [rows, 1, n] windows: floating results only."""
    rows, _, n = x.shape
    w = torch.ones(1, dtype=torch.float64, device=x.device)
    tmin, tmax = case["tmin"], min(case["tmax"], n // 2)
    whole, _ = _detect64(x, tmin, tmax, w, max(1, (1 << 24) // n))
    out = {"smpdur_next": np.zeros(rows), "diff": np.zeros(rows), "err": np.zeros(rows)}
    t_init, verdict = whole["period"].tolist(), whole["verdict"].tolist()
    dur = float(n - 1)
    for b in range(rows):
        t = float(t_init[b])
        if verdict[b] != 0:
            continue
        if dur < C_MEASURE * t:
            out["smpdur_next"][b] = C_MEASURE * t - dur
            out["err"][b] = float(whole["err"][b])
            continue
        start, found = max(0.0, dur - (2.0 + C_EVAL * STEP) * t), []
        while (dur - start) / t >= C_MEASURE:
            y = x[b:b + 1, :, int(math.floor(start)):]
            m = y.shape[2]
            if min(tmax, m // 2) >= tmin + 2:
                o, _ = _detect64(y, tmin, min(tmax, m // 2), w, 1)
                if int(o["verdict"]) == 0:
                    found.append((int(o["period"]), float(o["err"])))
            start += STEP * t
        if not found:
            return None
        ts = [p for p, _ in found]
        diff = abs(max(ts) - min(ts)) / (sum(ts) / len(ts))
        out["diff"][b], out["err"][b] = diff, min(e for _, e in found)
        out["smpdur_next"][b] = -1.0 if diff < DIFF_THRESHOLD else math.ceil(dur / max(ts)) * max(ts) - dur
    return out


def _spectral64(x, case):
    n = case["n"]
    length = 1 << max(6, (n - 1).bit_length())
    w = torch.tensor(_weights(case) or [1.0], dtype=torch.float64, device=x.device)
    rows = {"max_peak": [], "amplitudes": []}
    for b in range(0, x.shape[0], 32):
        y = x[b:b + 32].double()
        amp = torch.fft.rfft(y - y.mean(2, keepdim=True), n=length).abs()
        amp = (amp * w[None, :, None]).sum(1)
        mid = amp[:, 2:-1]
        peak = (mid > amp[:, 1:-2]) & (mid >= amp[:, 3:])
        heights = torch.where(peak, mid, torch.zeros_like(mid))
        top = heights.amax(1)
        k = torch.arange(2, amp.shape[1] - 1, device=x.device)
        period = (2 * length + k) // (2 * k)
        fits = (period >= case["tmin"]) & (period <= min(case["tmax"], n // 2))
        good = peak & (mid > C_PEAK * top[:, None]) & fits
        rows["max_peak"].append(top)
        rows["amplitudes"].append(torch.where(good, mid, torch.zeros_like(mid)).topk(16, 1).values)
    none = dict.fromkeys(("count", "n_peaks", "periods", "bins"))
    return dict(none, **{k: torch.cat(v) for k, v in rows.items()})


def exact(case, seed):
    x, period = _inputs(case, seed)
    kind, n = case["kind"], case["n"]
    w = torch.tensor(_weights(case) or [1.0], dtype=torch.float64, device=DEVICE)
    if kind == "detect":
        windows = x.unfold(0, n, case["stride"])[:, None, :] if case["stride"] else x
        step = max(1, (1 << 24) // (n * case["channels"]))
        fields, scores = _detect64(windows, case["tmin"], min(case["tmax"], n // 2), w, step)
        return dict(fields, scores=scores)
    if kind == "rolling":
        found = _rolling64(x, case)
        if found is None:
            return None
        none = dict.fromkeys(("period", "verdict", "stable", "n_windows", "t_init", "best",
                              "flags", "periods", "starts"))
        return dict(none, **found)
    if kind == "spectral":
        return _spectral64(x, case)
    windows, lags = (v.tolist() for v in _queries(case, period))
    if kind == "similarity":
        one = lambda b, t: _similarity64(x[b, 0].double(), t, case["groups"])
    else:
        one = lambda b, t: _centred64(x[b, 0].double(), t)
    return torch.stack([one(b, t) for b, t in zip(windows, lags)])
