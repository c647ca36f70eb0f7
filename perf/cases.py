"""Performance cases of the dedispersion framework: the calls a user's program makes, through
the Python entry points, from the smallest block to the full-size workload.

listed() names the cases, draw() gives more of the same ranges, prepare() builds what a program
holds before the call (device input, plan, stream), run() is one call, work() the bytes and
operations the result needs, exact() the result in 64-bit arithmetic, from the definitions alone.

Bands (the repository's own): "mid" is 408-428 MHz sampled at 51.2 us, "low" is 120-180 MHz
sampled at 81.92 us.
"""
import math

import numpy as np
import torch

import paper_1401_8258_amd as dd

BANDS = {"mid": (428.0, 20.0, 51.2e-6), "low": (180.0, 60.0, 81.92e-6)}
DTYPES = {"f32": torch.float32, "f16": torch.float16, "u8": torch.uint8}
BYTES = {"f32": 4, "f16": 2, "u8": 1}
K_DM = 4.15e3
DEV = "cuda"
EXACT_ADDS = 6e11   # some 6 s of 64-bit gathers and adds on the device


def listed():
    return [
        # The small FP32 observation (64 channels, 0.84 s, 128 trials): launches and latency count.
        dict(name="f32_small", kind="plain", band="mid", nchan=64, nsamp=16384, ndm=128, step=0.1, dtype="f32", k=6.0),
        # The full FP32 observation (53.7 s of the 408-428 MHz band, 2048 trials).
        dict(name="f32_full", kind="plain", band="mid", nchan=1024, nsamp=1 << 20, ndm=2048, step=0.1, dtype="f32",
             k=6.0),
        # One FP32 beam followed in real time: a 1 s block pushed into its ring.
        dict(name="f32_stream_1s", kind="stream", band="mid", nchan=1024, block=19531, ndm=1024, step=0.1,
             dtype="f32", k=6.0),
        # A few seconds of FP16 power, an odd number of samples, channels and trials.
        dict(name="f16_ragged", kind="plain", band="mid", nchan=1001, nsamp=131071, ndm=901, step=0.1, dtype="f16",
             k=6.0),
        # An 8-bit beam of the usual band, 13 s.
        dict(name="u8_beam_mid", kind="plain", band="mid", nchan=1024, nsamp=1 << 18, ndm=2000, step=0.1, dtype="u8",
             k=6.0),
        # A short 8-bit beam with few, wide channels and a coarse DM step.
        dict(name="u8_short_256ch", kind="plain", band="mid", nchan=256, nsamp=20011, ndm=501, step=0.2, dtype="u8",
             k=6.0),
        # An 8-bit low-frequency beam: 4096 channels, delays of up to 73k samples.
        dict(name="u8_beam_low", kind="plain", band="low", nchan=4096, nsamp=200003, ndm=750, step=0.05, dtype="u8",
             k=6.0),
        # A serving step: the blocks that have arrived for four 8-bit beams, in one batched call.
        dict(name="u8_serving", kind="serving", n_mid=3, n_low=1, ndm_mid=2048, ndm_low=2048, k=6.0),
        # Time binning above the diagonal DM, half of the full FP32 observation.
        dict(name="binned_f32", kind="binned", band="mid", nchan=1024, nsamp=1 << 19, ndm=2048, step=0.1, max_log2=4,
             dtype="f32", k=6.0),
        # Two-step subband dedispersion of the same input, the lower half of the DM range.
        dict(name="subband_f32", kind="subband", band="mid", nchan=1024, nsamp=1 << 19, ndm=960, step=0.1, csub=32,
             dgroup=16, dtype="f32", k=6.0),
        # RFI mitigation of a filterbank before dedispersion (the raw data are kept).
        dict(name="rfi_f32", kind="rfi", band="mid", nchan=1024, nsamp=1 << 18, window=256, order=6, dtype="f32"),
        # Detrending, normalisation and the boxcar search over dedispersed series.
        dict(name="search", kind="search", nrows=1024, n=250007, max_log2=6, k=6.5),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["plain"] * 6 + ["stream", "serving", "binned", "subband", "rfi", "search"])
    if kind == "plain":
        while True:
            band = rng.choice(["mid", "mid", "low"])
            dtype = rng.choice(["f32", "f16", "u8"]) if band == "mid" else "u8"
            nchan = 4096 if band == "low" else rng.choice([64, 256, 512, 1024, _log_int(rng, 64, 1024)])
            step = rng.choice([0.05, 0.1, 0.2]) if band == "mid" else 0.05
            ndm = _log_int(rng, 100, 2048 if band == "mid" else 900)
            nsamp = _log_int(rng, 16384, 1 << 19)
            case = dict(kind=kind, band=band, nchan=nchan, nsamp=nsamp, ndm=ndm, step=step, dtype=dtype, k=6.0)
            if 2 * _maxdelay(case) <= nsamp and _adds(case) <= 1.0e12:
                return case
    if kind == "stream":
        return dict(kind=kind, band="mid", nchan=rng.choice([256, 512, 1024]), block=_log_int(rng, 4000, 40000),
                    ndm=_log_int(rng, 200, 2048), step=0.1, dtype=rng.choice(["f32", "u8"]), k=6.0)
    if kind == "serving":
        return dict(kind=kind, n_mid=rng.randint(1, 5), n_low=rng.randint(0, 1), ndm_mid=_log_int(rng, 500, 2048),
                    ndm_low=_log_int(rng, 500, 2048), k=6.0)
    if kind == "binned":
        return dict(kind=kind, band="mid", nchan=rng.choice([256, 512, 1024]), nsamp=_log_int(rng, 1 << 16, 1 << 19),
                    ndm=_log_int(rng, 500, 2048), step=0.1, max_log2=rng.randint(2, 4),
                    dtype=rng.choice(["f32", "u8"]), k=6.0)
    if kind == "subband":
        dgroup = rng.choice([16, 48])
        return dict(kind=kind, band="mid", nchan=rng.choice([512, 1024]), nsamp=_log_int(rng, 1 << 16, 1 << 19),
                    ndm=_log_int(rng, 400, 960 if dgroup == 16 else 2048), step=0.1, csub=32, dgroup=dgroup,
                    dtype="f32", k=6.0)
    if kind == "rfi":
        return dict(kind=kind, band="mid", nchan=rng.choice([256, 512, 1024]), nsamp=_log_int(rng, 19531, 1 << 18),
                    window=rng.choice([128, 256, 500]), order=6, dtype=rng.choice(["f32", "u8"]))
    return dict(kind="search", nrows=_log_int(rng, 128, 1024), n=_log_int(rng, 16000, 250007),
                max_log2=rng.randint(3, 6), k=6.5)


# ---------------------------------------------------------------- geometry

def _freq(band, nchan):
    top, bw, _ = BANDS[band]
    return top - np.arange(nchan, dtype=np.float64) * (bw / nchan)


def _dms(ndm, step):
    return np.arange(ndm, dtype=np.float64) * step


def _delays(freq, dms, tsamp, f_ref=None):
    """round(k DM (f^-2 - f_ref^-2) / tsamp), half away from zero: [nchan][ndm] int64."""
    ref = float(np.max(freq)) if f_ref is None else float(f_ref)
    diff = 1.0 / (freq * freq) - 1.0 / (ref * ref)
    x = ((K_DM * dms)[None, :] * diff[:, None]) / tsamp
    fl = np.floor(x)
    return (fl + (x - fl >= 0.5)).astype(np.int64)


def _maxdelay(case):
    f = _freq(case["band"], case["nchan"])
    return int(_delays(f[-1:], _dms(case["ndm"], case["step"])[-1:], BANDS[case["band"]][2], f[0]).max())


def _adds(case):
    return case["ndm"] * case["nchan"] * (case["nsamp"] - _maxdelay(case))


def _serving_beams(case):
    """(band, nchan, ndm, step, block) per beam: blocks of 1 s."""
    return ([("mid", 1024, case["ndm_mid"], 0.1, 19531)] * case["n_mid"] +
            [("low", 4096, case["ndm_low"], 0.05, 12207)] * case["n_low"])


# ---------------------------------------------------------------- inputs

def _noise(nchan, nsamp, dtype, gen):
    """Filterbank power as stored: N(0, 1), or codes of 128 + 16 N(0, 1)."""
    x = torch.randn((nchan, nsamp), generator=gen, device=DEV)
    if dtype == "u8":
        return x.mul_(16.0).add_(128.0).round_().clamp_(0, 255).to(torch.uint8)
    return x.to(DTYPES[dtype])


def _filterbank(case, nsamp, gen, npulse=4):
    """Noise with a few dispersed top-hat pulses along the band's delay curve."""
    nchan = case["nchan"]
    x = torch.randn((nchan, nsamp), generator=gen, device=DEV)
    f = _freq(case["band"], nchan)
    top = float(_dms(case["ndm"], case["step"])[-1])
    u = torch.rand((npulse, 2), generator=gen, device=DEV).cpu().numpy()
    ch = torch.arange(nchan, device=DEV)[:, None]
    for i in range(npulse):
        dl = _delays(f, np.array([u[i, 0] * top]), BANDS[case["band"]][2])[:, 0]
        w = (1, 4, 12, 32)[i % 4]
        t0 = int(u[i, 1] * max(nsamp - int(dl.max()) - w, 1))
        t = torch.from_numpy(dl).to(DEV)[:, None] + t0 + torch.arange(w, device=DEV)[None, :]
        x[ch, t.clamp_(max=nsamp - 1)] += (8.0 + 3.0 * i) / math.sqrt(nchan)
    if case["dtype"] == "u8":
        return x.mul_(16.0).add_(128.0).round_().clamp_(0, 255).to(torch.uint8)
    return x.to(DTYPES[case["dtype"]])


def _rfi_input(case, gen):
    """Noise on a curved bandpass with bursts in some channels and a few broadband spikes."""
    nchan, n = case["nchan"], case["nsamp"]
    c = torch.linspace(-1, 1, nchan, device=DEV, dtype=torch.float64)
    base = (100.0 + 8.0 * c - 6.0 * c * c).to(torch.float32)[:, None]
    x = torch.randn((nchan, n), generator=gen, device=DEV).mul_(8.0).add_(base)
    u = torch.rand((12, 2), generator=gen, device=DEV).cpu().numpy()
    for i in range(8):
        a = int(u[i, 1] * (n - 2000))
        x[int(u[i, 0] * nchan), a:a + 2000] += 60.0
    for i in range(8, 12):
        x[:, int(u[i, 1] * n)] += 40.0
    if case["dtype"] == "u8":
        return x.round_().clamp_(0, 255).to(torch.uint8)
    return x


def _series(case, gen):
    """Dedispersed series: noise with a slow drift and rare pulses."""
    x = torch.randn((case["nrows"], case["n"]), generator=gen, device=DEV).mul_(30.0)
    x += torch.linspace(0.0, 20.0, case["n"], device=DEV)[None, :] + 500.0
    t = torch.randint(0, case["n"] - 64, (case["nrows"],), generator=gen, device=DEV)
    rows = torch.arange(case["nrows"], device=DEV)
    for j in range(8):
        x[rows, t + j] += 120.0
    return x


def prepare(case, seed):
    gen = torch.Generator(device=DEV)
    gen.manual_seed(int(seed))
    kind = case["kind"]
    st = {"case": case}
    if kind == "search":
        st["x"] = _series(case, gen)
        return st
    if kind == "rfi":
        st["x"] = _rfi_input(case, gen)
        return st
    if kind == "serving":
        st["streams"], st["blocks"], st["outputs"] = [], [], []
        plans = {}
        for band, nchan, ndm, step, block in _serving_beams(case):
            key = (band, ndm)
            if key not in plans:  # beams of one kind share their plan
                plans[key] = dd.Plan(_freq(band, nchan), BANDS[band][2], _dms(ndm, step), dtype="u8")
            plan = plans[key]
            s = dd.Stream(plan, block)
            b = _noise(nchan, block, "u8", gen)
            for _ in range(plan.maxdelay // block):
                s.append(b)
            st["streams"].append(s)
            st["blocks"].append(b)
            st["outputs"].append(dd.api.alloc_outputs(ndm, block, DEV, case["k"], 1 << 16))
        run(st)  # the block with which every ring is full
        return st
    tsamp = BANDS[case["band"]][2]
    f, dms = _freq(case["band"], case["nchan"]), _dms(case["ndm"], case["step"])
    if kind == "stream":
        plan = dd.Plan(f, tsamp, dms, dtype=case["dtype"])
        st["stream"] = dd.Stream(plan, case["block"])
        st["x"] = _noise(case["nchan"], case["block"], case["dtype"], gen)
        for _ in range(plan.maxdelay // case["block"] + 1):
            st["stream"].push(st["x"], k_sigma=case["k"])
        return st
    if kind == "plain":
        st["plan"] = dd.Plan(f, tsamp, dms, dtype=case["dtype"])
    elif kind == "binned":
        st["plan"] = dd.BinnedPlan(f, tsamp, dms, dtype=case["dtype"], max_log2=case["max_log2"])
    else:
        st["plan"] = dd.SubbandPlan(f, tsamp, dms, chans_per_sub=case["csub"], dms_per_group=case["dgroup"])
    st["x"] = _filterbank(case, case["nsamp"], gen)
    st["plan"].workspace(case["nsamp"], torch.device(DEV))
    return st


# ---------------------------------------------------------------- one pass

def _list(records, cap):
    """The detections as a program's fixed-size event list: cap records, the rest zero."""
    ev = np.zeros(cap, dtype=records.dtype)
    ev[:records.size] = records
    return {name: ev[name] for name in records.dtype.names if name != "reserved"}


def run(st):
    case = st["case"]
    kind = case["kind"]
    if kind == "plain":
        cap = 65536 if case["nsamp"] > 1 << 19 else 4096
        r = st["plan"].dedisperse(st["x"], k_sigma=case["k"], cand_cap=cap)
        return {"out": r.out, "mean": r.mean, "rms": r.rms, "cands": _list(r.candidates(), cap)}
    if kind == "stream":
        r = st["stream"].push(st["x"], k_sigma=case["k"])
        return {"out": r.out, "mean": r.mean, "rms": r.rms, "ncand": r.ncand()}
    if kind == "serving":
        jobs, outs = [], []
        for s, b, o in zip(st["streams"], st["blocks"], st["outputs"]):
            w = s.append(b)
            if w is not None:
                jobs.append((s, w))
                outs.append(o)
        res = dd.batch_dedisperse(jobs, k_sigma=case["k"], cand_cap=1 << 16, outputs=outs)
        return [{"out": r.out, "mean": r.mean, "rms": r.rms, "ncand": r.ncand()} for r in res]
    if kind == "binned":
        r = st["plan"].dedisperse(st["x"], k_sigma=case["k"])
        parts = [{"out": p.out, "mean": p.mean, "rms": p.rms} for _, p in r.segments]
        return {"runs": parts, "cands": _list(r.candidates(), 1 << 16)}
    if kind == "subband":
        r = st["plan"].dedisperse(st["x"], k_sigma=case["k"])
        return {"out": [p.out for _, p in r], "mean": torch.cat([p.mean for _, p in r]),
                "rms": torch.cat([p.rms for _, p in r])}
    if kind == "rfi":
        x = st["x"].clone()
        thr = (12.0, 6.0)
        fit, rmse, fmean, flags = dd.rfi_mitigate(x, case["order"], thr[0], case["window"], thr[1])
        return {"data": x, "fit": fit, "rmse": rmse, "fit_mean": fmean, "flags": flags}
    s = st["x"].clone()
    rms = dd.detrend(s, normalise=True)
    p = dd.boxcar_search(s, max_log2=case["max_log2"], k_sigma=case["k"], cap=1 << 18)
    return {"series": s, "rms": rms, "pulses": _list(p, 1 << 18)}


# ---------------------------------------------------------------- what a pass cannot do without

def _binned_runs(case):
    """(log2, d0, d1) of the trials, split at 2^k times the diagonal DM."""
    f, dms = np.sort(_freq(case["band"], case["nchan"])), _dms(case["ndm"], case["step"])
    diag = 1.0 / np.max((K_DM * (1.0 / (f[:-1] * f[:-1]) - 1.0 / (f[1:] * f[1:]))) / BANDS[case["band"]][2])
    k = np.zeros(dms.size, dtype=np.int64)
    for j in range(case["max_log2"]):
        k += dms > diag * 2.0 ** j
    cut = [0] + [i for i in range(1, k.size) if k[i] != k[i - 1]] + [k.size]
    return [(int(k[a]), a, b) for a, b in zip(cut[:-1], cut[1:])]


def _subband_geometry(case):
    f, dms, ts = _freq(case["band"], case["nchan"]), _dms(case["ndm"], case["step"]), BANDS[case["band"]][2]
    subs = [(a, min(case["nchan"], a + case["csub"])) for a in range(0, case["nchan"], case["csub"])]
    groups = [(a, min(case["ndm"], a + case["dgroup"])) for a in range(0, case["ndm"], case["dgroup"])]
    nominal = dms[[a + (b - a - 1) // 2 for a, b in groups]]
    d1 = [_delays(f[a:b], nominal, ts) for a, b in subs]
    d2 = _delays(np.array([f[a] for a, _ in subs]), dms, ts)
    len1 = case["nsamp"] - max(int(d.max()) for d in d1)
    return subs, groups, d1, d2, len1


def work(case):
    kind = case["kind"]
    if kind in ("plain", "stream"):
        n_in = case["nsamp"] if kind == "plain" else case["block"]
        nout = n_in - _maxdelay(case) if kind == "plain" else n_in
        return {"bytes": case["nchan"] * n_in * BYTES[case["dtype"]] + 4 * case["ndm"] * nout,
                "flops": case["ndm"] * case["nchan"] * nout}
    if kind == "serving":
        b = f = 0
        for _, nchan, ndm, _, block in _serving_beams(case):
            b += nchan * block + 4 * ndm * block
            f += nchan * ndm * block
        return {"bytes": b, "flops": f}
    if kind == "binned":
        ts = BANDS[case["band"]][2]
        fr, dms = _freq(case["band"], case["nchan"]), _dms(case["ndm"], case["step"])
        b = case["nchan"] * case["nsamp"] * BYTES[case["dtype"]]
        fl = case["nchan"] * case["nsamp"]
        for k, a, e in _binned_runs(case):
            nout = (case["nsamp"] >> k) - int(_delays(fr, dms[e - 1:e], ts * 2 ** k).max())
            b += 4 * (e - a) * nout
            fl += (e - a) * case["nchan"] * nout
        return {"bytes": b, "flops": fl}
    if kind == "subband":
        subs, groups, _, d2, len1 = _subband_geometry(case)
        fl = len(groups) * case["nchan"] * len1
        b = 4 * case["nchan"] * case["nsamp"]
        for a, e in groups:
            nout = len1 - int(d2[:, a:e].max())
            fl += (e - a) * len(subs) * nout
            b += 4 * (e - a) * nout
        return {"bytes": b, "flops": fl}
    if kind == "rfi":
        n = case["nchan"] * case["nsamp"]
        return {"bytes": 2 * n * BYTES[case["dtype"]], "flops": 4 * n}
    n = case["nrows"] * case["n"]
    return {"bytes": 8 * n, "flops": n * (6 + 2 * case["max_log2"])}


# ---------------------------------------------------------------- the result in 64 bits

def _dedisperse64(x, delays, nout):
    acc = torch.zeros((delays.shape[1], nout), dtype=torch.float64, device=x.device)
    idx = torch.from_numpy(delays).to(x.device)
    for c in range(x.shape[0]):
        acc += x[c].to(torch.float64).unfold(0, nout, 1).index_select(0, idx[c])
    return acc


def _with_stats(out):
    mean = out.mean(dim=1)
    rms = torch.empty_like(mean)
    for i in range(0, out.shape[0], 64):
        rms[i:i + 64] = ((out[i:i + 64] - mean[i:i + 64, None]) ** 2).mean(dim=1).sqrt()
    return {"out": out, "mean": mean, "rms": rms}


_NO_EVENTS = {"dm_index": None, "t": None, "value": None, "snr": None}
_NO_PULSES = {"row": None, "width": None, "t": None, "value": None, "snr": None}


def exact(case, seed):
    kind = case["kind"]
    if work(case)["flops"] > EXACT_ADDS and kind in ("plain", "stream", "serving", "binned", "subband"):
        return None
    gen = torch.Generator(device=DEV)
    gen.manual_seed(int(seed))
    if kind == "search":
        x = _series(case, gen).to(torch.float64)
        t = torch.arange(case["n"], dtype=torch.float64, device=DEV) - (case["n"] - 1) / 2.0
        x -= x.mean(dim=1, keepdim=True)
        x -= ((x @ t) / (t @ t))[:, None] * t[None, :]
        rms = (x * x).mean(dim=1).sqrt()
        return {"series": x / rms[:, None], "rms": rms, "pulses": _NO_PULSES}
    if kind == "rfi":
        return _rfi64(case, _rfi_input(case, gen))
    if kind == "serving":
        res = []
        for band, nchan, ndm, step, block in _serving_beams(case):
            b = _noise(nchan, block, "u8", gen)
            res.append(dict(_stream64(b, _delays(_freq(band, nchan), _dms(ndm, step), BANDS[band][2])), ncand=None))
        return res
    f, dms, ts = _freq(case["band"], case["nchan"]), _dms(case["ndm"], case["step"]), BANDS[case["band"]][2]
    if kind == "stream":
        b = _noise(case["nchan"], case["block"], case["dtype"], gen)
        return dict(_stream64(b, _delays(f, dms, ts)), ncand=None)
    x = _filterbank(case, case["nsamp"], gen)
    if kind == "plain":
        d = _delays(f, dms, ts)
        return dict(_with_stats(_dedisperse64(x, d, case["nsamp"] - int(d.max()))), cands=_NO_EVENTS)
    if kind == "binned":
        runs, cur, lvl = [], 0, x.to(torch.float64)
        for k, a, e in _binned_runs(case):
            while cur < k:
                m = lvl.shape[1] // 2
                lvl = lvl[:, 0:2 * m:2] + lvl[:, 1:2 * m:2]
                cur += 1
            d = _delays(f, dms[a:e], ts * 2 ** k)
            runs.append(_with_stats(_dedisperse64(lvl, d, lvl.shape[1] - int(d.max()))))
        return {"runs": runs, "cands": _NO_EVENTS}
    subs, groups, d1, d2, len1 = _subband_geometry(case)
    red = torch.stack([_dedisperse64(x[a:b], d, len1) for (a, b), d in zip(subs, d1)])
    res = []
    for g, (a, e) in enumerate(groups):
        d = d2[:, a:e]
        res.append(_with_stats(_dedisperse64(red[:, g], d, len1 - int(d.max()))))
    return {"out": [r["out"] for r in res], "mean": torch.cat([r["mean"] for r in res]),
            "rms": torch.cat([r["rms"] for r in res])}


def _stream64(block, delays):
    """The window of a stream whose every block is `block`, once its ring is full: the last
    block of outputs, starting maxdelay samples before the end of a period."""
    n = block.shape[1]
    maxd = int(delays.max())
    start = (delays - maxd) % n
    ext = torch.cat([block, block], dim=1)
    return _with_stats(_dedisperse64(ext, start, n))


def _rfi64(case, raw):
    u8 = case["dtype"] == "u8"
    x = raw.to(torch.float64)
    nchan, n = x.shape
    w = case["window"]
    avg = x.mean(dim=1).cpu().numpy()
    c = np.linspace(-1.0, 1.0, nchan)
    q, _ = np.linalg.qr(np.polynomial.chebyshev.chebvander(c, case["order"]))
    fit = q @ (q.T @ avg)
    fmean = float(fit.mean())
    ft = torch.from_numpy(fit).to(x.device)[:, None]
    rep = torch.clamp(torch.floor(ft + 0.5), 0, 255) if u8 else ft.to(torch.float32).to(torch.float64)
    full = n // w
    means = x[:, :full * w].reshape(nchan, full, w).mean(dim=2)
    if full * w < n:
        means = torch.cat([means, x[:, full * w:].mean(dim=1, keepdim=True)], dim=1)
    flag = (means - ft).abs() > 12.0
    hit = flag.clone()
    hit[:, 1:] |= flag[:, :-1]
    hit[:, :-1] |= flag[:, 1:]
    mask = hit.repeat_interleave(w, dim=1)[:, :n]
    x = torch.where(mask, rep, x)
    spec = (x.mean(dim=0) - fmean).abs() > 6.0
    x = torch.where(spec[None, :], rep, x)
    data = x.to(torch.uint8) if u8 else x - rep
    return {"data": data, "fit": fit, "rmse": float(np.sqrt(np.mean((fit - avg) ** 2))), "fit_mean": fmean,
            "flags": flag.to(torch.int32)}
