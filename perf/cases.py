"""Workloads of the search for performance work, each through the public calls.

A case is a dict of plain values whose "kind" names the call it makes:

  search      Plan.search of one series or spectrum (FFT or 16-bit matrix correlator, plain or half-bin plane)
  batch       Plan.search_batch of several series of mixed lengths
  td          TdPlan.search, the time-domain resampling search
  dedisperse  dedisperse of a filterbank to one series per DM
  refine      Plan.refine of chosen candidate records

Inputs are white noise with a few weak drifting pulsars, as nearly all trials
of a survey are: tens to some hundreds of candidates, not a bright pulsar's
hundreds of thousands.  Records come back in a buffer of the program's own, of
RECORDS entries and zero after the ones found.
"""
import functools
import math
import random

import numpy as np
import torch

import paper_1511_07343_amd as fdas

DEV = "cuda"
K_DM = 4.148808e3  # s MHz^2 pc^-1 cm^3
RECORDS = 1 << 14


# ------------------------------------------------------------------ the cases
def _search(name, log2n, zmax, nz, seg, nharm, window=1024, sigma=6.0, source="series", corr="fft", interbin=False,
            pinned=True, plane=False):
    c = {"kind": "search", "log2n": log2n, "zmax": zmax, "nz": nz, "seg": seg, "nharm": nharm, "window": window,
         "sigma": sigma, "source": source, "corr": corr, "interbin": interbin, "pinned": pinned, "plane": plane}
    return dict(c, name=name) if name else c


def _dedisperse(name, nchan, ndm, nout, f_top, band, tsamp, dm_max):
    c = {"kind": "dedisperse", "nchan": nchan, "ndm": ndm, "nout": nout, "f_top": f_top, "band": band, "tsamp": tsamp,
         "dm_max": dm_max}
    return dict(c, name=name) if name else c


def listed():
    return [
        # the smallest call: a short series, few templates, records into ordinary memory (launch latency counts)
        _search("tiny", 15, 20.0, 21, 512, 4, window=512, sigma=5.5, pinned=False),
        # the small search of the benchmark: 2^17 samples, 101 templates, powers only
        _search("small", 17, 100.0, 101, 2048, 1),
        # the named SKA-shaped trial: 2^23 samples, 201 templates, 16 harmonics
        _search("ska_trial", 23, 200.0, 201, 8192, 16),
        # a fine bank over a wide drift range, powers only, in the default precision
        _search("fine_bank", 22, 400.0, 801, 8192, 1),
        # the same bank through the 16-bit matrix correlator (as in all its cases, the plane is kept: near a
        # threshold its candidates differ from those of a plane in full precision)
        _search("fine_bank_bf16", 22, 400.0, 801, 8192, 1, corr="bf16", plane=True),
        # the half-bin plane, which keeps more of a tone between two bins
        _search("half_bin", 21, 200.0, 201, 4096, 8, interbin=True),
        # a spectrum from elsewhere, an even number of templates and the plane kept for inspection
        _search("spectrum_plane", 20, 64.0, 160, 1024, 8, window=512, source="spectrum", plane=True),
        # an observation's trials of mixed lengths in one call, resident in HBM
        {"name": "batch", "kind": "batch", "log2n": 22, "lengths": "22,21,22,20,22,21", "zmax": 200.0, "nz": 201,
         "seg": 2048, "nharm": 16, "sigma": 6.0},
        # the time-domain search of a short series
        {"name": "time_domain", "kind": "td", "log2n": 20, "alpha_max": 0.02, "nalpha": 101, "nharm": 16, "sigma": 6.0,
         "window": 1024},
        # the front end at the benchmark's size: 64 channels to 256 DM trials of 2^23 samples
        _dedisperse("dedisperse_beam", 64, 256, 1 << 23, 1500.0, 300.0, 64e-6, 500.0),
        # a short odd-sized filterbank with many channels
        _dedisperse("dedisperse_odd", 257, 33, 60001, 1450.0, 300.0, 256e-6, 300.0),
        # the most significant records of a search moved off the grid
        {"name": "refine", "kind": "refine", "log2n": 21, "zmax": 200.0, "nz": 201, "seg": 8192, "records": 256,
         "levels": 6},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _templates(rng, zmax, low, high):
    """Template counts of drift steps from half a bin up."""
    return _log_int(rng, low, max(low + 1, min(high, int(4 * zmax) + 1)))


def _bank_and_seg(rng, most_z):
    zmax = rng.choice([z for z in (8.0, 20.0, 50.0, 100.0, 200.0, 301.0, 400.0) if z <= most_z])
    h = math.ceil(zmax / 2) + 16
    return zmax, rng.choice([s for s in (256, 512, 1024, 2048, 4096, 8192) if s >= 4 * h])


def draw(rng):
    kind = rng.choice(["search", "search", "search", "matrix", "half_bin", "batch", "td", "dedisperse", "dedisperse",
                       "refine"])
    nharm, window = rng.choice([1, 2, 4, 8, 16]), rng.choice([256, 512, 1024, 2048])
    sigma = round(rng.uniform(5.5, 7.0), 2)
    if kind == "search":
        log2n = rng.randint(14, 23)
        zmax, seg = _bank_and_seg(rng, 400.0)
        nz = _templates(rng, zmax, 11, min(801, 201 << (23 - log2n)))
        source = rng.choice(["series", "series", "spectrum"])
        return _search(None, log2n, zmax, nz, seg, nharm, window, sigma, source, pinned=rng.random() < 0.5,
                       plane=log2n <= 20 and rng.random() < 0.3)
    if kind == "matrix":
        log2n = rng.randint(17, 22)
        zmax, seg = _bank_and_seg(rng, 400.0)
        return _search(None, log2n, zmax, _templates(rng, zmax, 21, 801), seg, nharm, window, sigma,
                       corr=rng.choice(["bf16", "f16"]), plane=True)
    if kind == "half_bin":
        log2n = rng.randint(16, 22)
        zmax, seg = _bank_and_seg(rng, 200.0)
        return _search(None, log2n, zmax, _templates(rng, zmax, 21, 201), seg, nharm, window, sigma, interbin=True)
    if kind == "batch":
        log2n = rng.randint(17, 22)
        zmax, seg = _bank_and_seg(rng, 200.0)
        lens = [log2n] + [rng.randint(max(15, log2n - 3), log2n) for _ in range(rng.randint(1, 7))]
        return {"kind": "batch", "log2n": log2n, "lengths": ",".join(map(str, lens)), "zmax": zmax,
                "nz": _templates(rng, zmax, 21, 201), "seg": seg, "nharm": nharm, "sigma": sigma}
    if kind == "td":
        log2n = rng.randint(14, 23)
        return {"kind": "td", "log2n": log2n, "alpha_max": round(rng.uniform(0.001, 0.05), 5),
                "nalpha": _log_int(rng, 5, min(201, 101 << max(0, 23 - log2n))), "nharm": nharm, "sigma": sigma,
                "window": window}
    if kind == "dedisperse":
        nchan, ndm = _log_int(rng, 8, 512), _log_int(rng, 1, 256)
        nout = _log_int(rng, 1 << 14, min(1 << 23, (64 * 256 << 23) // (nchan * ndm)))
        if rng.random() < 0.5:
            nout = 1 << (nout.bit_length() - 1)
        f_top = rng.choice([400.0, 800.0, 1450.0])
        return _dedisperse(None, nchan, ndm, nout, f_top, round(f_top * rng.uniform(0.05, 0.3), 3),
                           rng.choice([64e-6, 256e-6, 512e-6]), round(rng.uniform(20.0, 500.0), 1))
    zmax, seg = _bank_and_seg(rng, 200.0)
    return {"kind": "refine", "log2n": rng.randint(16, 22), "zmax": zmax, "nz": _templates(rng, zmax, 21, 201), "seg": seg,
            "records": _log_int(rng, 3, 400), "levels": rng.randint(2, 8)}


# ------------------------------------------------------------------ inputs
def _gen(seed):
    return torch.Generator(device=DEV).manual_seed(int(seed))


def _series(log2n, zmax, seed, pulsars=2, top=8, alphas=None):
    """White noise of unit variance and `pulsars` weak drifting pulsars, with
    drifts in bins up to zmax, or of relative drifts from alphas."""
    n = 1 << log2n
    x = torch.randn(n, generator=_gen(seed), device=DEV, dtype=torch.float32).double()
    rng = random.Random(seed * 7919 + log2n)
    u = torch.arange(n, device=DEV, dtype=torch.float64) / n
    for _ in range(pulsars):
        nharm = rng.choice([1, 2, 4, top])
        r = rng.uniform(0.02, 0.45 / nharm) * n / 2
        z = rng.uniform(-0.9, 0.9) * zmax / nharm if alphas is None else rng.choice(list(alphas)) * r
        amp = 2.0 * math.sqrt(rng.uniform(40.0, 70.0) / n)  # a tone of this amplitude has power 40 .. 70
        cycles = torch.remainder(rng.random() + (r - z / 2) * u + z * u * u / 2, 1.0)
        for j in range(1, nharm + 1):
            x += amp * torch.cos(2 * math.pi * torch.remainder(j * cycles, 1.0))
    return x.float()


def _alphas(c):
    return -c["alpha_max"] + np.arange(c["nalpha"]) * (2 * c["alpha_max"] / (c["nalpha"] - 1))


def _spectrum(x):
    X = torch.fft.rfft(x.double())[:-1].clone()
    X[0] = 0
    return X.to(torch.complex64)


def _records(c, seed):
    """Records as a search reports them: cells of harmonic sums over the whole plane."""
    rng = np.random.default_rng(seed)
    n, nb = c["records"], 1 << (c["log2n"] - 1)
    rec = np.zeros(n, dtype=fdas.CAND_DTYPE)
    rec["nharm"] = rng.choice([1, 2, 4, 8, 16], n)
    rec["k"] = rng.integers(nb // 50, nb - 400, n)
    rec["iz"] = rng.integers(0, c["nz"], n)
    rec["r"] = rec["k"] / rec["nharm"]
    rec["z"] = (-c["zmax"] + rec["iz"] * (2 * c["zmax"] / (c["nz"] - 1))) / rec["nharm"]
    return rec


def _delays(c):
    f = c["f_top"] - (c["band"] / c["nchan"]) * np.arange(c["nchan"])
    dms = np.linspace(0.0, c["dm_max"], c["ndm"]) if c["ndm"] > 1 else np.array([c["dm_max"]])
    lag = K_DM * dms[:, None] * (1.0 / (f * f) - 1.0 / (c["f_top"] * c["f_top"])) / c["tsamp"]
    return dms, np.floor(lag + 0.5).astype(np.int64)


def _filterbank(c, seed):
    _, d = _delays(c)
    nsamp = c["nout"] + int(d.max())
    g = torch.randn((c["nchan"], nsamp), generator=_gen(seed), device=DEV, dtype=torch.float32)
    return g.mul_(16.0).add_(128.0).round_().clamp_(0, 255).to(torch.uint8)


def _buffer(records, pinned=True):
    out = fdas.pinned_candidates(records) if pinned else np.empty(records, dtype=fdas.CAND_DTYPE)
    out[:] = np.zeros((), dtype=fdas.CAND_DTYPE)
    return out


def _plan(c, **more):
    bank = fdas.make_templates(c["zmax"], 2 * c["zmax"] / (c["nz"] - 1))
    return fdas.Plan(bank, 1 << c["log2n"], c["seg"], **more)


def prepare(case, seed):
    c = case
    if c["kind"] == "search":
        s = {"case": c, "out": _buffer(RECORDS, c["pinned"]), "plane": None}
        s["plan"] = _plan(c, nharm_max=c["nharm"], sigma=c["sigma"], median_window=c["window"], correlator=c["corr"],
                          interbin=c["interbin"])
        x = _series(c["log2n"], c["zmax"], seed)
        s["in"] = x if c["source"] == "series" else _spectrum(x)
        s["in_kind"] = fdas.IN_SERIES if c["source"] == "series" else fdas.IN_SPECTRUM
        if c["plane"]:
            s["plane"] = torch.empty((c["nz"], s["plan"].plane_columns), dtype=torch.float32, device=DEV)
        return s
    if c["kind"] == "batch":
        lens = [int(v) for v in c["lengths"].split(",")]
        return {"case": c, "plan": _plan(c, nharm_max=c["nharm"], sigma=c["sigma"]), "caps": [RECORDS] * len(lens),
                "series": [_series(v, c["zmax"], seed + 1000 * i, pulsars=i % 3) for i, v in enumerate(lens)],
                "out": _buffer(RECORDS * len(lens))}
    if c["kind"] == "td":
        return {"case": c, "in": _series(c["log2n"], 0.0, seed, alphas=_alphas(c)),
                "plan": fdas.TdPlan(1 << c["log2n"], c["alpha_max"], c["nalpha"], nharm_max=c["nharm"],
                                    sigma=c["sigma"], median_window=c["window"]),
                "out": _buffer(RECORDS)}
    if c["kind"] == "dedisperse":
        return {"case": c, "fil": _filterbank(c, seed), "dms": _delays(c)[0],
                "out": torch.empty((c["ndm"], c["nout"]), dtype=torch.float32, device=DEV)}
    s = {"case": c, "plan": _plan(c, nharm_max=16, sigma=8.0), "in": _spectrum(_series(c["log2n"], c["zmax"], seed)),
         "rec": _records(c, seed)}
    s["plan"].search(s["in"], kind=fdas.IN_SPECTRUM, cap=1 << 16)
    return s


# ------------------------------------------------------------------ one pass
def _fields(rec):
    return {f: rec[f] for f in fdas.CAND_DTYPE.names}


def run(state):
    s, c = state, state["case"]
    if c["kind"] == "search":
        found = s["plan"].search(s["in"], kind=s["in_kind"], plane=s["plane"], out=s["out"])[1]
        return {"found": found, "candidates": _fields(s["out"]), "plane": s["plane"]}
    if c["kind"] == "batch":
        found = [len(r) for r in s["plan"].search_batch(s["series"], caps=s["caps"], out=s["out"])]
        return {"found": found, "candidates": _fields(s["out"])}
    if c["kind"] == "td":
        found = s["plan"].search(s["in"], out=s["out"])[1]
        return {"found": found, "candidates": _fields(s["out"])}
    if c["kind"] == "dedisperse":
        return fdas.dedisperse(s["fil"], c["f_top"], c["band"] / c["nchan"], c["tsamp"], s["dms"], c["nout"],
                               out=s["out"])
    return _fields(s["plan"].refine(s["rec"], c["levels"]))


def work(case):
    c = case
    if c["kind"] == "dedisperse":
        nsamp = c["nout"] + int(_delays(c)[1].max())
        return {"bytes": c["nchan"] * nsamp + 4 * c["ndm"] * c["nout"], "flops": c["ndm"] * c["nchan"] * c["nout"]}
    n = 1 << c["log2n"]
    if c["kind"] == "td":
        per = 2.5 * n * c["log2n"] + 8 * n + (n / 2) * (3 + c["nharm"])
        return {"bytes": 4 * n, "flops": c["nalpha"] * per}
    taps = 2 * (math.ceil(c["zmax"] / 2) + 16) + 1
    if c["kind"] == "refine":  # two Fresnel integrals of ~40 operations and the sums per response
        nh = 31 / 5
        return {"bytes": c["records"] * (taps + 2) * 16 * 8 * nh, "flops": c["records"] * (1 + 8 * c["levels"]) * nh * taps * 100}
    if c["kind"] == "batch":
        lens = [1 << int(v) for v in c["lengths"].split(",")]
    else:
        lens = [n]
    cpb = 2 if c.get("interbin") else 1
    flops = 0.0
    for m in lens:
        nb = m / 2
        if c.get("corr", "fft") == "fft":
            valid = c["seg"] - taps + 1
            corr = cpb * c["nz"] * nb / valid * (c["seg"] * (5 * math.log2(c["seg"]) + 6) + 3 * valid)
        else:
            corr = c["nz"] * nb * (4 * taps + 3)
        flops += corr + cpb * c["nz"] * nb * (c["nharm"] - 1) + 2.5 * m * math.log2(m)
    got = 4 * sum(lens) + (4 * c["nz"] * n // 2 * cpb if c.get("plane") else 0)
    return {"bytes": got, "flops": flops}


# ------------------------------------------------------------------ the same in 64 bits
@functools.lru_cache(maxsize=4)
def _nodes(m):
    x, w = np.polynomial.legendre.leggauss(m)
    return (torch.from_numpy((x + 1) / 2).to(DEV), torch.from_numpy(w / 2).to(DEV))


def _cis(turns):
    t = 2 * math.pi * torch.remainder(turns, 1.0)
    return torch.complex(torch.cos(t), torch.sin(t))


def _response(base, z, h):
    """A(base - t, z) for t = 0 .. 2h, one row per (base, z), by quadrature of the defining integral."""
    u, w = _nodes(1024)
    lead = _cis(base[:, None] * u + z[:, None] * (u * u - u) / 2) * w
    steps = torch.arange(2 * h + 1, device=DEV, dtype=torch.float64)
    return lead @ _cis(-u[:, None] * steps)


def _medians(power, window):
    nb = power.numel()
    nblk = -(-nb // window)
    s = torch.sort(power.reshape(nblk, window), dim=1).values  # both are powers of two
    med = 0.5 * (s[:, (window - 1) // 2] + s[:, window // 2])
    x = torch.arange(nb, device=DEV, dtype=torch.float64)
    pos = ((x - 0.5 * (window - 1)) / window).clamp(0, nblk - 1)
    b = pos.floor().long().clamp(max=max(nblk - 2, 0))
    return med[b] + (med[(b + 1).clamp(max=nblk - 1)] - med[b]) * (pos - b)


def _normalised(x, window):
    X = (torch.fft.rfft(x.double())[:-1].clone() if not x.is_complex() else x.to(torch.complex128))
    if not x.is_complex():
        X[0] = 0
    return X * torch.sqrt(math.log(2.0) / _medians(X.abs().square(), window))


def _plane(X, zmax, nz, half):
    """|sum_q X[k - q] T_z[q]|^2 per template, over the bins (half: and the points between them)."""
    nb, h = X.numel(), math.ceil(zmax / 2) + 16
    z = torch.from_numpy(-zmax + np.arange(nz) * (2 * zmax / (nz - 1))).to(DEV)
    size = nb + nb // 4
    F = torch.fft.fft(X, size)
    P = torch.empty((nz, nb, 2 if half else 1), dtype=torch.float64, device=DEV)
    for part in range(P.shape[2]):
        # column t holds offset q = h - t (half: q + 1/2 with q = h - 1 - t, 2h of them)
        A = _response(torch.full((nz,), h - 0.5 if part else float(h), dtype=torch.float64, device=DEV), z, h)
        if part:
            A = A[:, :-1]
        T = (A.conj() / A.abs().square().sum(1, keepdim=True).sqrt()).flip(1)  # ascending q from -h
        for i in range(nz):
            Y = torch.fft.ifft(F * torch.fft.fft(T[i], size))
            P[i, :, part] = Y.roll(-h)[:nb].abs().square()  # Y[m] = sum over q of X[m - h - q]
    return P.reshape(nz, -1)


def _thr(sigma, nh):
    target = math.log(0.5 * math.erfc(sigma / math.sqrt(2)))
    lo, hi = 0.0, 4000.0
    for _ in range(200):
        mid = 0.5 * (lo + hi)
        lo, hi = (mid, hi) if _log_q(nh, mid) > target else (lo, mid)
    return lo


def _log_q(n, s):
    terms = [i * math.log(s) - math.lgamma(i + 1) if s > 0 else (0.0 if i == 0 else -math.inf) for i in range(n)]
    top = max(terms)
    return -s + top + math.log(sum(math.exp(t - top) for t in terms))


def _log_tail(x):
    if x < 25.0:
        return math.log(0.5 * math.erfc(x / math.sqrt(2)))
    y = 1 / (x * x)
    return -0.5 * x * x - math.log(x * math.sqrt(2 * math.pi)) + math.log1p(-y + 3 * y**2 - 15 * y**3 + 105 * y**4)


def _sigma(power, nh):
    target, lo, hi = _log_q(nh, power), -40.0, math.sqrt(2 * power) + 50.0
    for _ in range(80):
        mid = 0.5 * (lo + hi)
        lo, hi = (mid, hi) if _log_tail(mid) > target else (lo, mid)
    return lo


def _candidates(P, izc, nharm, sigma, half):
    """Thresholded 3x3 maxima of the harmonic sums: {k, iz, nharm, power}, sorted."""
    nz, ncol = P.shape
    k = torch.arange(ncol, device=DEV)
    S = P.clone()
    got = {"k": [], "iz": [], "nharm": [], "power": []}
    nh = 1
    while True:
        if nh > 1:
            for j in range(16 // nh, 16, 32 // nh):
                col = (j * k + 8) >> 4
                for iz in range(nz):
                    d = iz - izc
                    row = iz if izc < 0 else izc + (1 if d > 0 else -1) * ((abs(d) * j + 8) >> 4)
                    S[iz] += P[row].index_select(0, col)
        at = torch.nonzero(S >= _thr(sigma, nh))
        if at.numel():
            iz, kk = at[:, 0], at[:, 1]
            v, keep = S[iz, kk], torch.ones(at.shape[0], dtype=torch.bool, device=DEV)
            for n in range(9):
                di, dk = n // 3 - 1, n % 3 - 1
                if n == 4:
                    continue
                inside = (iz + di >= 0) & (iz + di < nz) & (kk + dk >= 0) & (kk + dk < ncol)
                other = S[(iz + di).clamp(0, nz - 1), (kk + dk).clamp(0, ncol - 1)]
                keep &= ~inside | ((v > other) if n < 4 else (v >= other))
            iz, kk, v = iz[keep].cpu().numpy(), kk[keep].cpu().numpy(), v[keep].cpu().numpy()
            order = np.lexsort((iz, kk))
            got["k"].append(kk[order])
            got["iz"].append(iz[order].astype(np.int32))
            got["nharm"].append(np.full(len(order), nh, dtype=np.int32))
            got["power"].append(v[order])
        if nh == nharm:
            break
        nh *= 2
    out = {f: np.concatenate(v) if v else np.zeros(0) for f, v in got.items()}
    out["r"] = out["k"] / np.maximum(out["nharm"] * (2 if half else 1), 1)
    out["sigma"] = np.array([_sigma(float(p), int(m)) for p, m in zip(out["power"], out["nharm"])])
    return out


def _with_drift(rec, value, td):
    v = value[rec["iz"].astype(np.int64)] if len(rec["k"]) else np.zeros(0)
    rec["z"] = v * rec["r"] if td else v / np.maximum(rec["nharm"], 1)
    return rec


def _found(recs):
    """What run() returns for the records of one search (a dict of fields) or of a batch (a list of them)."""
    many = recs if isinstance(recs, list) else [recs]
    n = [len(r["k"]) for r in many]
    out = {f: np.zeros((len(many), RECORDS), dtype=fdas.CAND_DTYPE[f] if fdas.CAND_DTYPE[f].kind == "i" else np.float64)
           for f in fdas.CAND_DTYPE.names}
    for i, r in enumerate(many):
        for f in out:
            out[f][i, :n[i]] = r[f]
    return {"found": n if isinstance(recs, list) else n[0], "candidates": {f: v.reshape(-1) for f, v in out.items()}}


def _exact_search(x, c, nharm, window, half=False):
    P = _plane(_normalised(x, window), c["zmax"], c["nz"], half)
    rec = _candidates(P, (c["nz"] - 1) // 2, nharm, c["sigma"], half)
    return _with_drift(rec, -c["zmax"] + np.arange(c["nz"]) * (2 * c["zmax"] / (c["nz"] - 1)), False), P


def _exact_refine(X, c, rec):
    nb, h = X.numel(), math.ceil(c["zmax"] / 2) + 16
    dz, izc = 2 * c["zmax"] / (c["nz"] - 1), (c["nz"] - 1) // 2
    t = torch.arange(2 * h + 1, device=DEV, dtype=torch.float64)

    def power(r, z):
        first = torch.ceil(r - h)
        A = _response(r - first, z, h) * (t <= (torch.floor(r + h) - first)[:, None])
        k = (first[:, None] + t).long()
        Xk = torch.where((k >= 0) & (k < nb), X[k.clamp(0, nb - 1)], torch.zeros((), dtype=X.dtype, device=DEV))
        return (Xk * A.conj()).sum(1).abs().square() / A.abs().square().sum(1)

    out = {f: np.array(rec[f], dtype=np.float64) for f in ("r", "z", "power", "sigma")}
    for nh in (1, 2, 4, 8, 16):
        at = np.nonzero(rec["nharm"] == nh)[0]
        if not len(at):
            continue
        j = torch.arange(1, nh + 1, device=DEV, dtype=torch.float64)

        def total(r, z):
            return power((r.reshape(-1, 1) * j).reshape(-1), (z.reshape(-1, 1) * j).reshape(-1)).reshape(*r.shape, nh).sum(-1)

        r = torch.from_numpy(rec["k"][at] / nh).to(DEV)
        z = torch.from_numpy(((rec["iz"][at] - izc) * dz) / nh).to(DEV)
        best = total(r, z)
        for level in range(1, c["levels"] + 1):
            sr, sz = 2.0**-level / nh, dz * 2.0**-level / nh
            a = torch.tensor([-1, 0, 1, -1, 1, -1, 0, 1], device=DEV, dtype=torch.float64)
            b = torch.tensor([-1, -1, -1, 0, 0, 1, 1, 1], device=DEV, dtype=torch.float64)
            rr, zz = r[:, None] + a * sr, z[:, None] + b * sz
            S = torch.where((nh * zz).abs() > c["zmax"], torch.full_like(rr, -1.0), total(rr, zz))
            top, i = S.max(1)
            move = top > best
            r = torch.where(move, rr.gather(1, i[:, None])[:, 0], r)
            z = torch.where(move, zz.gather(1, i[:, None])[:, 0], z)
            best = torch.where(move, top, best)
        out["r"][at], out["z"][at], out["power"][at] = r.cpu().numpy(), z.cpu().numpy(), best.cpu().numpy()
        out["sigma"][at] = [_sigma(float(p), nh) for p in out["power"][at]]
    return dict(out, k=rec["k"], iz=rec["iz"], nharm=rec["nharm"])


def exact(case, seed):
    c = case
    if c["kind"] == "dedisperse":
        fil, (_, d) = _filterbank(c, seed), _delays(c)
        out = torch.empty((c["ndm"], c["nout"]), dtype=torch.float64, device=DEV)
        for i in range(c["ndm"]):
            acc = torch.zeros(c["nout"], dtype=torch.int32, device=DEV)
            for ch in range(c["nchan"]):
                acc += fil[ch, int(d[i, ch]):int(d[i, ch]) + c["nout"]]
            out[i] = acc
        return out
    if c["kind"] == "search":
        x = _series(c["log2n"], c["zmax"], seed)
        rec, P = _exact_search(x if c["source"] == "series" else _spectrum(x), c, c["nharm"], c["window"], c["interbin"])
        if c["corr"] != "fft":
            return {"found": None, "candidates": None, "plane": P}
        return dict(_found(rec), plane=P if c["plane"] else None)
    if c["kind"] == "batch":
        return _found([_exact_search(_series(int(v), c["zmax"], seed + 1000 * i, pulsars=i % 3), c, c["nharm"], 1024)[0]
                       for i, v in enumerate(c["lengths"].split(","))])
    if c["kind"] == "td":
        n = 1 << c["log2n"]
        x = _series(c["log2n"], 0.0, seed, alphas=_alphas(c)).double()
        x1 = torch.cat([x[1:], torch.zeros(1, dtype=x.dtype, device=DEV)])
        tau = torch.arange(n, device=DEV, dtype=torch.float64) / n - 0.5
        alphas = _alphas(c)
        P = torch.empty((c["nalpha"], n // 2), dtype=torch.float64, device=DEV)
        for i, al in enumerate(alphas):
            pos = n * (2 * tau / (1 + torch.sqrt(1 + 2 * al * tau)) + 0.5)
            at = pos.floor()
            inside = (at >= 0) & (at <= n - 1)
            at_i = at.clamp(0, n - 1).long()
            y = torch.where(inside, x[at_i] * (1 - (pos - at)) + x1[at_i] * (pos - at), torch.zeros_like(pos))
            P[i] = _normalised(y, c["window"]).abs().square()
        return _found(_with_drift(_candidates(P, -1, c["nharm"], c["sigma"], False), alphas, True))
    X = _normalised(_spectrum(_series(c["log2n"], c["zmax"], seed)), 1024)
    return _exact_refine(X, c, _records(c, seed))
