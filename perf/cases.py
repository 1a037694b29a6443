"""Cases that stand for the work users have this framework do, each through its
public entry points (``paper_1611_09704_amd.binding``).

Kinds of case and what they stand for:

* ``detect``  one de-dispersed plane through ``spd_detect``: statistics,
              boxcars, per-sample SNR and width, candidate count.  ``pad``
              says whether the caller pads its output rows to 64 bytes or
              takes plain contiguous arrays.
* ``chunk``   one chunk of a running stream on the device: ``msd_compute``
              merged into the carried state, then ``boxcar_snr`` for the
              candidates alone, fetched to the host.
* ``dit``     statistics plus the decimated search (``boxcar_snr_dit``).
* ``peaks``   ``select_candidates`` over stored outputs, then
              ``cluster_candidates``; the peaks are fetched to the host.
* ``dedisp``  ``DedispPlan.run``: an 8-bit filterbank to the DM x time plane.
* ``batch``   a ``BatchPlan`` over uneven beams, replayed as a graph, its
              candidates fetched to the host.
* ``serve``   a ``Server`` fed chunks from host memory until every result is
              back (the whole call: copies, statistics, search, candidates);
              with ``dms`` the chunks are 8-bit filterbanks, de-dispersed on
              the device first.

A candidate list is unordered by contract; where a case returns one, it is in
the host's hands by then and is put, in order of beam, row and time, into a
table of fixed length (zeros past the last).  The
``detect`` and ``dit`` cases return the SNR and width planes, which hold every
candidate, and the count.
"""
import math

import numpy as np
import torch

from paper_1611_09704_amd import binding as B
from paper_1611_09704_amd import synth

DTYPES = {"f32": torch.float32, "f16": torch.float16, "u8": torch.uint8}
ELEM = {"f32": 4, "f16": 2, "u8": 1}
CAPACITY = 1 << 18
TABLE = 1 << 15             # entries of the host's candidate table
SAMPLE_S = 64e-6


def widths_of(case):
    """"1..n", "ska" (1..16, then 18..256 step 2) or the decimated search's list."""
    if case["kind"] == "dit":
        return B.dit_widths(case["levels"])
    return list(synth.SKA_WIDTHS) if case["widths"] == "ska" else list(range(1, int(case["widths"].split("..")[1]) + 1))


def listed():
    return [
        # the smallest ordinary call: a handful of trials, where launches and latency count
        dict(name="detect-64x65536-f32-w32", kind="detect", rows=64, cols=65536, dtype="f32", widths="1..32",
             sigma="sqrtn", pad=False),
        # the headline workload: an SKA-like plane, 136 widths, signal-dominated rows
        dict(name="detect-4096x2^20-f32-ska", kind="detect", rows=4096, cols=1 << 20, dtype="f32", widths="ska",
             sigma="auto", pad=True),
        # the paper's measured setting (widest boxcar 16) on a plane as de-dispersion leaves it: an odd
        # number of columns, contiguous rows
        dict(name="detect-2048x524281-f32-w16", kind="detect", rows=2048, cols=524281, dtype="f32", widths="1..16",
             sigma="auto", pad=False),
        # 8-bit storage with per-row scale, plain contiguous outputs
        dict(name="detect-1024x262144-u8-w64", kind="detect", rows=1024, cols=262144, dtype="u8", widths="1..64",
             sigma="auto", pad=False),
        # one 8.4 s chunk of a beam's FP16 stream with its 255-sample halo, widths 1..256
        dict(name="chunk-1024x131072-f16-w256", kind="chunk", rows=1024, cols=131072, dtype="f16", widths="1..256",
             sigma="auto"),
        # the decimated search up to width 256
        dict(name="dit-2048x2^19-f32", kind="dit", rows=2048, cols=1 << 19, dtype="f32", levels=4, sigma="auto",
             pad=True),
        # a stored SNR plane thresholded again and reduced to its peaks
        dict(name="peaks-1024x262144", kind="peaks", rows=1024, cols=262144, bumps=400, dm_radius=2, t_radius=256),
        # de-dispersion at survey size: 4,096 channels, 6,000 trials, 8.4 s of 64 us samples
        dict(name="dedisp-4096ch-6000dm-2^17", kind="dedisp", chans=4096, dms=6000, samples=1 << 17, dm_step=1.0),
        # de-dispersion of a narrow search: few channels and trials, an odd length
        dict(name="dedisp-256ch-200dm-50001", kind="dedisp", chans=256, dms=200, samples=50001, dm_step=1.0),
        # uneven beams in one run, every shape filling the device by itself
        dict(name="batch-12-uneven-f32-w128", kind="batch", beams=12, rows=512, cols=1 << 18, dtype="f32",
             widths="1..128", sigma="sqrtn"),
        # many small beams, where one launch for all of them is what matters
        dict(name="batch-128-small-f32-w32", kind="batch", beams=128, rows=32, cols=16384, dtype="f32",
             widths="1..32", sigma="sqrtn"),
        # real-time serving from the filterbank on: 2 beams, 2 chunks each from pinned host memory
        dict(name="serve-2x1024ch-1000dm-w16", kind="serve", beams=2, rows=1024, cols=32768, chunks=2,
             widths="1..16", sigma="auto", dms=1000),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["detect", "detect", "detect", "chunk", "dit", "peaks", "dedisp", "dedisp", "batch", "serve"])
    widths = rng.choice(["1..8", "1..12", "1..16", "1..32", "1..64", "1..100", "1..128", "1..256", "ska"])
    sigma, dtype = rng.choice(["sqrtn", "auto"]), rng.choice(["f32", "f32", "f16", "u8"])
    pad = rng.random() < 0.5
    if kind in ("detect", "dit"):
        rows = _log(rng, 8, 4096)
        cols = _log(rng, 4096, min(1 << 20, (1 << 29) // rows))
        if rng.random() < 0.5:
            cols = max(1024, cols // 256 * 256)
        c = dict(kind=kind, rows=rows, cols=cols, dtype=dtype, sigma=sigma, pad=pad)
        return dict(c, levels=rng.randint(1, 4)) if kind == "dit" else dict(c, widths=widths)
    if kind == "chunk":
        return dict(kind=kind, rows=_log(rng, 64, 2048), cols=_log(rng, 4096, 131072),
                    dtype=rng.choice(["f16", "f32"]), widths=widths, sigma=sigma)
    if kind == "peaks":
        return dict(kind=kind, rows=_log(rng, 16, 2048), cols=_log(rng, 4096, 262144), bumps=_log(rng, 10, 1000),
                    dm_radius=rng.randint(0, 8), t_radius=_log(rng, 1, 1024))
    if kind == "dedisp":
        chans = _log(rng, 32, 4096)
        dms = _log(rng, 16, 6000)
        most = max(8192, min(1 << 17, 2 * 10 ** 12 // (chans * dms)))
        return dict(kind=kind, chans=chans, dms=dms, samples=dms * 2 + _log(rng, 4096, most),
                    dm_step=rng.choice([0.25, 0.5, 1.0, 1.0, 2.0]))
    if kind == "batch":
        return dict(kind=kind, beams=rng.randint(2, 64), rows=_log(rng, 8, 256), cols=1 << rng.randint(12, 16),
                    dtype=rng.choice(["f32", "f32", "f16"]), widths=widths, sigma=sigma)
    c = dict(kind=kind, beams=rng.randint(1, 6), rows=_log(rng, 32, 512), cols=1024 * rng.randint(4, 64),
             chunks=rng.randint(1, 3), widths=widths, sigma=sigma)
    return dict(c, dms=_log(rng, 32, 2048)) if rng.random() < 0.5 else c


def _seed(seed, k=0):
    return int(seed) * 1009 + k


# ---------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------

def _store(x, dtype, row_sigma, row_mu):
    """The plane as stored: (data, scale, zero)."""
    if dtype == "u8":
        return synth.quantize_u8(x, row_sigma, row_mu=row_mu)
    return x.to(DTYPES[dtype]), None, None


def _plane(case, seed):
    """An SKA-like plane: per-row offset and scale, pulses of widths up to the list's widest, and (AUTO sigma)
    some signal-dominated rows."""
    rows, cols, nmax = case["rows"], case["cols"], widths_of(case)[-1]
    p = synth.make_plane(rows, cols, seed=_seed(seed), device="cuda", n_pulses=max(2, rows // 20),
                         pulse_widths=range(1, nmax + 1), snr_range=(6.0, 50.0), gap=nmax, mean_range=(-5.0, 5.0),
                         scale_range=(0.5, 2.0), n_bright=rows // 500 + 1 if case["sigma"] == "auto" else 0,
                         t_margin=nmax - 1)
    return _store(p.x, case["dtype"], p.row_sigma, p.row_mu)


def _chunk_inputs(case, seed):
    """The chunk before, and this chunk behind its halo."""
    cs, _ = synth.stream_chunks(2, case["rows"], case["cols"], seed=_seed(seed), device="cuda",
                                wmax=widths_of(case)[-1], dtype=DTYPES[case["dtype"]])
    halo = widths_of(case)[-1] - 1
    return cs[0], torch.cat([cs[0][:, cs[0].shape[1] - halo:], cs[1]], dim=1)


def _snr_inputs(case, seed):
    """An SNR plane with the clouds that bright pulses leave, and width indices."""
    g = torch.Generator(device="cuda").manual_seed(_seed(seed))
    rows, cols = case["rows"], case["cols"]
    snr = torch.randn((rows, cols), generator=g, device="cuda")
    rng = np.random.default_rng(_seed(seed))
    for _ in range(case["bumps"]):
        r0, t0 = int(rng.integers(0, rows)), int(rng.integers(0, cols))
        dr, dt, peak = float(rng.uniform(0.5, 4.0)), float(rng.uniform(2.0, 100.0)), float(rng.uniform(8.0, 30.0))
        a, b = max(0, r0 - 8), min(rows, r0 + 9)
        lo, hi = max(0, t0 - 500), min(cols, t0 + 501)
        rr = torch.arange(a, b, device="cuda", dtype=torch.float32)[:, None]
        tt = torch.arange(lo, hi, device="cuda", dtype=torch.float32)[None, :]
        snr[a:b, lo:hi] += peak * torch.exp(-(rr - r0).abs() / dr - (tt - t0).abs() / dt)
    widx = torch.randint(0, 32, (rows, cols), generator=g, device="cuda", dtype=torch.uint8)
    return snr, widx


def _band(chans, dms, dm_step=1.0):
    """1550 MHz down by 300 MHz; trial DMs `dm_step` samples of delay apart at the lowest channel."""
    bw = 300.0 / chans
    f_low = 1550.0 - (chans - 1) * bw
    per_dm = 4.148808e3 * (1.0 / f_low ** 2 - 1.0 / 1550.0 ** 2) / SAMPLE_S
    return (1550.0, bw, SAMPLE_S), np.arange(dms) * dm_step / per_dm


def _beam_shapes(case):
    """Beams of uneven shape around the case's rows and columns (the same for every seed)."""
    rng = np.random.default_rng(case["beams"] * 7919 + case["rows"])
    return [(max(1, int(case["rows"] * rng.choice([0.5, 1, 2]))), int(case["cols"] * rng.choice([1, 1, 2])))
            for _ in range(case["beams"])]


def _beams(case, seed):
    """Noise; every eighth beam holds four pulses."""
    nmax = widths_of(case)[-1]
    out = []
    for k, (r, c) in enumerate(_beam_shapes(case)):
        p = synth.make_plane(r, c, seed=_seed(seed, k), device="cuda", n_pulses=0 if k % 8 else 4,
                             pulse_widths=range(1, nmax + 1), snr_range=(8.0, 30.0), gap=nmax, t_margin=nmax - 1)
        out.append(p.x.to(DTYPES[case["dtype"]]))
    return out


def _stream(case, seed, beam):
    """One beam's consecutive chunks: a plane with pulses across the cuts, or (with trials) a filterbank with
    two dispersed pulses."""
    if case.get("dms"):
        band, dm = _band(case["rows"], case["dms"])
        cols = case["cols"] * case["chunks"]
        fb = synth.filterbank(case["rows"], cols, seed=_seed(seed, beam), device="cuda")
        delays, most = B.dedisp_delay_table(case["rows"], *band, dm)
        rng = np.random.default_rng(_seed(seed, beam))
        for _ in range(2):
            synth.inject_along(fb, delays[int(rng.integers(0, case["dms"]))], int(rng.integers(0, cols - most - 64)),
                               int(rng.integers(1, 17)), 4)
        return [fb[:, k * case["cols"]:(k + 1) * case["cols"]].contiguous() for k in range(case["chunks"])]
    return synth.stream_chunks(case["chunks"], case["rows"], case["cols"], seed=_seed(seed, beam), device="cuda",
                               wmax=widths_of(case)[-1])[0]


def _outputs(rows, nout, pad):
    stride = (nout + 15) // 16 * 16 if pad else nout
    snr = torch.empty((rows, stride), dtype=torch.float32, device="cuda")[:, :nout]
    widx = torch.empty((rows, stride), dtype=torch.uint8, device="cuda")[:, :nout]
    return snr, widx


# ---------------------------------------------------------------------------
# one pass
# ---------------------------------------------------------------------------

def prepare(case, seed):
    kind = case["kind"]
    s = dict(kind=kind)
    if kind in ("detect", "dit"):
        W = widths_of(case)
        s["x"], s["scale"], s["zero"] = _plane(case, seed)
        s["params"] = B.Params(W, 7.0, "row", case["sigma"], 1.0)
        s["snr"], s["widx"] = _outputs(case["rows"], case["cols"] - W[-1] + 1, case["pad"])
        s["stats"] = torch.empty((case["rows"], B.STATS_FIELDS), dtype=torch.float64, device="cuda")
        s["cand"] = B.new_candidates(CAPACITY, "cuda")
        s["count"] = torch.zeros(1, dtype=torch.int64, device="cuda")
        s["ws"] = torch.empty(B.workspace_bytes(s["x"], s["params"], s["scale"], s["zero"]), dtype=torch.uint8,
                              device="cuda")
        s["levels"] = case.get("levels")
    elif kind == "chunk":
        W = widths_of(case)
        prev, s["x"] = _chunk_inputs(case, seed)
        s["params"] = B.Params(W, 7.0, "row", case["sigma"], 1.0)
        s["state"] = torch.zeros((case["rows"], B.STATE_FIELDS), dtype=torch.float64, device="cuda")
        s["stats"] = B.msd_compute(prev, s["params"], state=s["state"])
        s["cand"] = B.new_candidates(CAPACITY, "cuda")
        s["count"] = torch.zeros(1, dtype=torch.int64, device="cuda")
        s["ws"] = torch.empty(B.workspace_bytes(s["x"], s["params"]), dtype=torch.uint8, device="cuda")
        s["t0"] = case["cols"] - (W[-1] - 1)
    elif kind == "peaks":
        s["snr"], s["widx"] = _snr_inputs(case, seed)
        s["params"] = B.Params(list(range(1, 33)), 6.0)
        s["cand"] = B.new_candidates(1 << 20, "cuda")
        s["count"] = torch.zeros(1, dtype=torch.int64, device="cuda")
        s["peaks"] = B.new_candidates(1 << 16, "cuda")
        s["n_peaks"] = torch.zeros(1, dtype=torch.int64, device="cuda")
        s["radii"] = case["dm_radius"], case["t_radius"]
    elif kind == "dedisp":
        band, dm = _band(case["chans"], case["dms"], case["dm_step"])
        s["plan"] = B.DedispPlan(case["chans"], *band, dm)
        s["fb"] = synth.filterbank(case["chans"], case["samples"], seed=_seed(seed), device="cuda")
        s["out"] = torch.empty((case["dms"], case["samples"] - s["plan"].max_delay), dtype=torch.float32,
                               device="cuda")
    elif kind == "batch":
        s["beams"] = _beams(case, seed)
        s["plan"] = B.BatchPlan(s["beams"], B.Params(widths_of(case), 7.0, "row", case["sigma"], 1.0), autotune=False)
        s["cand"] = B.new_candidates(CAPACITY, "cuda")
        s["count"] = torch.zeros(1, dtype=torch.int64, device="cuda")
    else:
        plan = None
        if case.get("dms"):
            band, dm = _band(case["rows"], case["dms"])
            plan = B.DedispPlan(case["rows"], *band, dm)
        s["server"] = B.Server(case["beams"], case["rows"], case["cols"],
                               B.Params(widths_of(case), 7.0, "row", case["sigma"], 1.0), dtype=torch.float16,
                               cand_capacity=1 << 16, dedisp=plan)
        s["chunks"] = [[c.cpu().pin_memory() for c in _stream(case, seed, b)] for b in range(case["beams"])]
        s["seq"] = 0
    return s


def _fields(c):
    """The host's candidate table: in order of beam, row and time, one array a field."""
    c = c[np.lexsort((c["t"], c["row"], c["beam"]))][:TABLE]
    out = {}
    for k, kind in (("beam", np.int32), ("row", np.int32), ("t", np.int64), ("width", np.int32), ("snr", np.float32)):
        out[k] = np.zeros(TABLE, dtype=kind)
        out[k][:c.size] = c[k]
    return out


def _table(snrs):
    """The table's SNR column from blocks of SNRs in order."""
    v = torch.cat(snrs)[:TABLE]
    return torch.nn.functional.pad(v, (0, TABLE - v.numel()))


def _fetch(cand, count):
    return _fields(B.candidates_to_numpy(cand, int(count.item())))


def run(s):
    kind = s["kind"]
    if kind == "detect":
        B.spd_detect(s["x"], s["params"], scale=s["scale"], zero=s["zero"], stats=s["stats"], snr=s["snr"],
                     widx=s["widx"], cand=s["cand"], cand_count=s["count"], workspace=s["ws"])
        return {k: s[k] for k in ("stats", "snr", "widx", "count")}
    if kind == "dit":
        B.msd_compute(s["x"], s["params"], scale=s["scale"], zero=s["zero"], stats=s["stats"], workspace=s["ws"])
        B.boxcar_snr_dit(s["x"], s["params"], s["levels"], s["stats"], scale=s["scale"], zero=s["zero"],
                         snr=s["snr"], widx=s["widx"], cand=s["cand"], cand_count=s["count"])
        return {k: s[k] for k in ("stats", "snr", "widx", "count")}
    if kind == "chunk":
        B.msd_compute(s["x"], s["params"], new_col_begin=s["params"].nmax - 1, accumulate=True, state=s["state"],
                      stats=s["stats"], workspace=s["ws"])
        B.boxcar_snr(s["x"], s["params"], s["stats"], t_offset=s["t0"], cand=s["cand"], cand_count=s["count"])
        return {"state": s["state"], "stats": s["stats"], "cands": _fetch(s["cand"], s["count"])}
    if kind == "peaks":
        B.select_candidates(s["snr"], s["widx"], s["params"], cand=s["cand"], cand_count=s["count"])
        B.cluster_candidates(s["snr"], s["cand"], s["count"], *s["radii"], peaks=s["peaks"], peak_count=s["n_peaks"])
        return {"count": s["count"], "peaks": _fetch(s["peaks"], s["n_peaks"])}
    if kind == "dedisp":
        return s["plan"].run(s["fb"], out=s["out"])
    if kind == "batch":
        s["plan"].run(s["cand"], s["count"], use_graph=True)
        return _fetch(s["cand"], s["count"])
    srv, n, got = s["server"], len(s["chunks"][0]), {}
    for k in range(n):
        for b, chunks in enumerate(s["chunks"]):
            srv.submit(b, s["seq"] + k, chunks[k])
    while len(got) < n * len(s["chunks"]):
        r = srv.poll(wait_ms=100)
        if r is not None:
            got[r[0]["beam"], r[0]["seq"]] = r
    s["seq"] += n
    order = [got[key] for key in sorted(got)]
    return {"t_offset": np.array([res["t_offset"] for res, _ in order]),
            "n": np.array([res["n_cands"] for res, _ in order]),
            "cands": _fields(np.concatenate([c for _, c in order]))}


# ---------------------------------------------------------------------------
# what a pass cannot do without
# ---------------------------------------------------------------------------

def _evals(case):
    """(start, width) pairs per row of cols columns."""
    W = widths_of(case)
    nout = case["cols"] - W[-1] + 1
    if case["kind"] != "dit":
        return nout * len(W)
    return sum((nout + (1 << lv) - 1 >> lv) * (16 if lv == 0 else 8) for lv in range(case["levels"] + 1))


def work(case):
    """Bytes: inputs once, outputs once.  flops: an add, a multiply and a compare per (start, width); one addition
    per (trial, channel, start) for de-dispersion."""
    kind = case["kind"]
    if kind in ("detect", "dit"):
        n = case["rows"] * case["cols"]
        nout = case["rows"] * (case["cols"] - widths_of(case)[-1] + 1)
        return {"bytes": n * ELEM[case["dtype"]] + 5 * nout, "flops": 3 * case["rows"] * _evals(case) + 4 * n}
    if kind == "chunk":
        n = case["rows"] * (case["cols"] + widths_of(case)[-1] - 1)
        return {"bytes": n * ELEM[case["dtype"]], "flops": 3 * case["rows"] * case["cols"] * len(widths_of(case))}
    if kind == "peaks":
        return {"bytes": 4 * case["rows"] * case["cols"], "flops": case["rows"] * case["cols"]}
    if kind == "dedisp":
        band, dm = _band(case["chans"], case["dms"], case["dm_step"])
        nout = case["samples"] - int(math.floor((case["dms"] - 1) * case["dm_step"] + 0.5))
        return {"bytes": case["chans"] * case["samples"] + 4 * case["dms"] * nout,
                "flops": case["chans"] * case["dms"] * nout}
    if kind == "batch":
        W, n, pairs = widths_of(case), 0, 0
        for r, c in _beam_shapes(case):
            n, pairs = n + r * c, pairs + r * (c - W[-1] + 1) * len(W)
        return {"bytes": n * ELEM[case["dtype"]], "flops": 3 * pairs + 4 * n}
    n = case["beams"] * case["chunks"] * case["cols"]
    if case.get("dms"):
        return {"bytes": n * case["rows"], "flops": n * case["dms"] * (case["rows"] + 3 * len(widths_of(case)))}
    return {"bytes": 2 * n * case["rows"], "flops": 3 * n * case["rows"] * len(widths_of(case))}


# ---------------------------------------------------------------------------
# the same results in 64 bits, in plain torch
# ---------------------------------------------------------------------------

def _steps(W, levels=None):
    """(width, stride of its starts) of the list."""
    return [(w, 1 if levels is None or i < 16 else 1 << (1 + (i - 16) // 8)) for i, w in enumerate(W)]


def _row_stats(x, W, mode):
    """[rows, 5] statistics of a float64 block (flags in the last column's low word)."""
    nmax = W[-1]
    out = torch.zeros((x.shape[0], 5), dtype=torch.float64, device=x.device)
    mean = x.mean(dim=1)
    d = x - mean[:, None]
    sigma = (d * d).mean(dim=1).sqrt()
    out[:, 0], out[:, 1] = mean, sigma
    if mode != "sqrtn":
        p = torch.nn.functional.pad(d.cumsum(dim=1), (1, 0))
        y = p[:, nmax:] - p[:, :-nmax]
        out[:, 2] = y.var(dim=1, unbiased=False).sqrt()
        _linear(out, nmax)
    return out


def _linear(out, nmax):
    """AUTO: the anchored linear coefficient where sigma_Nmax is over twice sqrt(Nmax) sigma."""
    base = math.sqrt(nmax) * out[:, 1]
    on = out[:, 2] > 2.0 * base
    out[:, 3] = torch.where(on, (out[:, 2] - base) / max(1, nmax - 1), torch.zeros_like(base))
    out.view(torch.int32)[:, 8] = 2 * on.to(torch.int32)


def _best_snr(x, st, steps):
    """Highest SNR per start of a float64 block, given its rows' statistics."""
    d = x - st[:, :1]
    p = torch.nn.functional.pad(d.cumsum(dim=1), (1, 0))
    del d
    nmax = steps[-1][0]
    nout = x.shape[1] - nmax + 1
    best = torch.full((x.shape[0], nout), -math.inf, dtype=torch.float64, device=x.device)
    for w, step in steps:
        inv = 1.0 / (math.sqrt(w) * st[:, 1:2] + (w - 1) * st[:, 3:4])
        b = (p[:, w:w + nout:step] - p[:, 0:nout:step]).mul_(inv)
        best[:, ::step] = torch.maximum(best[:, ::step], b)
    return best


def _blocks(x, scale, zero):
    """Row blocks of a stored plane in float64."""
    per = max(1, (1 << 25) // x.shape[1])
    for r in range(0, x.shape[0], per):
        v = x[r:r + per].double()
        yield r, v if scale is None else (v - zero[r:r + per, None].double()) * scale[r:r + per, None].double()


def exact(case, seed):
    kind = case["kind"]
    if kind in ("detect", "dit"):
        x, scale, zero = _plane(case, seed)
        W = widths_of(case)
        steps = _steps(W, case.get("levels"))
        stats = torch.empty((case["rows"], 5), dtype=torch.float64, device="cuda")
        snr = torch.empty((case["rows"], case["cols"] - W[-1] + 1), dtype=torch.float64, device="cuda")
        for r, v in _blocks(x, scale, zero):
            stats[r:r + v.shape[0]] = st = _row_stats(v, W, case["sigma"])
            snr[r:r + v.shape[0]] = _best_snr(v, st, steps)
        return {"stats": stats, "snr": snr, "widx": None, "count": None}
    if kind == "chunk":
        prev, x = _chunk_inputs(case, seed)
        W = widths_of(case)
        nmax = W[-1]
        state = torch.zeros((case["rows"], 6), dtype=torch.float64, device="cuda")
        stats = torch.zeros((case["rows"], 5), dtype=torch.float64, device="cuda")
        snrs = []
        for r, v in _blocks(x, None, None):
            q, rows = prev[r:r + v.shape[0]].double(), slice(r, r + v.shape[0])
            raw = torch.cat([q, v[:, nmax - 1:]], dim=1)
            mean = raw.mean(dim=1, keepdim=True)
            ys = []
            for part in (q, v):
                p = torch.nn.functional.pad(part.cumsum(dim=1), (1, 0))
                ys.append(p[:, nmax:] - p[:, :-nmax])
            y = torch.cat(ys, dim=1)
            state[rows, 0], state[rows, 1] = raw.shape[1], raw.sum(dim=1)
            state[rows, 2] = (raw - mean).square().sum(dim=1)
            stats[rows, 0], stats[rows, 1] = mean[:, 0], (state[rows, 2] / raw.shape[1]).sqrt()
            if case["sigma"] != "sqrtn":
                state[rows, 3], state[rows, 4] = y.shape[1], y.sum(dim=1)
                state[rows, 5] = (y - y.mean(dim=1, keepdim=True)).square().sum(dim=1)
                stats[rows, 2] = (state[rows, 5] / y.shape[1]).sqrt()
                st = stats[rows].clone()
                _linear(st, nmax)
                stats[rows] = st
            best = _best_snr(v, stats[rows], _steps(W))
            snrs.append(best[best >= 7.0])               # in order of row and time
        return {"state": state, "stats": stats, "cands": {"snr": _table(snrs)}}
    if kind == "dedisp":
        if case["chans"] * case["dms"] > 300000:
            return None                                  # over about 20 s of single additions
        band, dm = _band(case["chans"], case["dms"], case["dm_step"])
        delays, most = B.dedisp_delay_table(case["chans"], *band, dm)
        fb = synth.filterbank(case["chans"], case["samples"], seed=_seed(seed), device="cuda").double()
        n = case["samples"] - most
        out = torch.zeros((case["dms"], n), dtype=torch.float64, device="cuda")
        for d in range(case["dms"]):
            for c in range(case["chans"]):
                k = int(delays[d, c])
                out[d] += fb[c, k:k + n]
        return out
    if kind == "batch":
        W, snrs = widths_of(case), []
        for x in _beams(case, seed):
            for r, v in _blocks(x, None, None):
                st = _row_stats(v, W, case["sigma"])
                best = _best_snr(v, st, _steps(W))
                snrs.append(best[best >= 7.0])           # in order of beam, row and time
        return {"snr": _table(snrs)}
    return None
