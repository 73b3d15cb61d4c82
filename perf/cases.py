"""Timed workloads of the framework, through its public Python entry points.

Each case is a plain dict. ``kind`` says which entry point it exercises:

  plane     Plan.convolve: one spectrum -> one z-r power plane
  batch     Plan.convolve_batch / convolve_batch_noalloc: many series at once
  peaks     Plan.peaks and decode_peaks: threshold + peak picking, no plane
  frontend  FrontEnd: real series -> normalised spectrum
  fft       FFT: the standalone batched transform
  bank      make_bank: a new Fourier-domain template bank

Sizes are those of the workload recipes (``synth.WORKLOADS``), of the tests
and of the microbenchmarks, and generic odd ones. Inputs are white noise with
a few accelerated sinusoids, as a search meets them.
"""

from __future__ import annotations

import math

import numpy as np
import torch

from paper_1711_10855_amd import fdas

DZ = 2.0      # drift step of every workload recipe
PEAKS = 4096  # room for the peaks of one observation


# ---- the cases ---------------------------------------------------------------

def _plane(name, precision, nbins, zmax, m, seg_len, split=False, interbin=False, pad=False):
    c = {"kind": "plane", "precision": precision, "nbins": nbins, "zmax": zmax, "m": m,
         "seg_len": seg_len, "split": split, "interbin": interbin, "pad": pad}
    return dict(c, name=name) if name else c


def _batch(name, precision, nseries, lo, hi, mixed_zmax, zmax, m, seg_len, split=False,
           noalloc=False, pad=True):
    c = {"kind": "batch", "precision": precision, "nseries": nseries, "lo": lo, "hi": hi,
         "mixed_zmax": mixed_zmax, "zmax": zmax, "m": m, "seg_len": seg_len, "split": split,
         "noalloc": noalloc, "pad": pad}
    return dict(c, name=name) if name else c


def listed():
    return [
        # a short observation: 2^15 bins, 17 drifts; the smallest plane of use
        _plane("plane_fp32_small", "fp32", 1 << 15, 16.0, 64, 256),
        # one full observation in plain FP32: 2^21 bins, 101 drifts, the
        # paper's segment length
        _plane("plane_fp32", "fp32", 1 << 21, 100.0, 256, 2048),
        # the same search on the matrix cores
        _plane("plane_fp16", "fp16", 1 << 21, 100.0, 256, 4096),
        # an observation of no round length: odd number of bins, rows packed
        # without padding, so no row after the first is 16-byte aligned
        _plane("plane_fp16_odd", "fp16", 1048573, 64.0, 256, 4096),
        # near-FP32 accuracy on the matrix cores, half-length observation
        _plane("plane_bf16_split", "bf16", 1 << 20, 100.0, 256, 4096, split=True),
        # a night's beams of different lengths and drift ranges in one call
        _batch("batch_fp32_uneven", "fp32", 12, 1 << 19, 1 << 21, True, 100.0, 256, 2048),
        # wide filters over several full observations: the largest case
        _batch("batch_fp16_wide", "fp16", 8, 1 << 21, 1 << 21, False, 200.0, 512, 4096),
        # detection without a plane: threshold 30, peaks decoded on the host
        {"name": "peaks_fp32", "kind": "peaks", "nbins": 1 << 21, "zmax": 100.0, "m": 256,
         "seg_len": 2048, "threshold": 30.0},
        # spectrum of a short and of a full observation
        {"name": "frontend_small", "kind": "frontend", "n": 1 << 16, "series": 1},
        {"name": "frontend_full", "kind": "frontend", "n": 1 << 22, "series": 1},
        # the standalone transform, as the paper times it (1024 points)
        {"name": "fft_1024", "kind": "fft", "n": 1024, "batch": 100000, "direction": -1},
        # a new filter bank (templates and their transforms)
        {"name": "bank", "kind": "bank", "zmax": 100.0, "m": 256, "seg_len": 2048,
         "interbin": False},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _filter(rng):
    """A drift range and a width: the default width of that range, or an
    uneven one a little under it."""
    zmax = rng.choice([16.0, 32.0, 64.0, 100.0, 200.0])
    m = 1
    while m < 2 * zmax + 32:
        m *= 2
    if rng.random() < 0.25:
        m -= 2 * rng.randrange(1, 9)
    return zmax, m


def _fp32_len(rng, m):
    lens = [n for n in (256, 512, 1024, 2048, 4096) if n >= 4 * m or n == 4096]
    return rng.choice(lens)


def draw(rng):
    kind = rng.choice(["plane", "plane", "plane", "plane", "batch", "batch", "peaks",
                       "frontend", "fft", "bank"])
    if kind == "plane":
        zmax, m = _filter(rng)
        nbins = _log_int(rng, 1 << 14, 1 << 21)
        if rng.random() < 0.4:
            nbins -= nbins % 256  # round lengths are common too
        pad = rng.random() < 0.5
        form = rng.choice(["fp32", "fp32", "fp16", "fp16", "fp16-2048", "bf16-split",
                           "fp16-split", "bf16"])
        inter = rng.random() < 0.2
        if form == "fp32":
            return _plane(None, "fp32", nbins, zmax, m, _fp32_len(rng, m), interbin=inter, pad=pad)
        seg = 2048 if form.endswith("2048") else 4096
        return _plane(None, form[:4], nbins, zmax, m, seg, split=form.endswith("split"),
                      interbin=inter, pad=pad)
    if kind == "batch":
        n = rng.randrange(3, 13)
        hi = _log_int(rng, 1 << 16, 1 << 19)
        lo = max(1 << 14, hi // rng.choice([1, 2, 4]))
        zmax, m = rng.choice([(100.0, 256), (200.0, 512)])
        form = rng.choice(["fp32", "fp16", "bf16-split"])
        seg = 4096 if form != "fp32" else rng.choice([2048, 4096])
        return _batch(None, form[:4], n, lo, hi, zmax == 100.0, zmax, m, seg,
                      split=form.endswith("split"), noalloc=rng.random() < 0.3,
                      pad=rng.random() < 0.7)
    if kind == "peaks":
        zmax, m = _filter(rng)
        return {"kind": "peaks", "nbins": _log_int(rng, 1 << 15, 1 << 21), "zmax": zmax, "m": m,
                "seg_len": _fp32_len(rng, m), "threshold": float(rng.randrange(20, 41))}
    if kind == "frontend":
        # several series of one length through one plan, one after the other
        return {"kind": "frontend", "n": 1 << rng.randrange(14, 24), "series": rng.randrange(2, 9)}
    if kind == "fft":
        n = rng.choice([256, 512, 1024, 2048, 4096])
        return {"kind": "fft", "n": n, "batch": _log_int(rng, 64, (1 << 27) // n),
                "direction": rng.choice([-1, 1])}
    zmax, m = _filter(rng)
    return {"kind": "bank", "zmax": zmax, "m": m, "seg_len": _fp32_len(rng, m),
            "interbin": rng.random() < 0.3}


# ---- sizes -------------------------------------------------------------------

def _flags(case):
    return ((fdas.FLAG_SPLIT if case.get("split") else 0)
            | (fdas.FLAG_INTERBIN if case.get("interbin") else 0))


def _rows(zmax, interbin=False):
    nz = int(round(2 * zmax / DZ)) + 1
    return 2 * nz if interbin else nz


def _series_sizes(case):
    """(bins, zmax) of each series of a batch: lengths spread between lo and
    hi, and for a mixed batch the drift ranges of the uneven workload."""
    n, lo, hi = case["nseries"], case["lo"], case["hi"]
    out = []
    for j in range(n):
        u = (0.5 + j * 0.6180339887498949) % 1.0
        bins = int(round(lo * (hi / lo) ** u))
        out.append((bins, (32.0, 64.0, 100.0)[j % 3] if case["mixed_zmax"] else case["zmax"]))
    return out


def _conv_flops(nbins, rows, m, seg_len):
    """Segment transforms of an overlap-and-save (one forward, one inverse
    per row) with the product and the power."""
    nseg = nbins / (seg_len - m)
    return nseg * seg_len * (5 * math.log2(seg_len) * (rows + 1) + 9 * rows)


def work(case):
    k = case["kind"]
    if k == "plane":
        rows = _rows(case["zmax"], case["interbin"])
        return {"bytes": case["nbins"] * (8 + 4 * rows),
                "flops": _conv_flops(case["nbins"], rows, case["m"], case["seg_len"])}
    if k == "batch":
        sizes = _series_sizes(case)
        return {"bytes": sum(b * (8 + 4 * _rows(z)) for b, z in sizes),
                "flops": sum(_conv_flops(b, _rows(z), case["m"], case["seg_len"])
                             for b, z in sizes)}
    if k == "peaks":  # the spectrum in; what comes out is a few records
        return {"bytes": case["nbins"] * 8,
                "flops": _conv_flops(case["nbins"], _rows(case["zmax"]), case["m"],
                                     case["seg_len"])}
    if k == "frontend":
        n = case["n"]
        return {"bytes": case["series"] * 8 * n,
                "flops": case["series"] * (2.5 * n * math.log2(n) + 6 * n)}
    if k == "fft":
        n = case["n"] * case["batch"]
        return {"bytes": 16 * n, "flops": 5 * n * math.log2(case["n"])}
    rows, L = _rows(case["zmax"], case["interbin"]), case["seg_len"]
    return {"bytes": 8 * rows * L, "flops": rows * 5 * L * math.log2(L)}


# ---- inputs --------------------------------------------------------------------

def _generator(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    return g


def _observation(n, seed, zlim, nbins):
    """Real series of n samples: N(0, 1) noise and eight accelerated
    sinusoids of S/N 8 to 30 in the first nbins Fourier bins."""
    g = _generator(seed)
    x = torch.randn(n, generator=g, device="cuda", dtype=torch.float64)
    r = np.random.default_rng(seed)
    s = torch.arange(n, device="cuda", dtype=torch.float64) / n - 0.5
    for _ in range(8):
        r0 = r.uniform(0.02, 0.98) * nbins
        z0 = r.uniform(-0.9 * zlim, 0.9 * zlim)
        a = 2.0 * r.uniform(8.0, 30.0) / math.sqrt(n)
        turns = r0 * s + (0.5 * z0) * s * s + r.uniform()
        x += a * torch.cos((2.0 * math.pi) * (turns - turns.round()))
    return x


def _spectrum(nbins, seed, zlim):
    """Normalised complex64 spectrum: the first nbins bins of an observation
    whose length is a power of two."""
    n = 1 << (2 * nbins - 1).bit_length()
    a = torch.fft.rfft(_observation(n, seed, zlim, nbins))[:nbins].clone()
    a[0] = 0
    power = a[1:].real.square() + a[1:].imag.square()
    a /= math.sqrt(float(power.median()) / math.log(2.0))
    return a.to(torch.complex64)


def _out(rows, nbins, pad):
    ld = (nbins + 63) // 64 * 64 if pad else nbins
    return torch.empty((rows, ld), dtype=torch.float32, device="cuda")


def _spectra(case, seed):
    return [_spectrum(b, 1000 * seed + j, z) for j, (b, z) in enumerate(_series_sizes(case))]


def _time_series(case, seed):
    n = case["n"]
    return [_observation(n, 1000 * seed + j, 100.0, n // 2).to(torch.float32)
            for j in range(case["series"])]


def prepare(case, seed):
    k = case["kind"]
    s = {"case": case}
    if k == "plane":
        s["plan"] = fdas.Plan(case["zmax"], DZ, case["m"], case["seg_len"], case["precision"],
                              _flags(case))
        s["spec"] = _spectrum(case["nbins"], seed, case["zmax"])
        s["out"] = _out(s["plan"].nz, case["nbins"], case["pad"])
    elif k == "batch":
        s["plan"] = fdas.Plan(case["zmax"], DZ, case["m"], case["seg_len"], case["precision"],
                              _flags(case))
        s["spectra"] = _spectra(case, seed)
        sizes = _series_sizes(case)
        s["zmaxs"] = [z for _, z in sizes]
        s["outs"] = [_out(_rows(z), b, case["pad"]) for b, z in sizes]
    elif k == "peaks":
        s["plan"] = fdas.Plan(case["zmax"], DZ, case["m"], case["seg_len"])
        s["spec"] = _spectrum(case["nbins"], seed, case["zmax"])
    elif k == "frontend":
        s["frontend"] = fdas.FrontEnd(case["n"])
        s["series"] = _time_series(case, seed)
        s["out"] = [torch.empty(case["n"] // 2, dtype=torch.complex64, device="cuda")
                    for _ in s["series"]]
        s["stats"] = [torch.empty(2, dtype=torch.float32, device="cuda") for _ in s["series"]]
    elif k == "fft":
        s["fft"] = fdas.FFT(case["n"])
        s["x"] = torch.randn((case["batch"], case["n"]), generator=_generator(seed),
                             device="cuda", dtype=torch.complex64)
        s["out"] = torch.empty_like(s["x"])
    else:
        # the filter's drift range is data here: each seed asks for a bank of
        # the same size whose grid ends a little elsewhere
        s["scale"] = _bank_scale(seed)
    return s


def _bank_scale(seed):
    return 1.0 - (1 + seed % 997) / 65536.0


def _peak_table(row, r, power, n_cand):
    """Peaks in (row, bin) order in a table of fixed size, unused entries -1."""
    index = np.full((2, PEAKS), -1, dtype=np.int64)
    index[0, : row.size], index[1, : row.size] = row[:PEAKS], r[:PEAKS]
    table = np.full(PEAKS, -1.0, dtype=power.dtype)
    table[: row.size] = power[:PEAKS]
    return {"index": index, "power": table, "peaks": int(row.size), "candidates": n_cand}


def run(state):
    c = state["case"]
    k = c["kind"]
    if k == "plane":
        state["plan"].convolve(state["spec"], out=state["out"])
        return state["out"][:, : c["nbins"]]
    if k == "batch":
        call = state["plan"].convolve_batch_noalloc if c["noalloc"] else state["plan"].convolve_batch
        outs = call(state["spectra"], state["zmaxs"], state["outs"])
        return [o[:, : a.numel()] for o, a in zip(outs, state["spectra"])]
    if k == "peaks":
        rec, counts, _, _ = state["plan"].peaks(state["spec"], c["threshold"],
                                                peak_capacity=PEAKS)
        row, r, power, n_cand, n_peak = fdas.decode_peaks(rec, counts)
        order = np.lexsort((r, row))  # the list comes in no fixed order
        return _peak_table(row[order], r[order], power[order], n_cand)
    if k == "frontend":
        for x, out, stats in zip(state["series"], state["out"], state["stats"]):
            state["frontend"](x, out=out, stats=stats)
        return {"spectrum": state["out"], "stats": state["stats"]}
    if k == "fft":
        return state["fft"](state["x"], out=state["out"], direction=c["direction"])
    f = state["scale"]
    return fdas.make_bank(c["zmax"] * f, DZ * f, c["m"], c["seg_len"], _flags(c))


# ---- the same in 64 bits -----------------------------------------------------

def _templates(zmax, dz, m, interbin=False):
    """H_z(q) = int_{-1/2}^{1/2} exp(i pi z s^2) exp(-2 pi i q (s + 1/2)) ds
    by Gauss-Legendre quadrature, complex128 [rows, m + 1]."""
    panels, order = 32, 64
    node, weight = np.polynomial.legendre.leggauss(order)
    edge = np.linspace(-0.5, 0.5, panels + 1)
    s = (0.5 * (edge[:-1] + edge[1:])[:, None] + 0.5 / panels * node[None]).ravel()
    w = np.tile(0.5 / panels * weight, panels)
    s = torch.from_numpy(s).cuda()
    w = torch.from_numpy(w).cuda()
    z = -zmax + dz * torch.arange(_rows(zmax / dz * DZ), device="cuda", dtype=torch.float64)
    q = torch.arange(-(m // 2), m // 2 + 1, device="cuda", dtype=torch.float64)
    q = torch.cat([q, q - 0.5]) if interbin else q

    def unit(turns):
        turns = 2.0 * math.pi * (turns - turns.round())
        return torch.complex(torch.cos(turns), torch.sin(turns))

    chirp = unit(0.5 * z[:, None] * (s * s)[None]) * w
    h = torch.matmul(chirp, unit(-(s + 0.5)[:, None] * q[None]))
    # interbin: rows alternate between integer bins and half-way between them
    return h.reshape(h.shape[0] * 2, m + 1) if interbin else h


def _exact_plane(spec, h, m):
    nbins = spec.numel()
    n = 1
    while n < nbins + m + 1:
        n *= 2
    fa = torch.fft.fft(spec.to(torch.complex128), n)
    at = torch.arange(-(m // 2), m // 2 + 1, device="cuda") % n
    out = torch.empty((h.shape[0], nbins), dtype=torch.float64, device="cuda")
    for i in range(0, h.shape[0], 8):
        w = torch.zeros((h[i: i + 8].shape[0], n), dtype=torch.complex128, device="cuda")
        w[:, at] = h[i: i + 8]
        y = torch.fft.ifft(torch.fft.fft(w).conj().resolve_conj() * fa)[:, :nbins]
        out[i: i + 8] = y.real.square() + y.imag.square()
    return out


def _exact_peaks(plane, threshold):
    n_cand = int((plane >= threshold).sum())
    big = torch.nn.functional.pad(plane[None], (1, 1, 1, 1), value=-1.0)[0]
    top = plane >= threshold
    rows, cols = plane.shape
    for dz in range(3):
        for dr in range(3):
            if (dz, dr) != (1, 1):
                top &= plane > big[dz: dz + rows, dr: dr + cols]
    row, r = torch.nonzero(top, as_tuple=True)
    return _peak_table(row.cpu().numpy(), r.cpu().numpy(), plane[row, r].cpu().numpy(), n_cand)


def exact(case, seed):
    k = case["kind"]
    if k == "plane":
        h = _templates(case["zmax"], DZ, case["m"], case["interbin"])
        return _exact_plane(_spectrum(case["nbins"], seed, case["zmax"]), h, case["m"])
    if k == "batch":
        return [_exact_plane(a, _templates(z, DZ, case["m"]), case["m"])
                for a, (_, z) in zip(_spectra(case, seed), _series_sizes(case))]
    if k == "peaks":
        h = _templates(case["zmax"], DZ, case["m"])
        plane = _exact_plane(_spectrum(case["nbins"], seed, case["zmax"]), h, case["m"])
        return _exact_peaks(plane, case["threshold"])
    if k == "frontend":
        spectra, stats = [], []
        for x in _time_series(case, seed):
            a = torch.fft.rfft(x.double())[: case["n"] // 2].clone()
            power = a[1:].real.square() + a[1:].imag.square()
            median = float(power.median())
            scale = math.sqrt(math.log(2.0) / median)
            a[0] = 0
            spectra.append(a * scale)
            stats.append(torch.tensor([scale, median], dtype=torch.float64))
        return {"spectrum": spectra, "stats": stats}
    if k == "fft":
        x = torch.randn((case["batch"], case["n"]), generator=_generator(seed), device="cuda",
                        dtype=torch.complex64).to(torch.complex128)
        return torch.fft.fft(x) if case["direction"] < 0 else torch.fft.ifft(x, norm="forward")
    f = _bank_scale(seed)
    L, m = case["seg_len"], case["m"]
    h = _templates(case["zmax"] * f, DZ * f, m, case["interbin"])
    w = torch.zeros((h.shape[0], L), dtype=torch.complex128, device="cuda")
    w[:, torch.arange(-(m // 2), m // 2 + 1, device="cuda") % L] = h
    return torch.fft.fft(w).conj().resolve_conj() / L
