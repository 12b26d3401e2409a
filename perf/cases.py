"""The workloads this library is timed on: one case per kind of call a search program makes.

A case is a dict of plain values; ``kind`` says which call it stands for:

``plane``       one spectrum searched into a (templates x 2n) power plane (``Plan.search``), on the
                FP32 FFT path, the split-BF16 or FP16 matrix path, or the untuned mix of the two
                ("auto"). ``rows`` = 0 takes the whole bank; otherwise a slab of that many templates
                from the middle of the lattice, as a plane larger than the device memory is searched.
``peaks``       the strongest point of every template without a plane (``Plan.search_peaks``), what a
                search server returns for a request.
``candidates``  the search with candidate selection fused in (``Plan.search_candidates``), the
                result sorted on the device by (template, bin).
``batch``       several spectra of uneven lengths in one graph-replayed launch
                (``Plan.batch_search``), a slab of templates of each into its own plane.
``cold_grid``   a (z, w) grid seen for the first time: the template bank is generated, then a
                spectrum is searched for its row peaks; the first request a server gets for a grid.
``spectrum``    a float32 time series to the normalised spectrum the searches take
                (``prepare_spectrum``).
``select``      row statistics and threshold peaks of a plane slab already in memory
                (``plane_stats`` + ``find_candidates``).
``harmonics``   the incoherent harmonic sum of a full plane (``Plan.harmonic_sum``).

Sizes are those of this repository's benchmark and tests where they name one (2^15 bins with zmax 20
and wmax 60, 2^22 bins with zmax 200 and wmax 600, batches of 2^20-bin and ragged spectra with zmax
100 and wmax 300, requests with zmax from 50 up and wmax = 3 zmax, FDAS grids with wmax = 0).
Spectra are unit-mean-power noise with a few accelerated tones, as the benchmark makes them.
"""
import math

import numpy as np
import torch

import paper_1911_01353_amd as jerk

DEV = "cuda"
MARGIN = 16


def _case(kind, name=None, **kw):
    c = {"kind": kind}
    if name:
        c["name"] = name
    c.update(kw)
    return c


def listed():
    return [
        # the 2^15-bin search of 147 templates: one small launch, latency and the host path count
        _case("plane", "plane_2e15", n=1 << 15, zmax=20.0, wmax=60.0, path="fft", rows=0),
        # a constant-acceleration search (no jerk axis) over a spectrum of no round length
        _case("plane", "plane_fdas_ragged", n=(1 << 20) + 4321, zmax=200.0, wmax=0.0, path="fft", rows=0),
        # a slab of the 2^22-bin, 12261-template search, all widths of the grid's middle rows
        _case("plane", "plane_2e22_slab", n=1 << 22, zmax=200.0, wmax=600.0, path="fft", rows=201),
        # the matrix paths a request may ask for: split-BF16 (FP32-level error) and FP16
        _case("plane", "plane_split_bf16", n=1 << 20, zmax=100.0, wmax=300.0, path="split_bf16", rows=303),
        _case("plane", "plane_fp16", n=1 << 20, zmax=100.0, wmax=300.0, path="fp16", rows=303),
        # per-row peaks of a whole grid: a warm request to the server
        _case("peaks", "peaks_2e20", n=1 << 20, zmax=50.0, wmax=150.0, path="fft"),
        # search and selection in one call, the quantity a survey runs for each trial
        _case("candidates", "candidates_2e20", n=1 << 20, zmax=50.0, wmax=150.0, path="fft", k=12.0),
        # uneven spectra sharing one launch, 34 templates each
        _case("batch", "batch_uneven", n=(1 << 20) - 777, count=8, zmax=100.0, wmax=300.0, path="fft", rows=34),
        # a new grid: bank generation dominates the first request
        _case("cold_grid", "cold_grid_2e18", n=1 << 18, zmax=100.0, wmax=300.0, path="fft"),
        # preparation of the 2^22-bin workload's spectrum
        _case("spectrum", "spectrum_2e22", n=1 << 22),
        # selection over a stored slab
        _case("select", "select_slab", n=1 << 21, rows=128, k=10.0),
        # four harmonics over the plane of a 765-template search
        _case("harmonics", "harmonics_4", n=1 << 19, zmax=50.0, wmax=150.0, harm=4),
    ]


def _log_int(rng, lo, hi, odd):
    v = int(round(2.0 ** rng.uniform(math.log2(lo), math.log2(hi))))
    return v | 1 if odd else v


def draw(rng):
    kind = rng.choice(["plane", "plane", "plane", "peaks", "candidates", "batch", "cold_grid", "spectrum", "select",
                       "harmonics"])
    odd = rng.random() < 0.5
    if kind == "plane":
        path = rng.choice(["fft", "fft", "split_bf16", "fp16", "auto"])
        zmax = 2.0 * rng.randint(10, 110)
        wmax = rng.choice([0.0, 1.0, 3.0]) * zmax
        n = _log_int(rng, 1 << 15, 1 << 22, odd)
        templates = (int(zmax) + 1) * (2 * int(wmax // 20.0) + 1)
        most = max(8, (201 << 23) // (2 * n) // (1 if path == "fft" else 4))
        rows = min(templates, rng.randint(8, 320), most)
        return _case(kind, n=n, zmax=zmax, wmax=wmax, path=path, rows=0 if rows == templates else rows)
    if kind in ("peaks", "candidates"):
        zmax = 2.0 * rng.randint(10, 30)
        wmax = rng.choice([0.0, 3.0]) * zmax
        n = _log_int(rng, 1 << 16, 1 << 20, odd)
        c = _case(kind, n=n, zmax=zmax, wmax=wmax, path="fft" if kind == "candidates" else
                  rng.choice(["fft", "fft", "split_bf16"]))
        if kind == "candidates":
            c["k"] = float(rng.choice([12, 13, 14, 16]))
        return c
    if kind == "batch":
        zmax = 2.0 * rng.randint(25, 75)
        return _case(kind, n=_log_int(rng, 1 << 16, 1 << 20, odd), count=rng.randint(2, 8), zmax=zmax, wmax=3.0 * zmax,
                     path="fft", rows=rng.randint(8, 34))
    if kind == "cold_grid":
        zmax = 2.0 * rng.randint(10, 48)
        return _case(kind, n=_log_int(rng, 1 << 15, 1 << 18, odd), zmax=zmax, wmax=rng.choice([0.0, 3.0]) * zmax,
                     path=rng.choice(["fft", "fft", "split_bf16"]))
    if kind == "spectrum":
        return _case(kind, n=1 << rng.randint(12, 21))
    if kind == "select":
        return _case(kind, n=_log_int(rng, 1 << 16, 1 << 21, odd), rows=rng.randint(4, 120), k=float(rng.choice([10, 11, 12])))
    return _case(kind, n=_log_int(rng, 1 << 15, 1 << 18, odd), zmax=2.0 * rng.randint(12, 25), wmax=150.0,
                 harm=rng.choice([2, 3, 4, 8]))


# ---- inputs -------------------------------------------------------------------------------------

def _generator(seed, salt=0):
    g = torch.Generator(device=DEV)
    g.manual_seed((int(seed) * 1000003 + salt) & 0x7FFFFFFF)
    return g


def _series(n_samples, seed, salt, zmax, wmax):
    """Unit Gaussian noise and three tones inside the grid, float32."""
    g = _generator(seed, salt)
    x = torch.randn(n_samples, generator=g, device=DEV, dtype=torch.float32)
    u = torch.arange(n_samples, device=DEV, dtype=torch.float64) / n_samples
    draws = np.random.RandomState((int(seed) * 9176 + salt) & 0x7FFFFFFF).uniform(size=(3, 5))
    amp0 = 8.0 / math.sqrt(n_samples)  # a few sigma up to a few hundred in power
    for d in draws:
        r, z, w = (0.02 + 0.4 * d[0]) * n_samples / 2, (2 * d[1] - 1) * 0.8 * zmax, (2 * d[2] - 1) * 0.8 * wmax
        cyc = u * (r - z / 2 - w / 6 + u * (z / 2 + u * w / 6))
        x += (amp0 * (0.5 + d[3]) * torch.cos(2 * math.pi * (cyc - torch.floor(cyc) + d[4]))).float()
    return x


def _spectrum(n, seed, salt, zmax, wmax):
    """n bins of a unit-mean-power spectrum, complex64."""
    m = 1 << max(3, math.ceil(math.log2(n)))
    f = torch.fft.rfft(_series(2 * m, seed, salt, zmax, wmax).double())[:n]
    f[0] = 0
    f *= 1.0 / torch.sqrt(f.abs().square().sum() / max(1, n - 1))
    return f.to(torch.complex64).contiguous()


def _lengths(c):
    """Uneven spectrum lengths of a batch: n, then ever smaller odd shares of it."""
    return [max(64, (c["n"] * (2 * c["count"] - i)) // (2 * c["count"]) - 13 * i) for i in range(c["count"])]


def _slab(c, info):
    rows = c.get("rows") or info["n_templates"]
    t0 = (info["n_templates"] - rows) // 2
    return t0, t0 + rows


def prepare(case, seed):
    c = dict(case)
    kind = c["kind"]
    s = {"case": c}
    if kind == "spectrum":
        s["series"] = _series(2 * c["n"], seed, 0, 100.0, 300.0)
        s["out"] = torch.empty(c["n"], dtype=torch.complex64, device=DEV)
        s["ws"] = torch.empty(jerk.spectrum_workspace_bytes(2 * c["n"]), dtype=torch.uint8, device=DEV)
        return s
    if kind == "select":
        g = _generator(seed, 3)
        s["plane"] = torch.empty((c["rows"], 2 * c["n"]), dtype=torch.float32, device=DEV).exponential_(generator=g)
        s["stats"] = torch.empty((c["rows"], 2), dtype=torch.float64, device=DEV)
        s["ws"] = torch.empty(jerk.stats_workspace_bytes(c["rows"], 2 * c["n"]), dtype=torch.uint8, device=DEV)
        s["out"] = torch.empty((_capacity(c, c["rows"]), 4), dtype=torch.int32, device=DEV)
        s["count"] = torch.zeros(1, dtype=torch.int64, device=DEV)
        return s
    p = s["plan"] = jerk.Plan(c["n"], c["zmax"], c["wmax"], path=c.get("path", "fft"))
    info = s["info"] = p.info()
    if kind == "harmonics":
        g = _generator(seed, 5)
        s["plane"] = torch.empty((info["n_templates"], 2 * c["n"]), dtype=torch.float32, device=DEV).exponential_(generator=g)
        zf, wf, pf = p.harmonic_shape(2 * c["n"], c["harm"])
        s["out"] = torch.empty((zf * wf, pf), dtype=torch.float32, device=DEV)
        return s
    s["bank"] = p.new_bank()
    if kind == "cold_grid":
        s["groups"] = p.groups()
    else:
        p.build_templates(s["bank"])
    s["t"] = _slab(c, info)
    rows = s["t"][1] - s["t"][0]
    if kind == "batch":
        s["specs"] = [_spectrum(n, seed, 11 + i, c["zmax"], c["wmax"]) for i, n in enumerate(_lengths(c))]
        s["planes"] = [torch.empty((rows, 2 * x.shape[0]), dtype=torch.float32, device=DEV) for x in s["specs"]]
        s["ws"] = torch.empty(p.batch_workspace_bytes(c["count"]), dtype=torch.uint8, device=DEV)
        return s
    s["spec"] = _spectrum(c["n"], seed, 7, c["zmax"], c["wmax"])
    if kind == "plane":
        s["plane"] = torch.empty((rows, 2 * c["n"]), dtype=torch.float32, device=DEV)
    else:
        s["peaks"] = torch.empty((rows, 2), dtype=torch.int32, device=DEV)
        s["ws"] = torch.empty(8 * rows, dtype=torch.uint8, device=DEV)
    if kind == "candidates":
        need = p.search_candidates_workspace_bytes(c["n"], 0.9 * (1.0 + c["k"]))
        s["ws"] = torch.empty(need, dtype=torch.uint8, device=DEV)
        s["out"] = torch.empty((_capacity(c, rows), 4), dtype=torch.int32, device=DEV)
        s["count"] = torch.zeros(1, dtype=torch.int64, device=DEV)
    return s


# ---- one pass -----------------------------------------------------------------------------------

def _capacity(c, rows):
    """Candidate slots: ten times what noise gives at this threshold, and room for the tones."""
    return int(10 * 2 * c["n"] * rows * math.exp(-1.0 - c["k"])) // 4096 * 4096 + (1 << 15)


def _sorted_candidates(out, count):
    """The stored records by (template, bin), as a program sorts them before it sifts them: key and power."""
    key = (out[:, 0].to(torch.int64) << 32) | (out[:, 1].to(torch.int64) & 0xFFFFFFFF)
    key.masked_fill_(torch.arange(out.shape[0], device=out.device) >= count, 1 << 62)
    key, order = torch.sort(key)
    rec = out[order].view(torch.float32)[:, 2:]
    return {"count": count, "key": key, "power_sigma": rec.masked_fill((key == 1 << 62)[:, None], 0.0)}


def _peaks(out):
    return {"power": out.view(torch.float32)[:, 0], "p": out[:, 1]}


def run(state):
    s, c = state, state["case"]
    kind = c["kind"]
    if kind == "plane":
        s["plan"].search(s["bank"], s["spec"], s["plane"], s["t"][0], s["t"][1])
        return s["plane"]
    if kind == "peaks":
        return _peaks(s["plan"].search_peaks(s["bank"], s["spec"], out=s["peaks"], ws=s["ws"]))
    if kind == "cold_grid":
        s["plan"].build_templates(s["bank"])
        out = _peaks(s["plan"].search_peaks(s["bank"], s["spec"], out=s["peaks"], ws=s["ws"]))
        out["taps"] = [s["bank"][g["taps_offset"]:g["taps_offset"] + g["n_members"] * 2 * g["taps"] * 16].view(torch.float64)
                       for g in s["groups"]]
        return out
    if kind == "candidates":
        s["count"].zero_()
        s["plan"].search_candidates(s["bank"], s["spec"], c["k"], None, s["out"], s["count"], ws=s["ws"])
        return _sorted_candidates(s["out"], s["count"])
    if kind == "batch":
        s["plan"].batch_search(s["bank"], [(x, y, None) for x, y in zip(s["specs"], s["planes"])], s["ws"], s["t"][0],
                               s["t"][1], graph=True)
        return s["planes"]
    if kind == "spectrum":
        jerk.prepare_spectrum(s["series"], out=s["out"], ws=s["ws"])
        return s["out"]
    if kind == "select":
        jerk.plane_stats(s["plane"], s["stats"], ws=s["ws"])
        s["count"].zero_()
        jerk.find_candidates(s["plane"], s["stats"], c["k"], s["out"], s["count"])
        return {"stats": s["stats"], **_sorted_candidates(s["out"], s["count"])}
    s["plan"].harmonic_sum(s["plane"], c["harm"], out=s["out"])
    return s["out"]


# ---- what a pass cannot do without ----------------------------------------------------------------

def _lattice(c):
    """(zbar, w) of every template in order, and its half-width."""
    nz = int(math.floor(c["zmax"] + 1e-9)) + 1
    j = int(math.floor(c["wmax"] / 20.0 + 1e-9))
    z = np.tile(-c["zmax"] + 2.0 * np.arange(nz), 2 * j + 1)
    w = np.repeat(20.0 * np.arange(-j, j + 1), nz)
    return z, w, (np.ceil(np.abs(z) / 2 + np.abs(w) / 12) + MARGIN).astype(int)


def _correlation_work(c, t0, t1, lengths, to_plane):
    h = _lattice(c)[2][t0:t1]
    points = sum(2.0 * n * len(h) for n in lengths)
    taps = float(np.mean(2 * h))
    by = 8.0 * sum(lengths) + 32.0 * float(np.sum(h)) + (4.0 * points if to_plane else 8.0 * len(h))
    if c["path"] in ("split_bf16", "fp16"):
        per = 8.0 * taps * (3 if c["path"] == "split_bf16" else 1)
    else:  # overlap-save: product, inverse transform of four template lengths, power
        per = (6.0 + 5.0 * math.log2(4.0 * taps)) * 4.0 / 3.0 + 3.0
    return by, points * per


def work(case):
    c = case
    kind, n = c["kind"], c["n"]
    if kind == "spectrum":
        return {"bytes": 16.0 * n, "flops": 5.0 * n * math.log2(n) + 14.0 * n}
    if kind == "select":
        return {"bytes": 8.0 * n * c["rows"], "flops": 10.0 * n * c["rows"]}
    z, w, h = _lattice(c)
    if kind == "harmonics":
        i0, j0, harm = int(c["zmax"] / 2), int(c["wmax"] // 20.0), c["harm"]
        outs = (2 * (i0 // harm) + 1) * (2 * (j0 // harm) + 1) * ((2 * n - 1) // harm + 1)
        return {"bytes": 4.0 * outs * (1 + harm), "flops": 1.0 * outs * (harm - 1)}
    t0, t1 = _slab(c, {"n_templates": len(z)})
    by, fl = _correlation_work(c, t0, t1, _lengths(c) if kind == "batch" else [n], kind in ("plane", "batch"))
    if kind == "cold_grid":
        by += 32.0 * 2 * float(np.sum(h))
        fl += 8.0 * 16.0 * 2 * float(np.sum(2 * h * (np.abs(z) + np.abs(w) / 2 + 1)))
    return {"bytes": by, "flops": fl}


# ---- 64-bit values --------------------------------------------------------------------------------

def _exact_taps(z, w, hmax):
    """conj T(q + phase/2; z, w) of the tap window, complex128 (templates, 2, 2 hmax): tap j multiplies bin
    k0 - hmax + 1 + j. Composite Gauss-Legendre on panels of at most one cycle, the nodes shared."""
    cycles = 2.0 * hmax + 2.0 * np.abs(z).max() + np.abs(w).max() + 2.0
    panels = int(math.ceil(cycles))
    gx, gw = np.polynomial.legendre.leggauss(16)
    u = ((np.arange(panels)[:, None] + 0.5 + 0.5 * gx[None, :]) / panels).ravel()
    wt = np.tile(0.5 * gw / panels, panels)
    u, wt = torch.from_numpy(u).to(DEV), torch.from_numpy(wt).to(DEV)
    zt, wd = torch.from_numpy(z).to(DEV)[:, None], torch.from_numpy(w).to(DEV)[:, None]
    cyc = u * ((-0.5 * zt + wd / 12) + u * (0.5 * (zt - 0.5 * wd) + u * (wd / 6)))
    g = torch.polar(wt.expand_as(cyc).contiguous(), 2 * math.pi * (cyc - torch.round(cyc)))
    out = []
    for phase in (0.0, 0.5):
        q = hmax - 1 - torch.arange(2 * hmax, device=DEV, dtype=torch.float64) + phase
        c = u[:, None] * q
        e = torch.polar(torch.ones_like(c), 2 * math.pi * (c - torch.round(c)))
        out.append(torch.matmul(g, e).conj())
    return torch.stack(out, 1)


def _windowed(c, t0, t1):
    """Taps of templates [t0, t1), zero outside each one's own window."""
    z, w, h = (a[t0:t1] for a in _lattice(c))
    hmax = int(h.max())
    taps = torch.cat([_exact_taps(z[i:i + 512], w[i:i + 512], hmax) for i in range(0, len(z), 512)])
    j = torch.arange(2 * hmax, device=DEV)
    ht = torch.from_numpy(h).to(DEV)[:, None]
    return taps * ((j >= hmax - ht) & (j < hmax + ht))[:, None, :], hmax


def _exact_rows(spec, taps, hmax):
    """Yields each template's power row (2n) in float64, by overlap-save in complex128."""
    n = spec.shape[0]
    seg = 1 << max(13, math.ceil(math.log2(8 * hmax)))
    keep = seg - 2 * hmax + 1
    nseg = (n + keep - 1) // keep
    x = torch.zeros(nseg * keep + seg, dtype=torch.complex128, device=DEV)
    x[hmax - 1:hmax - 1 + n] = spec
    f = torch.fft.fft(x.unfold(0, seg, keep)[:nseg])
    for t in taps:
        row = torch.empty((n, 2), dtype=torch.float64, device=DEV)
        for phase in (0, 1):
            y = torch.fft.ifft(f * torch.fft.fft(t[phase].conj(), seg).conj())[:, :keep].reshape(-1)[:n]
            row[:, phase] = y.real.square() + y.imag.square()
        yield row.reshape(-1)


def _exact_plane(spec, c, t0, t1):
    taps, hmax = _windowed(c, t0, t1)
    out = torch.empty((t1 - t0, 2 * spec.shape[0]), dtype=torch.float64, device=DEV)
    for i, row in enumerate(_exact_rows(spec, taps, hmax)):
        out[i] = row
    return out


def _exact_select(rows, c, n_rows):
    """Statistics and sorted candidates of the rows that `rows` yields."""
    cap = _capacity(c, n_rows)
    key = torch.full((cap,), 1 << 62, dtype=torch.int64, device=DEV)
    rec = torch.zeros((cap, 2), dtype=torch.float64, device=DEV)
    stats = torch.empty((n_rows, 2), dtype=torch.float64, device=DEV)
    at = 0
    for t, p in enumerate(rows):
        p = p.double()
        mean = p.mean()
        sigma = (p - mean).square().mean().sqrt()
        stats[t, 0], stats[t, 1] = mean, sigma
        hit = p > mean + c["k"] * sigma
        hit[1:] &= p[1:] > p[:-1]
        hit[:-1] &= p[:-1] >= p[1:]
        i = torch.nonzero(hit).reshape(-1)
        i = i[:max(0, cap - at)]
        key[at:at + len(i)] = (t << 32) | i
        rec[at:at + len(i), 0] = p[i]
        rec[at:at + len(i), 1] = (p[i] - mean) / sigma
        at += len(i)
    return stats, {"count": None, "key": None, "power_sigma": rec}


def exact(case, seed):
    c = dict(case)
    kind, n = c["kind"], c["n"]
    if kind == "spectrum":
        f = torch.fft.fft(_series(2 * n, seed, 0, 100.0, 300.0).double())[:n].clone()
        f[0] = 0
        return f / torch.sqrt(f.abs().square().sum() / (n - 1))
    if kind == "select":
        g = _generator(seed, 3)
        plane = torch.empty((c["rows"], 2 * n), dtype=torch.float32, device=DEV).exponential_(generator=g)
        stats, found = _exact_select(iter(plane), c, c["rows"])
        return {"stats": stats, **found}
    z, w, h = _lattice(c)
    if kind == "harmonics":
        g = _generator(seed, 5)
        plane = torch.empty((len(z), 2 * n), dtype=torch.float32, device=DEV).exponential_(generator=g)
        harm, nz = c["harm"], int(math.floor(c["zmax"] + 1e-9)) + 1
        i0, j0 = nz // 2, int(c["wmax"] // 20.0)
        npf = (2 * n - 1) // harm + 1
        rows = []
        for dj in range(-(j0 // harm), j0 // harm + 1):
            for di in range(-(i0 // harm), i0 // harm + 1):
                rows.append(sum(plane[(j0 + k * dj) * nz + i0 + k * di][::k][:npf].double() for k in range(1, harm + 1)))
        return torch.stack(rows)
    t0, t1 = _slab(c, {"n_templates": len(z)})
    if kind == "batch":
        return [_exact_plane(_spectrum(m, seed, 11 + i, c["zmax"], c["wmax"]), c, t0, t1)
                for i, m in enumerate(_lengths(c))]
    spec = _spectrum(n, seed, 7, c["zmax"], c["wmax"])
    if kind == "plane":
        return _exact_plane(spec, c, t0, t1)
    taps, hmax = _windowed(c, t0, t1)
    if kind == "candidates":
        return _exact_select(_exact_rows(spec, taps, hmax), c, t1 - t0)[1]
    out = {"power": torch.stack([r.max() for r in _exact_rows(spec, taps, hmax)]), "p": None}
    if kind == "cold_grid":
        out["taps"] = []
        for k in range(16, 2 * hmax + 16, 16):  # width classes of 16 taps
            at = [i for i in range(len(h)) if (2 * h[i] + 15) // 16 * 16 == k]
            if at:
                own = torch.zeros((len(at), 2, max(k, 2 * hmax)), dtype=torch.complex128, device=DEV)
                lo = (own.shape[2] - 2 * hmax) // 2
                own[:, :, lo:lo + 2 * hmax] = taps[torch.tensor(at, device=DEV)]
                lo = (own.shape[2] - k) // 2
                out["taps"].append(torch.view_as_real(own[:, :, lo:lo + k].contiguous()).reshape(-1))
    return out
