"""Timed cases of the gridding library: the calls a user of it makes, from the
smallest map to the largest spectral survey, through the public entry points.

A case is a dict of plain values:

    call     'datacube' (clear + grid + normalise in one call), 'scans' (one
             grid() per scan, then get_datacube / get_weights), 'batch' (many
             jobs in one call) or 'replay' (the same, tuned and captured)
    target   'CAR' | 'SIN' | 'SFL' | 'ZEA' (FITS/WCS maps of nx x ny pixels),
             'sightlines' (nt positions) or 'healpix' (every pixel of nside)
    pix      pixel size (arcmin); sight lines: mean spacing of the targets
    n, chan  samples and channels; dtype of the data as delivered
    scan     'raster' (jittered scan lines, in time order) or 'random'
    prec     'fp32' (default), 'bf16' or 'fp16'
    kernel   'gauss1d', 'gauss2d', 'tapered_sinc' or 'table', of width
             sigma (arcmin), cut at support x sigma
    layout   'channel' or 'target' order of the cube
    scans    number of grid() calls of a 'scans' case
    jobs, mix  number of jobs of a batch, and which mix of sizes

Positions, values and sight lines come from the seed alone.
"""
import math
import random

import numpy as np
import torch

import paper_1604_06667_amd as cg

DEV = "cuda:0"
DEG = math.pi / 180.0
DTYPE = {"f64": torch.float64, "f32": torch.float32, "f16": torch.float16, "bf16": torch.bfloat16}
SIZE = {"f64": 8, "f32": 4, "f16": 2, "bf16": 2}


def case(name=None, **k):
    c = {"call": "datacube", "target": "SIN", "nx": 0, "ny": 0, "nt": 0, "nside": 0, "pix": 1.0,
         "n": 0, "chan": 1, "dtype": "f32", "scan": "random", "prec": "fp32", "kernel": "gauss1d",
         "sigma": 1.5, "support": 3.0, "layout": "channel", "scans": 1, "jobs": 0, "mix": 0}
    c.update(k)
    return c if name is None else dict(c, name=name)


def listed():
    return [
        # The smallest call: a cut-out of a few pixels around a source, where
        # the launches are what counts.
        case("tiny", target="SIN", nx=17, ny=65, n=3000, chan=2, dtype="f64"),
        # One ordinary single-channel map, as an interactive user grids it.
        case("map", target="CAR", nx=96, ny=96, pix=2.0, n=20000, chan=1, dtype="f64"),
        # A map from dense parallel scan lines with a wide 5-sigma support:
        # many pairs per pixel, few pixels.
        case("stripes", target="SFL", nx=151, ny=151, pix=0.6, n=22600, chan=1, scan="raster",
             sigma=1.27, support=5.0),
        # An all-sky survey in a few bands onto a plate carree map, poles and
        # seam included.
        case("allsky", target="CAR", nx=4320, ny=2160, pix=5.0, n=12_000_000, chan=8, sigma=6.0),
        # All-sky signal and noise onto a HEALPix map, 15 samples a pixel:
        # the largest number of samples, where the lookup weighs as much as
        # the sums.
        case("healpix", target="healpix", nside=512, pix=6.87, n=47_185_920, chan=2, sigma=5.82),
        # The spectral cube of a single-dish survey field on the matrix cores.
        case("cube-bf16", nx=600, ny=600, n=1_000_000, chan=1024, scan="raster", prec="bf16"),
        # The same cube in the default precision.
        case("cube-fp32", nx=600, ny=600, n=1_000_000, chan=1024, scan="raster"),
        # Half-precision spectra of a ragged channel count on an equal-area
        # map, single-product matrix-core mode.
        case("cube-fp16", target="ZEA", nx=397, ny=311, pix=1.3, n=300_000, chan=500, dtype="f16",
             prec="fp16", sigma=1.8),
        # A medium field of few channels on the matrix cores (continuum
        # sub-bands), spectra contiguous in the result.
        case("subbands-bf16", nx=700, ny=500, n=400_000, chan=48, prec="bf16", layout="target"),
        # Spectra at millions of positions of a catalogue (elliptical beam).
        case("sightlines-bf16", target="sightlines", nt=2_000_000, pix=1.27, n=10_000_000, chan=256,
             dtype="bf16", prec="bf16", kernel="gauss2d", sigma=3.0, layout="target"),
        # A survey gridded scan by scan into one accumulating cube (default
        # precision, elliptical beam).
        case("scans-fp32", call="scans", scans=8, nx=301, ny=257, n=320_000, chan=60, scan="raster",
             kernel="gauss2d", sigma=2.0),
        # Many small fields of very different sizes in one call.
        case("batch", call="batch", jobs=16, mix=4, dtype="bf16", prec="bf16"),
    ]


def _log(rng, lo, hi):
    return math.exp(rng.uniform(math.log(lo), math.log(hi)))


def draw(rng):
    kind = rng.choice(["map", "map", "cube", "cube", "cube", "sightlines", "healpix", "scans", "batch",
                       "replay"])
    if kind in ("batch", "replay"):
        return case(call=kind, jobs=rng.randint(3, 16), mix=rng.randint(5, 10_000), dtype="bf16", prec="bf16")
    kernel = rng.choice(["gauss1d", "gauss1d", "gauss1d", "gauss2d", "gauss2d", "tapered_sinc", "table"])
    layout = rng.choice(["channel", "channel", "target"])
    ratio = rng.uniform(0.9, 2.0)            # sigma over the pixel size
    support = rng.choice([3.0, 3.0, 4.0, 5.0])
    if kind == "map":
        pix = rng.uniform(0.5, 5.0)
        nx = int(_log(rng, 9, min(1500.0, 2000.0 / pix)))
        ny = max(3, int(nx * rng.uniform(0.4, 1.6)))
        n = int(min(4e6, max(500, nx * ny * _log(rng, 0.5, 12))))
        return case(target=rng.choice(["CAR", "SIN", "SFL", "ZEA"]), nx=nx, ny=ny, pix=pix, n=n,
                    chan=rng.randint(1, 16), dtype=rng.choice(["f64", "f32"]), kernel=kernel,
                    scan=rng.choice(["raster", "random"]), sigma=ratio * pix, support=support, layout=layout)
    if kind == "healpix":
        nside = rng.choice([16, 32, 64, 128, 256, 512])
        pix = 60.0 * math.degrees(math.sqrt(math.pi / 3.0)) / nside
        return case(target="healpix", nside=nside, pix=pix, n=int(12 * nside * nside * _log(rng, 1, 12)),
                    chan=rng.randint(1, 5), kernel=kernel, sigma=rng.uniform(0.7, 1.0) * pix, layout=layout)
    chan = int(_log(rng, 17, 1100))
    prec = rng.choice(["fp32", "bf16", "bf16", "fp16"])
    dtype = rng.choice(["f32", "f32", "bf16", "f16", "f64"])
    if kind == "sightlines":
        pix = rng.uniform(0.8, 3.0)
        nt = int(_log(rng, 500, 300_000))
        n = int(min(2e6, 1.5e9 / chan, max(2000, nt * _log(rng, 1, 8))))
        return _capped(case(target="sightlines", nt=nt, pix=pix, n=n, chan=min(chan, 400), dtype=dtype,
                            prec=prec, kernel=kernel, sigma=ratio * pix, layout=layout))
    pix = rng.uniform(0.5, 3.0)
    nx = int(_log(rng, 24, 500))
    ny = max(5, int(nx * rng.uniform(0.5, 1.2)))
    n = int(min(1.2e6, 8e8 / chan, max(1000, nx * ny * _log(rng, 0.7, 8))))
    c = case(target=rng.choice(["SIN", "ZEA", "CAR"]), nx=nx, ny=ny, pix=pix, n=n, chan=chan, dtype=dtype,
             prec=prec, kernel=kernel, scan=rng.choice(["raster", "random"]), sigma=ratio * pix, layout=layout)
    if kind == "scans":
        c.update(call="scans", scans=rng.randint(2, 12))
    return _capped(c)


def _capped(c, flops=1.0e11):
    """The case with fewer samples where it would cost more than the listed ones."""
    f = work(c)["flops"]
    return c if f <= flops else dict(c, n=max(500, int(c["n"] * flops / f)))


# ------------------------------------------------------------------- geometry

def _jobs(c):
    """The jobs of a batch: sizes from the mix number alone."""
    r = random.Random(1000 + int(c["mix"]))
    out = []
    for _ in range(int(c["jobs"])):
        side = int(_log(r, 64, 512))
        sigma = r.uniform(1.0, 4.0)
        out.append(_capped(case(nx=side, ny=side, pix=r.uniform(0.5, 3.0), n=int(_log(r, 5e3, 3e5)),
                                chan=int(_log(r, 16, 1500)), dtype="bf16", prec="bf16",
                                kernel="gauss2d" if r.random() < 0.25 else "gauss1d", sigma=sigma), 5.0e10))
    return out


def _centre(c):
    if c["target"] == "CAR" and c["nx"] * c["pix"] > 20000:
        return 0.0, 0.0
    return (120.0, 0.0) if c["target"] in ("CAR", "SFL") else (120.0, 30.0)


def _header(c):
    lon0, lat0 = _centre(c)
    return {"NAXIS": 3, "NAXIS1": c["nx"], "NAXIS2": c["ny"], "NAXIS3": c["chan"],
            "CTYPE1": "RA---" + c["target"], "CTYPE2": "DEC--" + c["target"],
            "CRPIX1": 0.5 * (c["nx"] + 1), "CRPIX2": 0.5 * (c["ny"] + 1), "CRVAL1": lon0, "CRVAL2": lat0,
            "CDELT1": -c["pix"] / 60.0, "CDELT2": c["pix"] / 60.0}


def _table():
    """A smooth radial profile that ends at the support."""
    d = np.linspace(0.0, 1.0, 257)
    return ((1.0 - d * d) * np.exp(-3.0 * d * d)).tolist()


def _kernel(c):
    """(kind, params, support, hpx_maxres), all in degrees."""
    s = c["sigma"] / 60.0
    rs = c["support"] * s
    if c["kernel"] == "gauss2d":
        return "gauss2d", (s, s * 2.0 / 3.0, 30.0), rs, s / 3.0
    if c["kernel"] == "tapered_sinc":
        return "tapered_sinc", (s, rs), rs, 0.5 * s     # first zero at the edge
    if c["kernel"] == "table":
        return "table", (rs, *_table()), rs, 0.5 * s
    return "gauss1d", (s,), rs, 0.5 * s


def _gen(seed, salt):
    g = torch.Generator(device=DEV)
    g.manual_seed((int(seed) * 1000003 + 7919 * salt) % (1 << 62))
    return g


def _rand(g, n):
    return torch.rand(n, generator=g, device=DEV, dtype=torch.float64)


def _sphere(g, n):
    return 360.0 * _rand(g, n), torch.rad2deg(torch.asin(2.0 * _rand(g, n) - 1.0))


def _place(lon0, lat0, x, y):
    """Points at the offsets (x east, y north, degrees) on the tangent plane."""
    a, d = lon0 * DEG, lat0 * DEG
    tx, ty = torch.tan(x * DEG), torch.tan(y * DEG)
    px = math.cos(d) * math.cos(a) - math.sin(a) * tx - math.sin(d) * math.cos(a) * ty
    py = math.cos(d) * math.sin(a) + math.cos(a) * tx - math.sin(d) * math.sin(a) * ty
    pz = math.sin(d) + math.cos(d) * ty
    lon = torch.rad2deg(torch.atan2(py, px)) % 360.0
    return lon, torch.rad2deg(torch.atan2(pz, torch.sqrt(px * px + py * py)))


def _span(c):
    """Width and height (degrees) of the sampled field."""
    if c["target"] == "sightlines":
        s = math.sqrt(c["nt"]) * c["pix"] / 60.0
        return s, s
    return c["nx"] * c["pix"] / 60.0, c["ny"] * c["pix"] / 60.0


def _whole_sky(c):
    return c["target"] == "healpix" or (c["target"] == "CAR" and c["nx"] * c["pix"] > 20000)


def _positions(c, seed):
    n = c["n"]
    g = _gen(seed, 1)
    if _whole_sky(c):
        return _sphere(g, n)
    w, h = _span(c)
    if c["scan"] == "raster":
        rows = max(2, int(round(math.sqrt(n * h / w * 0.6))))
        per = -(-n // rows)
        k = torch.arange(n, device=DEV)
        x = ((k % per).double() / max(1, per - 1) - 0.5) * w
        y = ((k // per).double() / max(1, rows - 1) - 0.5) * h
        j = 0.2 * c["pix"] / 60.0
        x = x + j * torch.randn(n, generator=g, device=DEV, dtype=torch.float64)
        y = y + j * torch.randn(n, generator=g, device=DEV, dtype=torch.float64)
    else:
        x = (_rand(g, n) - 0.5) * w
        y = (_rand(g, n) - 0.5) * h
    lon0, lat0 = _centre(c)
    return _place(lon0, lat0, x, y)


def _sightlines(c, seed):
    g = _gen(seed, 2)
    w, h = _span(c)
    lon0, lat0 = _centre(c)
    return _place(lon0, lat0, (_rand(g, c["nt"]) - 0.5) * w, (_rand(g, c["nt"]) - 0.5) * h)


def _values(c, seed, lon, lat):
    """Spectra: a line whose strength and centre vary over the field, on a
    sloping continuum, with noise."""
    n, chan = c["n"], c["chan"]
    g = _gen(seed, 3)
    out = torch.empty((n, chan), dtype=DTYPE[c["dtype"]], device=DEV)
    ch = torch.arange(chan, device=DEV, dtype=torch.float32)[None, :]
    step = max(1, (1 << 27) // chan)
    for s in range(0, n, step):
        e = min(n, s + step)
        x, y = lon[s:e].float()[:, None] * 1.7, lat[s:e].float()[:, None] * 2.3
        amp = 1.0 + torch.sin(x) * torch.cos(y)
        mid = chan * (0.5 + 0.3 * torch.sin(0.5 * x + y))
        v = 0.05 * torch.randn((e - s, chan), generator=g, device=DEV)
        v += amp * torch.exp(-((ch - mid) / (0.04 * chan + 1.0)) ** 2)
        v += 0.3 + 0.1 * torch.cos(y)
        out[s:e] = v.to(out.dtype)
    return out


# ------------------------------------------------------------------ the calls

def _gridder(c, seed):
    if c["target"] == "healpix":
        g = cg.HpxGrid(c["nside"], "ring", c["chan"])
    elif c["target"] == "sightlines":
        g = cg.SlGrid(*_sightlines(c, seed), c["chan"])
    else:
        g = cg.WcsGrid(_header(c))
    kind, params, rs, res = _kernel(c)
    g.set_kernel(kind, params, rs, res)
    g.set_precision(c["prec"])
    g.set_output_layout(c["layout"])
    return g


def _inputs(c, seed):
    lon, lat = _positions(c, seed)
    return lon, lat, _values(c, seed, lon, lat)


def prepare(c, seed):
    """Device arrays of the samples and the gridder a program keeps."""
    if c["call"] in ("batch", "replay"):
        jobs = _jobs(c)
        gs = [_gridder(j, seed + 31 * k) for k, j in enumerate(jobs)]
        ins = [_inputs(j, seed + 31 * k) for k, j in enumerate(jobs)]
        b = cg.Batch(gs, torch.bfloat16)
        outs = b.outputs()
        if c["call"] == "replay":
            b.tune(ins, outs)
            b.capture(ins, outs)
        return {"call": c["call"], "batch": b, "ins": ins, "outs": outs}
    lon, lat, data = _inputs(c, seed)
    s = {"call": c["call"], "g": _gridder(c, seed), "ins": (lon, lat, data)}
    if c["call"] == "scans":
        cut = [c["n"] * k // c["scans"] for k in range(c["scans"] + 1)]
        s["ins"] = [(lon[a:b], lat[a:b], data[a:b]) for a, b in zip(cut, cut[1:])]
    return s


def run(s):
    if s["call"] == "batch":
        s["batch"].grid(s["ins"], s["outs"])
        return s["outs"]
    if s["call"] == "replay":
        s["batch"].replay()
        return s["outs"]
    g = s["g"]
    if s["call"] == "scans":
        g.clear()
        for lon, lat, data in s["ins"]:
            g.grid(lon, lat, data)
        return g.get_datacube(), g.get_weights()
    return g.grid_datacube(*s["ins"])


def _targets(c):
    if c["target"] == "sightlines":
        return c["nt"]
    return 12 * c["nside"] ** 2 if c["target"] == "healpix" else c["nx"] * c["ny"]


def work(c):
    """Coordinates and data read once, cube and weights written once; per
    sample and target within the support the distance and, per channel, one
    multiply and one add."""
    if c["call"] in ("batch", "replay"):
        w = [work(j) for j in _jobs(c)]
        return {k: sum(x[k] for x in w) for k in ("bytes", "flops")}
    nt = _targets(c)
    if _whole_sky(c):
        area = 41252.96
    else:
        w, h = _span(c)
        area = w * h
    rs = c["support"] * c["sigma"] / 60.0
    pairs = float(c["n"]) * nt * min(1.0, math.pi * rs * rs / area)
    return {"bytes": c["n"] * (16.0 + c["chan"] * SIZE[c["dtype"]]) + nt * (c["chan"] * 4.0 + 4.0),
            "flops": pairs * (2.0 * c["chan"] + 12.0)}


# ------------------------------------------- the same results in 64 bits, plain

def _xyz(lon, lat):
    a, d = lon * DEG, lat * DEG
    return torch.stack([torch.cos(d) * torch.cos(a), torch.cos(d) * torch.sin(a), torch.sin(d)], 1)


def _target_lonlat(c, seed):
    """Target positions in output order; NaN outside a projection."""
    if c["target"] == "sightlines":
        return _sightlines(c, seed)
    if c["target"] == "healpix":
        ns = c["nside"]
        i = torch.arange(1, 4 * ns, device=DEV, dtype=torch.float64)
        cap = torch.minimum(i, 4.0 * ns - i)
        polar = cap < ns
        count = torch.where(polar, 4 * cap, torch.full_like(i, 4.0 * ns)).long()
        z = torch.where(polar, torch.sign(2.0 * ns - i) * (1.0 - cap * cap / (3.0 * ns * ns)),
                        4.0 / 3.0 - 2.0 * i / (3.0 * ns))
        shift = torch.where(polar | ((i.long() - ns) % 2 == 0), 0.5, 0.0).double()
        ring = torch.repeat_interleave(torch.arange(4 * ns - 1, device=DEV), count)
        first = torch.cumsum(count, 0) - count
        j = torch.arange(ring.numel(), device=DEV) - first[ring]
        # near the poles asin(z) loses digits: 1 - |z| = cap^2 / 3 nside^2 there
        s2 = torch.where(polar, cap * cap / (3.0 * ns * ns) * (2.0 - cap * cap / (3.0 * ns * ns)), 1.0 - z * z)
        lat = torch.rad2deg(torch.atan2(z, torch.sqrt(s2)))
        return 360.0 * (j.double() + shift[ring]) / count[ring].double(), lat[ring]
    lon0, lat0 = _centre(c)
    p = torch.arange(c["nx"] * c["ny"], device=DEV)
    x = -((p % c["nx"]).double() + 1.0 - 0.5 * (c["nx"] + 1)) * c["pix"] / 60.0
    y = ((p // c["nx"]).double() + 1.0 - 0.5 * (c["ny"] + 1)) * c["pix"] / 60.0
    nan = torch.full_like(x, math.nan)
    if c["target"] in ("CAR", "SFL"):
        dl = x if c["target"] == "CAR" else x / torch.cos(y * DEG)
        out = (y.abs() > 90.0) | ((dl.abs() > 180.0) & torch.tensor(c["target"] == "SFL", device=DEV))
        return torch.where(out, nan, (lon0 + dl) % 360.0), torch.where(out, nan, y)
    r = torch.sqrt(x * x + y * y) * DEG
    if c["target"] == "SIN":
        out = r > 1.0
        sr, cr = r.clamp(max=1.0), torch.sqrt((1.0 - r * r).clamp(min=0.0))
    else:
        out = r > 2.0
        cr = 1.0 - 0.5 * r * r
        sr = r * torch.sqrt((1.0 - 0.25 * r * r).clamp(min=0.0))
    # direction on the sky: cr along the centre, sr towards (x east, y north)
    f = torch.where(r > 0.0, sr / r.clamp(min=1e-300), torch.ones_like(r)) * DEG
    a, d = lon0 * DEG, lat0 * DEG
    px = cr * math.cos(d) * math.cos(a) - f * x * math.sin(a) - f * y * math.sin(d) * math.cos(a)
    py = cr * math.cos(d) * math.sin(a) + f * x * math.cos(a) - f * y * math.sin(d) * math.sin(a)
    pz = cr * math.sin(d) + f * y * math.cos(d)
    lon = torch.rad2deg(torch.atan2(py, px)) % 360.0
    lat = torch.rad2deg(torch.atan2(pz, torch.sqrt(px * px + py * py)))
    return torch.where(out, nan, lon), torch.where(out, nan, lat)


def _weights64(c, t, s, tlon, tlat):
    """Kernel weights [targets][samples] of unit vectors t, s."""
    e = [s[None, :, k] - t[:, None, k] for k in range(3)]
    c2 = e[0] * e[0] + e[1] * e[1] + e[2] * e[2]
    d = 2.0 * torch.asin(0.5 * torch.sqrt(c2).clamp(max=2.0))
    sig = c["sigma"] / 60.0 * DEG
    rs = c["support"] * sig
    if c["kernel"] == "gauss1d":
        w = torch.exp(-0.5 * (d / sig) ** 2)
    elif c["kernel"] == "tapered_sinc":
        w = torch.exp(-0.5 * (d / sig) ** 2) * torch.sinc(d / rs)
    elif c["kernel"] == "table":
        tab = torch.tensor(_table(), device=DEV, dtype=torch.float64)
        u = (d / rs * 256.0).clamp(max=256.0)
        k = u.floor().clamp(max=255.0).long()
        w = tab[k] + (u - k) * (tab[k + 1] - tab[k])
    else:
        a, b = tlon * DEG, tlat * DEG
        east = (-torch.sin(a), torch.cos(a), torch.zeros_like(a))
        north = (-torch.sin(b) * torch.cos(a), -torch.sin(b) * torch.sin(a), torch.cos(b))
        xe = sum(e[k] * east[k][:, None] for k in range(3))
        yn = sum(e[k] * north[k][:, None] for k in range(3))
        q = torch.atan2(xe, yn) - 30.0 * DEG
        w = torch.exp(-0.5 * d * d * ((torch.cos(q) / sig) ** 2 + (1.5 * torch.sin(q) / sig) ** 2))
    return torch.where(d <= rs, w, torch.zeros_like(w))


def _exact_one(c, seed):
    lon, lat = _positions(c, seed)
    data = _values(c, seed, lon, lat)
    tlon, tlat = _target_lonlat(c, seed)
    nt, chan = tlon.numel(), c["chan"]
    order = torch.argsort(lat)
    slat = lat[order]
    sxyz = _xyz(lon, lat)[order]
    txyz = _xyz(tlon, tlat)
    rs = c["support"] * c["sigma"] / 60.0
    # blocks of targets: latitude bands of height h cut in longitude
    h = max(8.0 * rs, 1e-3)
    ok = torch.isfinite(tlon)
    band = torch.where(ok, torch.floor((tlat + 90.0) / h), torch.full_like(tlat, -1.0))
    mid = ((band + 0.5) * h - 90.0).clamp(-90.0, 90.0) * DEG
    bins = torch.clamp(torch.floor(360.0 * torch.cos(mid) / h), min=1.0)
    key = (band * 1e6 + torch.floor(tlon / 360.0 * bins).clamp(min=0.0)).nan_to_num(-1e6)
    torder = torch.argsort(key, stable=True)
    vals, counts = torch.unique_consecutive(key[torder], return_counts=True)
    ends = torch.cumsum(counts, 0).cpu().tolist()
    keep = (vals >= 0).cpu().tolist()
    cube = torch.full((nt, chan), math.nan, dtype=torch.float32 if nt * chan > 1 << 27 else torch.float64,
                      device=DEV)
    wsum = torch.zeros(nt, dtype=torch.float64, device=DEV)
    tl = tlat[torder]
    start = 0
    lows = torch.searchsorted(slat, (tl - rs - 1e-6)).cpu()
    highs = torch.searchsorted(slat, (tl + rs + 1e-6), right=True).cpu()
    for end, good in zip(ends, keep):
        a, start = start, end
        if not good:
            continue
        lo, hi = int(lows[a:end].min()), int(highs[a:end].max())
        if hi <= lo:
            continue
        t_all = torder[a:end]
        p = txyz[t_all]
        m = p.mean(0)
        m = m / m.norm()
        reach = float(torch.asin(((p - m).norm(dim=1).max() * 0.5).clamp(max=1.0))) * 2.0 + rs * DEG + 1e-9
        cand = lo + torch.nonzero(sxyz[lo:hi] @ m >= math.cos(min(reach, math.pi)))[:, 0]
        if not cand.numel():
            continue
        s, rows = sxyz[cand], data[order[cand]].double()
        per = max(1, int(6e7) // cand.numel())
        for q in range(0, t_all.numel(), per):
            t = t_all[q:q + per]
            w = _weights64(c, txyz[t], s, tlon[t], tlat[t])
            tot = w.sum(1)
            wsum[t] = tot
            r = (w @ rows) / tot[:, None]
            r[tot <= 0.0] = math.nan
            cube[t] = r.to(cube.dtype)
    shape = (nt,) if c["target"] in ("sightlines", "healpix") else (c["ny"], c["nx"])
    if c["layout"] == "target":
        return cube.reshape(*shape, chan), wsum.reshape(shape)
    return cube.T.reshape(chan, *shape), wsum.reshape(shape)


def exact(c, seed):
    if c["call"] in ("batch", "replay"):
        return [_exact_one(j, seed + 31 * k) for k, j in enumerate(_jobs(c))]
    return _exact_one(c, seed)
