"""FP32 contraction of wide data on the FP64 matrix cores: channel counts at
the edges of its workgroup shapes, maps with few and many tiles, the layouts
and accumulation modes, and non-finite values.

Tolerance: the FP32 path's 1e-6 (FP32 weights and results, FP64 sums)."""
import dataclasses

import numpy as np
import pytest

import oracle
import synth
from gpu_util import flat, make_gridder, say, to_device

pytestmark = pytest.mark.gpu
TOL32 = 1e-6


def _wcs(nx, ny, pix):
    return {"kind": "wcs", "wcs": {"proj": "SIN", "naxis1": nx, "naxis2": ny, "crpix1": 0.5 * (nx + 1),
                                   "crpix2": 0.5 * (ny + 1), "crval1": 120.0, "crval2": 30.0,
                                   "cdelt1": -pix, "cdelt2": pix}}


def _field(nx, ny, n, nchan, dtype="f32", kernel=("gauss1d", (1.5 / 60.0,))):
    import torch
    rng = np.random.default_rng(nx * 1000 + nchan)
    pix = 1.0 / 60.0
    lon = 120.0 + (rng.random(n) - 0.5) * nx * pix / np.cos(np.radians(30.0))
    lat = 30.0 + (rng.random(n) - 0.5) * ny * pix
    data = torch.as_tensor(rng.normal(1.0, 0.5, (n, nchan)).astype(np.float32))
    if dtype == "f64":
        data = data.to(torch.float64)
    base = synth.config2(scale=0.02, nchan=4)
    return dataclasses.replace(base, lon=lon, lat=lat, data=data, dtype=dtype, target=_wcs(nx, ny, pix),
                               kernel=kernel, support=4.5 / 60.0, hpx_maxres=0.75 / 60.0)


def check_signed(cube, w, wl, ref, tol):
    """For kernels with negative parts, where the weights of a target may cancel
    (or sum to less than zero: no value): weights and weighted sums against
    the number of samples in the support, which bounds the sum of their sizes."""
    lon, lat = oracle.targets_of(wl)
    n = np.maximum(oracle.neighbour_sets(wl.lon, wl.lat, lon, lat, wl.support)["count"], 1)
    W, got = ref["W"], w.cpu().numpy().astype(np.float64).ravel()
    assert np.all(np.abs(got - W) <= 1e-6 * n)
    ok = (W > 1e-6 * n) & (got > 0)
    R = flat(cube, wl.nchan)
    top = np.abs(np.asarray(wl.data.double())).max()
    d = np.abs(R[:, ok] * got[ok] - np.asarray(ref["R"]).reshape(wl.nchan, -1)[:, ok] * W[ok])
    assert np.all(d <= tol * n[ok] * top)


def _check(cube, w, wl, ref):
    if wl.kernel[0] == "tapered_sinc" and wl.kernel[1][1] < wl.support:
        return check_signed(cube, w, wl, ref, TOL32)
    ev = oracle.e_val(flat(cube, wl.nchan), ref["R"], ref["W"])
    ew = oracle.e_weights(w.cpu().numpy().astype(np.float64).ravel(), ref["W"])
    say(f"  e_val={ev:.2e} e_W={ew:.2e}")
    assert ev <= TOL32 and ew <= TOL32


# few tiles: 64-channel workgroups splitting the candidates; many tiles: two
# and four channel blocks to a workgroup
@pytest.mark.parametrize("nx,ny,n,nchan", [
    (9, 3, 1, 17), (17, 9, 31, 64), (17, 9, 33, 65), (25, 24, 700, 128), (33, 31, 1500, 257),
    (190, 188, 9000, 17), (190, 188, 9000, 65), (190, 188, 9000, 128), (190, 188, 9000, 131)])
def test_channel_edges(nx, ny, n, nchan):
    wl = _field(nx, ny, n, nchan)
    say(f"wide gather {nx}x{ny} n={n} nchan={nchan}")
    ref = oracle.grid_workload(wl)
    lon, lat, d = to_device(wl)
    g = make_gridder(wl, "fp32")
    _check(*g.grid_datacube(lon, lat, d), wl, ref)
    # two scans accumulate to the same result
    g.clear()
    k = n // 2
    for a, b in ((0, k), (k, n)):
        if b > a:
            g.grid(lon[a:b], lat[a:b], d[a:b])
    _check(g.get_datacube(), g.get_weights(), wl, ref)
    g.set_output_layout("target")
    cube, w = g.grid_datacube(lon, lat, d)
    _check(cube.permute(2, 0, 1).contiguous(), w, wl, ref)


@pytest.mark.parametrize("kernel", [("gauss2d", (1.5 / 60.0, 1.0 / 60.0, 30.0)),
                                    ("tapered_sinc", (1.5 / 60.0, 4.5 / 60.0)),
                                    ("tapered_sinc", (1.5 / 60.0, 2.25 / 60.0)),
                                    ("table", (4.5 / 60.0, 1.0, 0.8, 0.4, 0.1, 0.0))],
                         ids=["gauss2d", "tapered_sinc", "two_zeros", "table"])
@pytest.mark.parametrize("nx,nchan", [(30, 70), (190, 140)])
def test_kernels(kernel, nx, nchan):
    wl = _field(nx, nx, 20 * nx, nchan, kernel=kernel)
    ref = oracle.grid_workload(wl)
    lon, lat, d = to_device(wl)
    g = make_gridder(wl, "fp32", nside=4096)
    _check(*g.grid_datacube(lon, lat, d), wl, ref)


@pytest.mark.parametrize("dtype", ["f32", "f64"])
@pytest.mark.parametrize("nx,nchan", [(30, 70), (190, 140)])
def test_unaligned_rows(nx, nchan, dtype):
    """Rows that do not start on a vector boundary."""
    import torch
    wl = _field(nx, nx, 20 * nx, nchan, dtype=dtype)
    ref = oracle.grid_workload(wl)
    lon, lat, d = to_device(wl)
    wide = torch.zeros((d.shape[0], nchan + 3), dtype=d.dtype, device=d.device)
    wide[:, 1:1 + nchan] = d
    g = make_gridder(wl, "fp32")
    _check(*g.grid_datacube(lon, lat, wide[:, 1:1 + nchan]), wl, ref)


@pytest.mark.parametrize("nx,nchan", [(30, 70), (190, 140)])
def test_non_finite_values_stay_in_their_support(nx, nchan):
    """A sample's inf or NaN reaches the targets that have the sample in their
    support, in its own channel, and no others."""
    import torch
    wl = _field(nx, nx, 20 * nx, nchan)
    lon, lat, d = to_device(wl)
    g = make_gridder(wl, "fp32")
    clean, w0 = g.grid_datacube(lon, lat, d)
    dirty = d.clone()
    rows, chans = [3, 50, 51, 400], [0, nchan - 1, 33, 64]
    for r, c, v in zip(rows, chans, [float("inf"), float("nan"), float("-inf"), float("nan")]):
        dirty[r, c] = v
    cube, w = g.grid_datacube(lon, lat, dirty)
    assert torch.equal(w, w0)
    tl, tb = (np.asarray(a) for a in oracle.targets_of(wl))
    for c in range(nchan):
        hit = np.zeros(nx * nx, dtype=bool)
        for r, cc in zip(rows, chans):
            if cc == c:
                a, b = np.radians(tl - wl.lon[r]), (np.radians(tb), np.radians(wl.lat[r]))
                cosd = np.sin(b[0]) * np.sin(b[1]) + np.cos(b[0]) * np.cos(b[1]) * np.cos(a)
                hit |= np.degrees(np.arccos(np.clip(cosd, -1, 1))) <= wl.support
        got = cube[c].reshape(-1).cpu().numpy()
        ref = clean[c].reshape(-1).cpu().numpy()
        assert np.array_equal(np.isfinite(got), np.isfinite(ref) & ~hit), c
        ok = np.isfinite(got)
        # the matrix products run over the same values in the same order
        assert np.array_equal(got[ok], ref[ok]), c
