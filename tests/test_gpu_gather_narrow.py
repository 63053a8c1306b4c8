"""FP32 contraction of narrow data: channel counts at the edges of its
instantiations, few tiles (several wavefronts each) and many, short and long
supports, tiles much smaller and much larger than the support.

Tolerance: the FP32 path's 1e-6 (FP32 weights and results, FP64 sums)."""
import numpy as np
import pytest

import oracle
from gpu_util import make_gridder, say, to_device
from test_gpu_gather_wide import _check, _field

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nx,ny,n", [(9, 3, 1), (17, 65, 700), (257, 258, 9000)])
@pytest.mark.parametrize("nchan", [1, 2, 3, 8, 9, 16])
def test_channel_edges(nx, ny, n, nchan):
    wl = _field(nx, ny, n, nchan)
    ref = oracle.grid_workload(wl)
    lon, lat, d = to_device(wl)
    g = make_gridder(wl, "fp32")
    _check(*g.grid_datacube(lon, lat, d), wl, ref)
    g.clear()
    k = n // 2
    for a, b in ((0, k), (k, n)):
        if b > a:
            g.grid(lon[a:b], lat[a:b], d[a:b])
    _check(g.get_datacube(), g.get_weights(), wl, ref)


# support in pixels of 1': well below a pixel, and (600': the long distance
# series) far above a tile; a table and the elliptical kernel in both
@pytest.mark.parametrize("support", [0.05, 0.7, 60.0, 600.0])
@pytest.mark.parametrize("kind", ["gauss1d", "gauss2d", "tapered_sinc", "two_zeros", "table"])
@pytest.mark.parametrize("nx", [20, 257])
def test_supports_and_kernels(support, kind, nx):
    import dataclasses
    s = support / 60.0
    kernel = {"gauss1d": ("gauss1d", (s / 3.0,)), "gauss2d": ("gauss2d", (s / 3.0, s / 4.5, 30.0)),
              "tapered_sinc": ("tapered_sinc", (s / 3.0, s)),
              "two_zeros": ("tapered_sinc", (s / 3.0, s / 2.0)),   # sinc beyond its first zero
              "table": ("table", (s, 1.0, 0.8, 0.4, 0.1, 0.0))}[kind]
    n = 4000 if support < 100.0 or nx < 100 else 150
    wl = _field(nx, nx, n, 2, kernel=kernel)
    if support < 1.0:   # samples next to pixel centres, so that some are in the support
        rng = np.random.default_rng(5)
        tl, tb = (np.asarray(a) for a in oracle.targets_of(wl))
        p = rng.integers(0, tl.size, n)
        wl = dataclasses.replace(wl, lon=tl[p] + rng.normal(0.0, 0.4 * s, n) / np.cos(np.radians(30.0)),
                                 lat=tb[p] + rng.normal(0.0, 0.4 * s, n))
    wl = dataclasses.replace(wl, support=s)
    say(f"narrow gather support {support}' {kind} {nx}")
    ref = oracle.grid_workload(wl)
    lon, lat, d = to_device(wl)
    g = make_gridder(wl, "fp32", nside=8192 if support < 100.0 else 128)
    _check(*g.grid_datacube(lon, lat, d), wl, ref)


@pytest.mark.parametrize("nt", [70, 70000])
def test_targets_over_the_whole_sphere(nt):
    """Tiles whose targets (and supports) lie far apart, poles among them."""
    import torch
    import paper_1604_06667_amd as cgp
    rng = np.random.default_rng(nt)
    n = 3000
    sph = lambda k: (rng.uniform(0.0, 360.0, k), np.degrees(np.arcsin(rng.uniform(-1.0, 1.0, k))))
    lon, lat = sph(n)
    tl, tb = sph(nt)
    tb[:2] = 90.0, -90.0
    t = lambda a: torch.as_tensor(a, dtype=torch.float64, device="cuda:0")
    vals = rng.normal(1.0, 0.5, (n, 3))
    g = cgp.SlGrid(t(tl), t(tb), 3)
    g.set_kernel("gauss1d", (1.0,), 3.0, 0.5)
    cube, w = g.grid_datacube(t(lon), t(lat), t(vals))
    pick = np.concatenate([[0, 1], rng.integers(0, nt, 60)])
    v = lambda a, b: np.stack([np.cos(np.radians(b)) * np.cos(np.radians(a)),
                               np.cos(np.radians(b)) * np.sin(np.radians(a)), np.sin(np.radians(b))], -1)
    ch = np.linalg.norm(v(tl[pick], tb[pick])[:, None] - v(lon, lat)[None], axis=-1)
    d = np.degrees(2.0 * np.arcsin(np.minimum(1.0, 0.5 * ch)))
    assert np.abs(d - 3.0).min() > 1e-9
    k = np.where(d <= 3.0, np.exp(-0.5 * d * d), 0.0)
    W = k.sum(1)
    np.testing.assert_allclose(w.cpu().numpy()[pick], W, rtol=1e-6, atol=0)
    R = (k @ vals.astype(np.float32).astype(np.float64)) / np.where(W > 0, W, np.nan)[:, None]
    np.testing.assert_allclose(cube.cpu().numpy()[:, pick].T, R, rtol=2e-6, atol=1e-6)


def test_non_finite_values_stay_in_their_support():
    wl = _field(40, 40, 800, 3)
    lon, lat, d = to_device(wl)
    g = make_gridder(wl, "fp32")
    import torch
    clean, _ = g.grid_datacube(lon, lat, d)
    d[7, 1] = float("inf")
    cube, _ = g.grid_datacube(lon, lat, d)
    assert torch.equal(torch.nan_to_num(cube[0]), torch.nan_to_num(clean[0]))
    changed = (cube[1] != clean[1]) & torch.isfinite(clean[1])
    assert 0 < int(changed.sum()) <= 81 and not torch.isfinite(cube[1][changed]).any()
