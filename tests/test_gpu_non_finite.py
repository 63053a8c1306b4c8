"""Non-finite values in the wide FP32 gather: which targets become NaN, +inf or
-inf, by the sign of the weights, in each workgroup shape and with more chunks
of candidates than the mask of chunks has bits; all other results are bitwise
those of the clean data."""
import numpy as np
import pytest

from gpu_util import make_gridder, say, to_device
from test_gpu_gather_wide import _field

pytestmark = pytest.mark.gpu
SINC = ("tapered_sinc", (1.5 / 60.0, 2.25 / 60.0))   # negative beyond 2.25'


def _near(wl, row):
    """Targets within the support of a sample, and the sign of its weight there."""
    import oracle
    tl, tb = (np.radians(np.asarray(a)) for a in oracle.targets_of(wl))
    sl, sb = np.radians(wl.lon[row]), np.radians(wl.lat[row])
    h = np.sin((tb - sb) / 2) ** 2 + np.cos(tb) * np.cos(sb) * np.sin((tl - sl) / 2) ** 2
    d = np.degrees(2.0 * np.arcsin(np.sqrt(h)))
    sign = np.ones_like(d)
    if wl.kernel[0] == "tapered_sinc":
        sign = np.sign(np.sinc(d / wl.kernel[1][1]))
    return d <= wl.support, sign


# workgroups of 1 x 8, 1 x 4, 2 x 2 and 4 x 1 wavefronts; then tiles of more
# than 64 chunks to a wavefront
@pytest.mark.parametrize("nx,n,nchan", [(30, 600, 70), (190, 3800, 20), (190, 3800, 100), (190, 3800, 140),
                                        (10, 60000, 20), (190, 300000, 140)])
@pytest.mark.parametrize("kernel,dtype", [(("gauss1d", (1.5 / 60.0,)), "f32"), (SINC, "f32"), (SINC, "f16"),
                                          (("gauss1d", (1.5 / 60.0,)), "f64")],
                         ids=["gauss", "sinc", "sinc-f16", "gauss-f64"])
def test_kinds(nx, n, nchan, kernel, dtype):
    import torch
    dt = {"f32": torch.float32, "f16": torch.float16, "f64": torch.float64}[dtype]
    wl = _field(nx, nx, n, nchan, kernel=kernel)
    lon, lat, d = to_device(wl)
    d = d.to(dt)
    g = make_gridder(wl, "fp32", nside=2048)
    clean, w0 = g.grid_datacube(lon, lat, d)
    inf, nan = float("inf"), float("nan")
    rows = [3, 50, 51, n // 2, n // 2 + 1, n - 2, n - 1]
    # a neighbour of the first row, with an infinity of the other sign in its channel
    near = int(np.argsort((wl.lon - wl.lon[3]) ** 2 + (wl.lat - wl.lat[3]) ** 2)[1])
    put = list(zip(rows, [0, nchan - 1, 0, 7, 7, 16, nchan - 1], [inf, nan, -inf, -inf, nan, inf, -inf]))
    put.append((near, 0, -inf))
    dirty = d.clone()
    for r, c, v in put:
        dirty[r, c] = v
    say(f"non-finite {nx}x{nx} n={n} nchan={nchan} {kernel[0]} {dtype}")
    cube, w = g.grid_datacube(lon, lat, dirty)
    assert torch.equal(w, w0)
    want = {}
    for r, c, v in put:
        v = float(dirty[r, c])
        hit, sign = _near(wl, r)
        kinds = want.setdefault(c, np.zeros((3, nx * nx), dtype=bool))   # +inf, -inf, NaN
        if np.isnan(v):
            kinds[2] |= hit
        else:
            kinds[0] |= hit & (sign * v > 0)
            kinds[1] |= hit & (sign * v < 0)
    for c in range(nchan):
        got = cube[c].reshape(-1).cpu().numpy()
        ref = clean[c].reshape(-1).cpu().numpy().copy()
        if c in want:
            up, dn, no = want[c]
            ok = np.isfinite(ref)
            ref[ok & up & ~dn & ~no] = np.inf
            ref[ok & dn & ~up & ~no] = -np.inf
            ref[ok & (no | (up & dn))] = np.nan
        assert np.array_equal(got, ref, equal_nan=True), c


def test_blanked_channels_and_rows():
    """Whole channels and whole samples of NaN."""
    import torch
    wl = _field(190, 190, 7600, 140)
    lon, lat, d = to_device(wl)
    g = make_gridder(wl, "fp32")
    clean, _ = g.grid_datacube(lon, lat, d)
    dirty = d.clone()
    dirty[:, ::17] = float("nan")
    cube, _ = g.grid_datacube(lon, lat, dirty)
    keep = torch.ones(140, dtype=torch.bool, device=d.device)
    keep[::17] = False
    assert torch.isnan(cube[~keep]).all()
    assert torch.equal(torch.nan_to_num(cube[keep], nan=-7.0), torch.nan_to_num(clean[keep], nan=-7.0))
    dirty = d.clone()
    dirty[100] = float("nan")
    hit = torch.as_tensor(_near(wl, 100)[0].reshape(190, 190), device=d.device)
    cube, _ = g.grid_datacube(lon, lat, dirty)
    assert torch.isnan(cube[:, hit]).all()
    assert torch.equal(torch.nan_to_num(cube[:, ~hit], nan=-7.0), torch.nan_to_num(clean[:, ~hit], nan=-7.0))
