"""Workspace of FP32 grids by channel count: one and two channels travel in
the sorted records and take no rows of their own; a workspace of exactly the
stated size is enough and nothing past it is written."""
import pytest

from gpu_util import make_gridder, to_device
from test_gpu_gather_wide import _field

pytestmark = pytest.mark.gpu


def test_rows_only_where_they_are_used():
    size = {c: make_gridder(_field(20, 20, 10, c), "fp32").workspace_size(100_000) for c in (1, 2, 3, 16, 17)}
    assert size[1] == size[2] == size[17]
    for c in (3, 16):
        assert size[c] - size[17] == 4 * c * 100_000 + (-4 * c * 100_000) % 256


@pytest.mark.parametrize("nchan", [1, 2, 3, 16, 17])
@pytest.mark.parametrize("n", [1, 100, 9001])
def test_exact_workspace(nchan, n):
    import torch
    wl = _field(20, 20, n, nchan)
    lon, lat, d = to_device(wl)
    g = make_gridder(wl, "fp32")
    want = g.grid_datacube(lon, lat, d)
    size = g.workspace_size(n)
    buf = torch.full((size + 4096,), 0x5A, dtype=torch.uint8, device="cuda:0")
    cube, w = (torch.empty_like(t) for t in want)
    g.grid_datacube(lon, lat, d, cube, w, ws=buf[:size])
    for a, b in zip((cube, w), want):
        assert torch.equal(torch.nan_to_num(a, nan=-7.0), torch.nan_to_num(b, nan=-7.0))
    assert bool((buf[size:] == 0x5A).all())
