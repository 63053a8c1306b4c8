"""Sample sort at the edges of its forms (one workgroup; 2048, 4096 and 8192
pairs per block): every target's neighbours, and a repeated call's cube, which
is bitwise the same only if the order of equal keys is."""
import numpy as np
import pytest

import oracle
from gpu_util import compare_neighbours, say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 2, 64, 1025, 8191, 8192, 8193, 524288, 524289, 1048577])
@pytest.mark.parametrize("nside", [64, 1024, 8192])
def test_neighbours(n, nside):
    import torch
    import paper_1604_06667_amd as cgp
    say(f"sort n={n} nside={nside}")
    rng = np.random.default_rng(n + nside)
    lon, lat = rng.uniform(0.0, 360.0, n), np.degrees(np.arcsin(rng.uniform(-1.0, 1.0, n)))
    k = n // 3                       # a third of the samples on few pixels, some of them equal
    lon[:k] = 40.0 + 1e-4 * rng.integers(0, 9, k)
    lat[:k] = 10.0
    tl = np.concatenate([[40.0, 40.0005, 0.0, 359.9], rng.uniform(0.0, 360.0, 60)])
    tb = np.concatenate([[10.0, 10.0003, 89.9, -89.9], rng.uniform(-80.0, 80.0, 60)])
    support = 1.0 if n > 10000 else 8.0
    dev = "cuda:0"
    t = lambda a: torch.as_tensor(np.ascontiguousarray(a), dtype=torch.float64, device=dev)
    g = cgp.SlGrid(t(tl), t(tb), 3)
    g.set_nside(nside)
    g.set_kernel("gauss1d", (support / 3.0,), support)
    counts, hashes = g.neighbour_stats(t(lon), t(lat))
    compare_neighbours(counts, hashes, oracle.neighbour_sets(lon, lat, tl, tb, support))
    data = torch.as_tensor(rng.normal(size=(n, 3)), dtype=torch.float32, device=dev)
    a, b = (g.grid_datacube(t(lon), t(lat), data) for _ in range(2))
    for x, y in zip(a, b):
        assert torch.equal(torch.nan_to_num(x, nan=-7.0), torch.nan_to_num(y, nan=-7.0))


@pytest.mark.parametrize("n", [(1 << 20) - 1, 1 << 20, 3000001])
@pytest.mark.parametrize("nside", [512, 2048])
def test_cell_table_lookup(n, nside):
    """Whole-sky map on either side of the rule for the table of pixel cells:
    the same neighbours as with the sample-centric lookup."""
    import torch
    import paper_1604_06667_amd as cgp
    say(f"cells n={n} nside={nside}")
    rng = np.random.default_rng(n)
    lon, lat = rng.uniform(0.0, 360.0, n), np.degrees(np.arcsin(rng.uniform(-1.0, 1.0, n)))
    lon[:n // 8], lat[:n // 8] = 77.0 + 1e-3 * rng.random(n // 8), 12.0   # one crowded cell
    lon[-3:], lat[-3:] = 10.0, [90.0, -90.0, 95.0]                        # poles; invalid
    t = lambda a: torch.as_tensor(a, dtype=torch.float64, device="cuda:0")
    g = cgp.HpxGrid(512, "ring", 1)
    g.set_nside(nside)
    g.set_kernel("gauss1d", (0.05,), 0.15)
    a = g.neighbour_stats(t(lon), t(lat))
    g.set_lookup("disk")
    b = g.neighbour_stats(t(lon), t(lat))
    assert int(a[0].sum()) > 0
    for x, y in zip(a, b):
        assert torch.equal(x, y)
