"""Supports near the resolution of FP64 unit vectors: the narrow FP32 gather,
whose candidates are marked in FP32, finds the pairs that the FP64 test of the
neighbour statistics and of the wide gather finds.  (The kernel is evaluated
on the same chords by all of them, so the comparison is exact to rounding
although the chords themselves are not.)"""
import numpy as np
import pytest

from gpu_util import say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("support", [2e-14, 1e-13, 1e-12, 1e-10])   # radians
@pytest.mark.parametrize("centre", [(40.0, 10.0), (120.0, 30.0), (200.0, -70.0)])
def test_narrow_finds_the_same_pairs(support, centre):
    import torch
    import paper_1604_06667_amd as cgp
    rng = np.random.default_rng(int(1e15 * support))
    t = lambda a: torch.as_tensor(np.ascontiguousarray(a), dtype=torch.float64, device="cuda:0")
    r = np.degrees(support)
    pts = lambda n: (t(centre[0] + rng.uniform(-3, 3, n) * r), t(centre[1] + rng.uniform(-3, 3, n) * r))
    tl, tb = pts(1280)
    lon, lat = pts(500)
    data = torch.ones((500, 17), dtype=torch.float32, device="cuda:0")
    got = {}
    for nchan in (1, 3, 16, 17):
        g = cgp.SlGrid(tl, tb, nchan)
        g.set_kernel("gauss1d", (r / 3.0,), r, 0.1)
        got[nchan] = g.grid_datacube(lon, lat, data[:, :nchan].contiguous())[1].cpu().numpy()
    count = g.neighbour_stats(lon, lat)[0].cpu().numpy()
    say(f"support {support} at {centre}: {int(count.sum())} pairs")
    for nchan in (1, 3, 16, 17):
        assert np.array_equal(got[nchan] > 0, count > 0)
        np.testing.assert_allclose(got[nchan], got[17], rtol=1e-6)
