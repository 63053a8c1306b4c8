"""Wide FP32 gather of 16-bit rows in the workgroups of two and four channel
blocks, aligned and not."""
import dataclasses

import pytest

import oracle
from gpu_util import make_gridder, to_device
from test_gpu_gather_wide import _check, _field

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["bf16", "f16"])
@pytest.mark.parametrize("nchan", [65, 128, 140, 256, 259])
def test_channel_blocks(dtype, nchan):
    import torch
    wl = _field(190, 188, 4000, nchan)
    dt = {"bf16": torch.bfloat16, "f16": torch.float16}[dtype]
    wl = dataclasses.replace(wl, data=wl.data.to(dt), dtype=dtype)
    ref = oracle.grid_workload(dataclasses.replace(wl, data=wl.data.to(torch.float64), dtype="f64"))
    lon, lat, d = to_device(wl)
    g = make_gridder(wl, "fp32")
    _check(*g.grid_datacube(lon, lat, d), wl, ref)
    wide = torch.zeros((d.shape[0], nchan + 3), dtype=d.dtype, device=d.device)
    wide[:, 1:1 + nchan] = d
    _check(*g.grid_datacube(lon, lat, wide[:, 1:1 + nchan]), wl, ref)
