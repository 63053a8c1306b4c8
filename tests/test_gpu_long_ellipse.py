"""Elliptical kernels of long supports on the matrix cores at the channel
counts where the workgroup changes: two blocks a wavefront for ragged counts
in BF16 mode, four for multiples of 1024 and in FP16 mode."""
import dataclasses

import pytest

import oracle
from gpu_util import make_gridder, to_device
from test_gpu_gather_wide import _field
from test_gpu_mfma_forms import _check, _kernel

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nchan", [512, 513, 1000, 1024, 1025])
@pytest.mark.parametrize("dtype", ["f32", "f64", "bf16", "f16"])
def test_channel_edges(nchan, dtype):
    import torch
    wl = dataclasses.replace(_field(33, 17, 400, nchan, kernel=_kernel("gauss2d", 0.9)), support=0.9)
    dt = {"f32": torch.float32, "f64": torch.float64, "bf16": torch.bfloat16, "f16": torch.float16}[dtype]
    wl = dataclasses.replace(wl, data=wl.data.to(dt), dtype=dtype)
    ref = oracle.grid_workload(dataclasses.replace(wl, data=wl.data.to(torch.float64), dtype="f64"))
    lon, lat, d = to_device(wl)
    for prec in ("bf16", "fp16"):
        g = make_gridder(wl, prec, nside=512)
        _check(*g.grid_datacube(lon, lat, d), wl, ref)
