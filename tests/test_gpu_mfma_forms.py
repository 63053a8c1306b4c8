"""Matrix-core contraction: channel counts at the edges of the workgroup
shapes, supports on both sides of the short-support form, the batch's kernel
forms, and a captured batch whose gridders' kernels change afterwards."""
import dataclasses

import numpy as np
import pytest

import oracle
from gpu_util import flat, make_gridder, say, to_device
from test_gpu_gather_wide import _field, check_signed

pytestmark = pytest.mark.gpu
TOL = 2e-3          # the matrix-core precisions' bound
TOLW = 1e-6


def _check(cube, w, wl, ref):
    if wl.kernel[0] == "tapered_sinc" and wl.kernel[1][1] < wl.support:
        return check_signed(cube, w, wl, ref, TOL)
    ev = oracle.e_val(flat(cube, wl.nchan), ref["R"], ref["W"])
    ew = oracle.e_weights(w.cpu().numpy().astype(np.float64).ravel(), ref["W"])
    say(f"  e_val={ev:.2e} e_W={ew:.2e}")
    assert ev <= TOL and ew <= TOLW


@pytest.mark.parametrize("nchan", [1, 31, 33, 64, 65, 128, 129, 256, 257, 512, 513])
@pytest.mark.parametrize("dtype", ["f32", "f64", "bf16", "f16"])
def test_channel_edges(nchan, dtype):
    import torch
    wl = _field(33, 17, 900, nchan)
    dt = {"f32": torch.float32, "f64": torch.float64, "bf16": torch.bfloat16, "f16": torch.float16}[dtype]
    wl = dataclasses.replace(wl, data=wl.data.to(dt), dtype=dtype)
    ref = oracle.grid_workload(dataclasses.replace(wl, data=wl.data.to(torch.float64), dtype="f64"))
    lon, lat, d = to_device(wl)
    for prec in ("bf16", "fp16"):
        g = make_gridder(wl, prec)
        _check(*g.grid_datacube(lon, lat, d), wl, ref)


def _kernel(kind, s):
    return {"gauss1d": ("gauss1d", (s / 3.0,)), "gauss2d": ("gauss2d", (s / 3.0, s / 4.5, 30.0)),
            "tapered_sinc": ("tapered_sinc", (s / 3.0, s)), "two_zeros": ("tapered_sinc", (s / 3.0, s / 2.0)),
            "table": ("table", (s, 1.0, 0.8, 0.4, 0.1, 0.0))}[kind]


# 0.57 deg divides the short-support form from the general one
@pytest.mark.parametrize("support", [0.075, 0.57, 0.58, 10.0])
@pytest.mark.parametrize("kind", ["gauss1d", "gauss2d", "tapered_sinc", "two_zeros", "table"])
@pytest.mark.parametrize("nchan", [40, 300])
def test_support_forms(support, kind, nchan):
    wl = _field(33, 17, 700, nchan, kernel=_kernel(kind, support))
    wl = dataclasses.replace(wl, support=support)
    ref = oracle.grid_workload(wl)
    lon, lat, d = to_device(wl)
    g = make_gridder(wl, "bf16", nside=2048 if support < 1.0 else 256)
    _check(*g.grid_datacube(lon, lat, d), wl, ref)


def _batch(kinds_supports, nchan=70):
    import torch
    import paper_1604_06667_amd as cgp
    wls, gs, ins = [], [], []
    for k, (kind, s) in enumerate(kinds_supports):
        wl = dataclasses.replace(_field(20 + 9 * k, 17, 500 + 100 * k, nchan, kernel=_kernel(kind, s)), support=s)
        wls.append(wl)
        gs.append(make_gridder(wl, "bf16", nside=2048))
        ins.append(to_device(wl))
    return wls, gs, ins, cgp.Batch(gs, torch.float32)


@pytest.mark.parametrize("kinds", [
    [("gauss1d", 0.075), ("gauss1d", 0.1)], [("gauss1d", 0.075), ("gauss2d", 0.1)],
    [("gauss2d", 0.075), ("gauss1d", 0.7)]], ids=["circular", "both", "long"])
def test_batch_forms(kinds):
    wls, gs, ins, b = _batch(kinds)
    outs = b.outputs()
    b.grid(ins, outs)
    b.sync()
    for wl, (cube, w) in zip(wls, outs):
        _check(cube, w, wl, oracle.grid_workload(wl))


def test_replay_after_a_kernel_change():
    """The captured graph was built for circular kernels; after a pass with an
    elliptical one on the same gridders a replay follows the pass."""
    import torch
    wls, gs, ins, b = _batch([("gauss1d", 0.075), ("gauss1d", 0.1)])
    outs = b.outputs()
    b.capture(ins, outs)
    for _ in range(3):
        b.replay()
    b.sync()
    for wl, (cube, w) in zip(wls, outs):
        _check(cube, w, wl, oracle.grid_workload(wl))
    wls[1] = dataclasses.replace(wls[1], kernel=_kernel("gauss2d", 0.1))
    gs[1].set_kernel(*wls[1].kernel, 0.1, 0.0)   # nside is fixed: the lookup tables stay as they are
    b.grid(ins, outs)
    b.sync()
    for cube, w in outs:
        cube.fill_(-1.0)
        w.fill_(-1.0)
    for _ in range(2):
        b.replay()
    b.sync()
    for wl, (cube, w) in zip(wls, outs):
        _check(cube, w, wl, oracle.grid_workload(wl))
