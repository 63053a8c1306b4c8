"""Replays of a captured batch after passes on other inputs: fewer samples,
slightly more (within the buffers' headroom), or other kernels.  A replay
grids the captured buffers with the captured sample counts, equal to each job
gridded alone."""
import gc
import weakref

import pytest

from gpu_util import say
from test_gpu_batch import _alone, _batch, _jobs, _out_np, _same

pytestmark = pytest.mark.gpu


def _check(b, gs, ins, outs, times=3):
    import torch
    for _ in range(times):
        for cube, w in outs:
            cube.fill_(-7.0)
            w.fill_(-7.0)
        torch.cuda.synchronize()
        b.replay()
        b.sync()
        got = [_out_np(cube, w, g.nchan) for g, (cube, w) in zip(gs, outs)]
        for g, (lon, lat, d), r in zip(gs, ins, got):
            _same(r, _alone(g, lon, lat, d))


def _other(ins, frac):
    """The jobs' inputs cut or stretched to frac of their samples, in buffers
    of their own and in another order."""
    import torch
    out = []
    for lon, lat, d in ins:
        n = lon.shape[0]
        k = torch.randperm(n, device=lon.device)
        k = torch.cat([k, k[:max(0, int(n * frac) - n)]])[:int(n * frac)]
        out.append((lon[k].contiguous(), lat[k].contiguous(), (d[k] * 2 + 1).contiguous()))
    return out


@pytest.mark.parametrize("frac", [0.0, 0.4, 0.97, 1.05])
def test_replay_after_a_pass_of_another_size(frac):
    b, gs, ins = _batch(_jobs(3, 0.02))
    outs, outs2 = b.outputs(), b.outputs()
    b.capture(ins, outs)
    other = _other(ins, frac)
    n = sum(i[0].shape[0] for i in ins), sum(i[0].shape[0] for i in other)
    say(f"captured {n[0]} samples, then a pass of {n[1]}")
    b.grid(other, outs2)
    b.sync()
    assert b.query(8) == 1 and b.query(1) == n[1]
    want = [_out_np(c, w, g.nchan) for g, (c, w) in zip(gs, outs2)]
    _check(b, gs, ins, outs)
    assert b.query(1) == n[0]
    for g, (c, w), r in zip(gs, outs2, want):   # the replays left the pass's outputs alone
        _same(_out_np(c, w, g.nchan), r, tol=0.0)


def test_replay_after_another_kernel_and_inputs():
    """As above with a job's kernel made elliptical in between: replays take
    the new kernel, on the captured inputs."""
    wls = _jobs(3, 0.02)
    b, gs, ins = _batch(wls)
    for g, wl in zip(gs, wls):
        g.set_kernel("gauss1d", (wl.support / 3.0,), wl.support, wl.hpx_maxres or 0.1)
    import paper_1604_06667_amd as cgp
    import torch
    b = cgp.Batch(gs, torch.bfloat16)
    outs, outs2 = b.outputs(), b.outputs()
    b.capture(ins, outs)
    b.grid(_other(ins, 0.5), outs2)
    s = wls[1].support
    gs[1].set_kernel("gauss2d", (s / 3.0, s / 4.5, 30.0), s, wls[1].hpx_maxres or 0.1)
    b.grid(_other(ins, 0.7), outs2)
    assert b.query(8) == 1
    _check(b, gs, ins, outs)


def test_captured_buffers_stay_alive():
    """The binding keeps what the graph points to until the graph is gone."""
    b, gs, ins = _batch(_jobs(2, 0.01))
    other = _other(ins, 0.5)
    outs = b.outputs()
    b.capture(ins, outs)
    refs = [weakref.ref(t) for i in ins for t in i[:2]] + [weakref.ref(c) for c, _ in outs]
    del ins, outs
    b.grid(other, b.outputs())
    gc.collect()
    assert all(r() is not None for r in refs)
    b.tune(other, b.outputs(), reps=1)   # drops the graph
    gc.collect()
    assert all(r() is None for r in refs)


def test_graph_survives_passes_of_fewer_samples():
    """Pair counts on both sides of the sizes where the sort's blocks double."""
    import dataclasses

    import numpy as np
    import torch
    import paper_1604_06667_amd as cgp
    from gpu_util import make_gridder, to_device
    from test_gpu_gather_wide import _field
    wl = _field(33, 17, 1_200_000, 17)
    g = make_gridder(wl, "bf16")
    lon, lat, d = to_device(wl)
    b = cgp.Batch([g], torch.float32)
    for n, fewer in ((600_000, (524_288, 500_000)), (1_150_000, (1_048_576, 1_000_000, 500_000))):
        ins, outs = [(lon[:n], lat[:n], d[:n])], b.outputs()
        b.capture(ins, outs)
        for m in fewer:
            b.grid([(lon[:m], lat[:m], d[:m])], b.outputs())
            assert b.query(8) == 1, (n, m)
        _check(b, [g], ins, outs, times=1)
