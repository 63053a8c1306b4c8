"""The device sort itself against a stable argsort: every digit width (8, 9 and
10 bits), the one-workgroup form and the three block sizes, values given or
formed by the first pass, and the batch's extra pass by job.  Keys repeat, so
an order of equal keys other than the input's fails."""
import ctypes as C

import numpy as np
import pytest

from gpu_util import say
from paper_1604_06667_amd import _cg

pytestmark = pytest.mark.gpu


def _fn(name, argtypes):
    f = getattr(C.CDLL(_cg.LIB_PATH), name)
    f.restype, f.argtypes = C.c_int, argtypes
    return f


def _sort(keys, bits, iota, joff=None):
    """(sorted keys, sorted values) of device keys, values 0, 1, 2, ..."""
    import torch
    n = keys.numel()
    elems = C.CDLL(_cg.LIB_PATH)._ZN2cg16radix_hist_elemsEl
    elems.restype, elems.argtypes = C.c_size_t, [C.c_int64]
    k = keys.clone()
    v = torch.full_like(k, -1) if iota else torch.arange(n, dtype=torch.int32, device=k.device)
    k2, v2 = torch.empty_like(k), torch.empty_like(k)
    hist = torch.empty(elems(n), dtype=torch.int32, device=k.device)
    p = [C.c_void_p(t.data_ptr()) for t in (k, v, k2, v2, hist)]
    st = C.c_void_p(torch.cuda.current_stream().cuda_stream)
    tmp = C.c_bool(False)
    if joff is None:
        f = _fn("_ZN2cg10radix_sortEPjS0_S0_S0_S0_libPbP12ihipStream_t",
                [C.c_void_p] * 5 + [C.c_int64, C.c_int, C.c_bool, C.POINTER(C.c_bool), C.c_void_p])
        assert f(*p, n, bits, iota, C.byref(tmp), st) == 0
    else:
        off = torch.as_tensor(joff, dtype=torch.int64, device=k.device)
        f = _fn("_ZN2cg15radix_sort_jobsEPjS0_S0_S0_S0_libPKliPbP12ihipStream_t",
                [C.c_void_p] * 5 + [C.c_int64, C.c_int, C.c_bool, C.c_void_p, C.c_int, C.POINTER(C.c_bool), C.c_void_p])
        assert f(*p, n, bits, iota, C.c_void_p(off.data_ptr()), len(joff) - 1, C.byref(tmp), st) == 0
    torch.cuda.synchronize()
    return (k2, v2) if tmp.value else (k, v)


def _keys(n, bits, rng):
    """Many repeats, a crowded key, and the largest key of the width."""
    import torch
    k = rng.integers(0, min(1 << bits, max(2, n // 3)), n, dtype=np.int64)
    k[rng.random(n) < 0.2] = (1 << bits) - 1
    k[rng.random(n) < 0.2] = 5 % (1 << bits)
    s = max(0, bits - 20)
    k[::7] = (k[::7] << s) & ((1 << bits) - 1)
    return torch.as_tensor(k.astype(np.int32), device="cuda:0")


@pytest.mark.parametrize("n", [1, 2, 63, 64, 65, 1025, 8191, 8192, 8193, 20000, 524288, 524289, 1048576, 1048577, 3000001])
@pytest.mark.parametrize("bits", [4, 8, 13, 16, 18, 20, 26, 27, 30])
def test_stable(n, bits):
    import torch
    keys = _keys(n, bits, np.random.default_rng(n + bits))
    order = torch.argsort(keys, stable=True)
    for iota in (True, False):
        k, v = _sort(keys, bits, iota)
        assert torch.equal(k, keys[order]) and torch.equal(v.long(), order), iota


@pytest.mark.parametrize("sizes", [[1, 0, 2], [3000, 5000], [4096] * 200, [700000, 1, 0, 400000], [5000] + [0] * 254 + [9000]],
                         ids=["tiny", "small", "many", "large", "256"])
def test_by_job(sizes):
    import torch
    joff = np.concatenate([[0], np.cumsum(sizes)])
    n = int(joff[-1])
    say(f"{len(sizes)} jobs, {n} samples")
    keys = _keys(n, 26, np.random.default_rng(n))
    job = torch.as_tensor(np.repeat(np.arange(len(sizes)), sizes), device=keys.device)
    order = torch.argsort(job * (1 << 32) + keys.long(), stable=True)
    k, v = _sort(keys, 26, False, joff)
    assert torch.equal(k, keys[order]) and torch.equal(v.long(), order)
