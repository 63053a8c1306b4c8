"""Scratch of the device sort: a buffer sized for n pairs holds any smaller
sort, also across the sizes where the pairs per block double."""
import ctypes as C

from paper_1604_06667_amd import _cg


def _elems():
    f = C.CDLL(_cg.LIB_PATH)._ZN2cg16radix_hist_elemsEl
    f.restype, f.argtypes = C.c_size_t, [C.c_int64]
    return f


def test_hist_elems_grow_with_the_pairs():
    f = _elems()
    jumps = [1, 2048, 8192, 524288, 1048576, 2097152, 1 << 31]
    ns = sorted({max(1, j + d) for j in jumps for d in (-4097, -1, 0, 1, 4097, 75000)} | set(range(1, 4_000_000, 1777)))
    sizes = [f(n) for n in ns]
    assert all(a <= b for a, b in zip(sizes, sizes[1:]))


def test_hist_elems_hold_every_pass():
    """1024 counts per block and 1024 totals, for the blocks of n's own form."""
    f = _elems()
    for n in (1, 2048, 2049, 524288, 524289, 1048576, 1048577, 47_185_920):
        tile = 512 * (4 if n <= 524288 else 8 if n <= 1048576 else 16)
        assert f(n) >= ((n + tile - 1) // tile + 1) * 1024
