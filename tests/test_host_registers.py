"""Register spills of the built kernels, from the metadata of the code objects
in libcg.so: forms that ran slower for them are held to what they took without."""
import re
import struct

import pytest

from paper_1604_06667_amd import _cg

msgpack = pytest.importorskip("msgpack")
MAGIC = b"__CLANG_OFFLOAD_BUNDLE__"


def _notes(elf):
    """Notes of a 64-bit little-endian ELF image: (type, payload)."""
    shoff, = struct.unpack_from("<Q", elf, 0x28)
    size, num = struct.unpack_from("<HH", elf, 0x3A)
    for k in range(num):
        kind, = struct.unpack_from("<I", elf, shoff + k * size + 4)
        if kind != 7:   # SHT_NOTE
            continue
        off, length = struct.unpack_from("<QQ", elf, shoff + k * size + 24)
        end = off + length
        while off + 12 <= end:
            n, d, t = struct.unpack_from("<III", elf, off)
            off += 12 + (n + 3) // 4 * 4
            yield t, elf[off:off + d]
            off += (d + 3) // 4 * 4


@pytest.fixture(scope="module")
def spills():
    """Mangled kernel name -> spilled vector registers."""
    blob = open(_cg.LIB_PATH, "rb").read()
    out = {}
    for m in re.finditer(MAGIC, blob):
        count, = struct.unpack_from("<Q", blob, m.start() + 24)
        at = m.start() + 32
        for _ in range(count):
            off, size, n = struct.unpack_from("<QQQ", blob, at)
            name = blob[at + 24:at + 24 + n]
            at += 24 + n
            if b"gfx950" not in name:
                continue
            for t, d in _notes(blob[m.start() + off:m.start() + off + size]):
                if t == 32:   # the AMDGPU metadata
                    for k in msgpack.unpackb(d)["amdhsa.kernels"]:
                        out[k[".name"]] = k[".vgpr_spill_count"]
    if not out:
        pytest.skip("no plain code objects in the library")
    return out


def _forms(spills, pattern):
    got = {k: v for k, v in spills.items() if re.search(pattern, k)}
    assert got, pattern
    return got


def test_wide_gather_of_fp64_rows(spills):
    """Gaussians in every workgroup shape, and the radial kernels in the widest."""
    for k, v in _forms(spills, r"13k_gather_wideILi\dELi\dELi[01]ELb[01]EdE").items():
        assert v <= 16, (k, v)
    for k, v in _forms(spills, r"13k_gather_wideILi4ELi1ELi3ELb[01]EdE").items():
        assert v <= 32, (k, v)


def test_matrix_core_contraction_of_fp64_rows(spills):
    """Up to 256 channels."""
    for k, v in _forms(spills, r"13k_gather_mfmaILi[48]ELi1E.*EdLi\dEE").items():
        assert v <= 16, (k, v)


def test_ragged_channels_under_a_long_ellipse(spills):
    """More than 512 channels, BF16 mode, elliptical kernel, support above 0.57 deg."""
    assert not [k for k in spills if re.search(r"13k_gather_mfmaILi8ELi4ELi1ELb0ELi0ELb0E(f|t|DF16_)Li", k)]
    for k, v in _forms(spills, r"13k_gather_mfmaILi8ELi2ELi1ELb0ELi0ELb0E(f|t|DF16_)Li").items():
        assert v == 0, (k, v)


def test_batch_contraction(spills):
    """Eight wavefronts of one block with FP32 rows, and FP64 rows in every shape."""
    for k, v in _forms(spills, r"12k_batch_mfmaILi8ELi1E.*EfEE").items():
        assert v == 0, (k, v)
    for k, v in _forms(spills, r"12k_batch_mfmaILi\dELi\d.*EdEE").items():
        assert v == 0, (k, v)
