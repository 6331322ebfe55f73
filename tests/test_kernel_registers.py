"""Registers and scratch of the built row and column kernels, from the metadata
of the code objects in libzk.so: the numbers that decide how many wavefronts a
SIMD holds (512 / registers, in blocks of 8)."""
import os
import re
import struct

import pytest

LIB = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2608_25203_amd", "libzk.so")
MAGIC = b"__CLANG_OFFLOAD_BUNDLE__"
msgpack = pytest.importorskip("msgpack")
pytestmark = pytest.mark.skipif(not os.path.exists(LIB), reason="libzk.so not built")


def code_objects(data):
    at = data.find(MAGIC)
    while at >= 0:
        n, = struct.unpack_from("<Q", data, at + len(MAGIC))
        p = at + len(MAGIC) + 8
        for _ in range(n):
            off, size, tl = struct.unpack_from("<QQQ", data, p)
            triple = data[p + 24:p + 24 + tl]
            p += 24 + tl
            if b"gfx" in triple and size:
                yield data[at + off:at + off + size]
        at = data.find(MAGIC, at + 1)


def metadata(elf):
    """The AMDGPU metadata note of a code object."""
    shoff, = struct.unpack_from("<Q", elf, 40)
    shentsize, shnum = struct.unpack_from("<HH", elf, 58)
    for i in range(shnum):
        typ, = struct.unpack_from("<I", elf, shoff + i * shentsize + 4)
        off, size = struct.unpack_from("<QQ", elf, shoff + i * shentsize + 24)
        if typ != 7:  # SHT_NOTE
            continue
        p = off
        while p < off + size:
            ns, ds, nt = struct.unpack_from("<III", elf, p)
            name = elf[p + 12:p + 12 + ns].rstrip(b"\0")
            d = p + 12 + (ns + 3) // 4 * 4
            if name == b"AMDGPU" and nt == 32:
                return msgpack.unpackb(elf[d:d + ds], strict_map_key=False)
            p = d + (ds + 3) // 4 * 4
    return {"amdhsa.kernels": []}


@pytest.fixture(scope="module")
def kernels():
    """(kernel, real, template integers...) -> (registers, scratch bytes a lane)"""
    out = {}
    for elf in code_objects(open(LIB, "rb").read()):
        for k in metadata(elf)["amdhsa.kernels"]:
            m = re.match(r"_ZN2zk\d+((?:row|col)_kernel_\w+?)I([fd])((?:L[ib]\d+E)+)", k[".name"])
            if m:
                args = tuple(int(x) for x in re.findall(r"L[ib](\d+)E", m.group(3)))
                out[(m.group(1), m.group(2)) + args] = (k[".vgpr_count"],  # both files' registers
                                                       k[".private_segment_fixed_size"])
    assert out
    return out


def waves(registers):
    return min(8, 512 // ((registers + 7) // 8 * 8))


@pytest.mark.parametrize("T", [16, 32, 64])
def test_fp32_radix9_rows_keep_three_wavefronts(kernels, T):
    """Rows of 96, 192 and 384 points: in a batch of tiles their launches fill the chip."""
    assert waves(kernels[("row_kernel_batch", "f", T, 9, 1, 0, 0)][0]) >= 3


@pytest.mark.parametrize("T", [16, 32, 64, 128, 24, 40, 48, 80, 96])
def test_fp64_small_team_rows_keep_four_wavefronts(kernels, T):
    """The plain form, which launches that fill the chip take."""
    assert waves(kernels[("row_kernel_batch", "d", T, 3, 1, 0, 0)][0]) >= 4


@pytest.mark.parametrize("T", [16, 32])
def test_fp32_small_team_rows_keep_six_wavefronts(kernels, T):
    assert waves(kernels[("row_kernel_batch", "f", T, 3, 1, 0, 0)][0]) >= 6


@pytest.mark.parametrize("T,E", [(16, 9), (32, 9), (64, 9), (16, 15), (32, 15), (64, 15)])
def test_fp32_columns_with_a_factor_3_or_5_use_no_scratch(kernels, T, E):
    """Padded columns of 96 to 384 and 160 to 640 points: the task record stays in registers."""
    assert kernels[("col_kernel_batch", "f", T, E, 0, 1)][1] == 0


@pytest.mark.parametrize("T", [16, 32, 64])
def test_fp32_radix15_rows_do_not_spill(kernels, T):
    """Rows of 160, 320 and 640 points: two wavefronts a SIMD without scratch."""
    regs, scratch = kernels[("row_kernel_batch", "f", T, 15, 1, 0, 0)]
    assert waves(regs) >= 2 and scratch == 0
