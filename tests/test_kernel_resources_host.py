"""Registers and scratch of the kernels that a shape's speed depends on, read from the
code objects of the built library (host only, no device).

gfx950: 512 registers per SIMD lane, given out in eights; a kernel of v registers
places 512 // v waves on a SIMD, at most 8.
"""
import os
import re
import struct

import pytest

msgpack = pytest.importorskip("msgpack")

from paper_2308_08417_amd import build

BUNDLE = b"__CLANG_OFFLOAD_BUNDLE__"


def code_objects(data):
    """The device ELF images of the library's offload bundles."""
    at = data.find(BUNDLE)
    while at >= 0:
        o = at + len(BUNDLE)
        (count,), o = struct.unpack_from("<Q", data, o), o + 8
        for _ in range(count):
            off, size, length = struct.unpack_from("<QQQ", data, o)
            name, o = data[o + 24:o + 24 + length], o + 24 + length
            if b"amdgcn" in name and size:
                yield data[at + off:at + off + size]
        at = data.find(BUNDLE, at + 1)


def kernels(elf):
    """The kernel records of an image's AMDGPU metadata note."""
    shoff, = struct.unpack_from("<Q", elf, 0x28)
    entsize, count = struct.unpack_from("<HH", elf, 0x3A)
    for i in range(count):
        kind, = struct.unpack_from("<I", elf, shoff + i * entsize + 4)
        off, size = struct.unpack_from("<QQ", elf, shoff + i * entsize + 24)
        end = off + size
        while kind == 7 and off < end:  # SHT_NOTE
            nsize, dsize, note = struct.unpack_from("<III", elf, off)
            name = elf[off + 12:off + 12 + nsize].rstrip(b"\0")
            desc = off + 12 + (nsize + 3) // 4 * 4
            if name == b"AMDGPU" and note == 32:
                yield from msgpack.unpackb(elf[desc:desc + dsize])["amdhsa.kernels"]
            off = desc + (dsize + 3) // 4 * 4


@pytest.fixture(scope="module")
def records():
    """Mangled name -> (waves per SIMD, scratch bytes per lane) of every kernel."""
    if not os.path.exists(build.LIB):
        pytest.skip("the library is not built")
    out = {}
    with open(build.LIB, "rb") as f:
        data = f.read()
    for elf in code_objects(data):
        for k in kernels(elf):
            regs = (k[".vgpr_count"] + 7) // 8 * 8
            out[k[".name"]] = (min(8, 512 // regs), k[".private_segment_fixed_size"])
    assert out
    return out


@pytest.fixture(scope="module")
def table(records):
    """(kernel, team shape, other template arguments) -> record, for the fixed-size kernels."""
    out = {}
    for name, r in records.items():
        m = re.match(r"_ZN2bs(?:\d+)(k_[a-z]+)INS_5ShapeILi(\d+)ELi(\d+)ELi(\d+)EEE((?:L[bi]\d+E)*)E", name)
        if m:
            args = tuple(int(a) for a in re.findall(r"L[bi](\d+)E", m[5]))
            out[(m[1], tuple(int(v) for v in m.group(2, 3, 4)), args)] = r
    return out


@pytest.mark.parametrize("team", [128, 256])
@pytest.mark.parametrize("kernel,args", [("k_cg", (1,)), ("k_bicgstab", (0, 1))])
def test_block_jacobi_of_long_rows(table, team, kernel, args):
    """64 slots on several waves with block Jacobi: nothing in scratch."""
    assert table[(kernel, (team, 1, 64), args)][1] == 0


@pytest.mark.parametrize("team", [128, 256, 512])
@pytest.mark.parametrize("nz,waves", [(4, 4), (8, 3), (16, 3), (32, 2)])
@pytest.mark.parametrize("args", [(0, 0), (0, 1), (1, 0)])
def test_gmres_on_several_waves(table, team, nz, waves, args):
    """FP64, block Jacobi and mixed: the waves per SIMD that rows and basis leave room
    for, nothing in scratch."""
    got, scratch = table[("k_gmres", (team, 1, nz), args)]
    assert got >= waves and scratch == 0


@pytest.mark.parametrize("lower", [0, 1])
@pytest.mark.parametrize("nz,waves", [(4, 6), (8, 4), (16, 3)])
def test_short_rows_of_one_wave_trsv(table, lower, nz, waves):
    """Small triangles live on resident waves."""
    assert table[("k_trsv", (64, 1, nz), (lower,))][0] >= waves


@pytest.mark.parametrize("nz", [8, 10])
@pytest.mark.parametrize("source", [0, 1, 2])
def test_uneven_few_tasks(records, nz, source):
    """BiCGSTAB on 512 lanes x 2 rows for launches of few tasks: everything in registers."""
    name = (f"_ZN2bs8k_varlenINS_8VarShapeILi512ELi2EEENS_7VarRowsIS2_Li{nz}ELi{source}ELb0EEE"
            "Li1ELb0ELb0ELb1EEEvNS_5VArgsE")
    assert records[name][1] == 0
