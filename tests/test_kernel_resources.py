"""Registers of the built kernels, from the metadata of their code objects: how many workgroups a compute unit holds is part of what the tiles
were chosen for, and a few registers too many change it without any result changing."""
import os
import struct
import subprocess

import msgpack
import pytest

import paper_2412_20386_amd.build as hip_build

MAGIC = b"__CLANG_OFFLOAD_BUNDLE__"


def _code_objects(path):
    data = open(path, "rb").read()
    at = data.find(MAGIC)
    while at >= 0:
        (n,) = struct.unpack_from("<Q", data, at + len(MAGIC))
        pos = at + len(MAGIC) + 8
        for _ in range(n):
            offset, size, length = struct.unpack_from("<QQQ", data, pos)
            if b"gfx950" in data[pos + 24:pos + 24 + length]:
                yield data[at + offset:at + offset + size]
            pos += 24 + length
        at = data.find(MAGIC, at + 1)


def _metadata(elf):
    """The kernels' records of an AMDGPU code object (ELF64, little endian): the msgpack map of its NT_AMDGPU_METADATA note."""
    shoff, = struct.unpack_from("<Q", elf, 0x28)
    shentsize, shnum = struct.unpack_from("<HH", elf, 0x3A)
    for i in range(shnum):
        kind, = struct.unpack_from("<I", elf, shoff + i * shentsize + 4)
        offset, size = struct.unpack_from("<QQ", elf, shoff + i * shentsize + 0x18)
        pos = offset
        while kind == 7 and pos < offset + size:  # SHT_NOTE
            name_size, desc_size, note = struct.unpack_from("<III", elf, pos)
            desc = pos + 12 + (name_size + 3) // 4 * 4
            if note == 32:
                yield from msgpack.unpackb(elf[desc:desc + desc_size])["amdhsa.kernels"]
            pos = desc + (desc_size + 3) // 4 * 4


@pytest.fixture(scope="module")
def kernels():
    if not os.path.exists(hip_build.LIB_PATH):
        pytest.skip("the library is not built")
    found = [k for elf in _code_objects(hip_build.LIB_PATH) for k in _metadata(elf)]
    names = subprocess.run(["c++filt"], input="\n".join(k[".name"] for k in found), capture_output=True, text=True, check=True).stdout.split("\n")
    return {name: k for name, k in zip(names, found)}


def waves_per_simd(kernel):
    registers = (kernel[".vgpr_count"] + 7) // 8 * 8  # (includes the accumulation registers)
    return min(8, 512 // registers)


def test_split_reduction_fits_four_workgroups(kernels):
    """Up to 1000 tiles of 32 x 32, a workgroup of four wavefronts each, are one round of 256 CUs."""
    found = {n: k for n, k in kernels.items() if "linear_mfma_splitk<" in n}
    assert len(found) >= 16
    for name, k in found.items():
        assert waves_per_simd(k) >= 4 and k[".private_segment_fixed_size"] == 0, name


@pytest.mark.parametrize("tile,workgroups", [("128, 256, 2, 4, 2", 2), ("128, 128, 2, 4, 2", 3), ("64, 128, 2, 2, 2", 4), ("64, 64, 2, 2, 2", 5), ("32, 64, 2, 2, 3", 5)])
def test_e2m3_tiles_share_a_compute_unit(kernels, tile, workgroups):
    """As many workgroups as the 160 KiB of LDS hold (for 64 x 64 tiles one less): a tile's epilogue runs under the products of the
    others."""
    _, _, wave_rows, wave_cols, _ = (int(v) for v in tile.split(", "))
    found = {n: k for n, k in kernels.items() if f"linear_e2m3_tile<{tile}, " in n}
    assert len(found) == 2  # without and with the accumulators
    for name, k in found.items():
        assert waves_per_simd(k) * 4 // (wave_rows * wave_cols) >= workgroups, name


def test_tiles_of_any_alignment_spill_nothing(kernels):
    found = {n: k for n, k in kernels.items() if "linear_mfma_tile<" in n and "Copy)0>" not in n}
    assert len(found) >= 40
    for name, k in found.items():
        assert k[".private_segment_fixed_size"] == 0, name
