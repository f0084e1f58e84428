"""Registers of the built kernels, as the metadata of their code objects has them."""
import os
import struct

import msgpack
import pytest

from paper_2108_08591_amd import build

MAGIC = b"__CLANG_OFFLOAD_BUNDLE__"


def _notes(elf):
    """Metadata map of an AMD GPU code object (note type 32)."""
    shoff, = struct.unpack_from("<Q", elf, 0x28)
    size, count = struct.unpack_from("<HH", elf, 0x3A)
    for k in range(count):
        _, kind, _, _, off, length = struct.unpack_from("<IIQQQQ", elf, shoff + k * size)
        end = off + length
        while kind == 7 and off < end:
            name, desc, note = struct.unpack_from("<III", elf, off)
            off += 12 + (name + 3 & ~3)
            if note == 32:
                return msgpack.unpackb(elf[off:off + desc])
            off += desc + 3 & ~3
    return {"amdhsa.kernels": []}


@pytest.fixture(scope="module")
def kernels():
    if not os.path.exists(build.LIB):
        build.build()
    with open(build.LIB, "rb") as f:
        data = f.read()
    found = {}
    at = data.find(MAGIC)
    while at >= 0:
        n, = struct.unpack_from("<Q", data, at + 24)
        o = at + 32
        for _ in range(n):
            off, size, length = struct.unpack_from("<QQQ", data, o)
            if b"gfx950" in data[o + 24:o + 24 + length]:
                for k in _notes(data[at + off:at + off + size])["amdhsa.kernels"]:
                    found[k[".name"]] = k
            o += 24 + length
        at = data.find(MAGIC, at + 24)
    return found


@pytest.mark.parametrize("kernel", ["6k_tile", "12k_tile_batch"])
@pytest.mark.parametrize("storage", [2, 3])
def test_two_blocks_of_16_wavefronts_fit_a_cu(kernels, kernel, storage):
    """The large tiles of the 16-bit formats run 1024 threads a block: 8
    wavefronts per SIMD, of 512 VGPRs and (in 16s, 16 of them the trap
    handler's) 800 SGPRs."""
    names = [n for n in kernels if f"{kernel}I" in n and f"Li{storage}ELb1ELi" in n]
    assert len(names) == 4 * 2 * 7                            # lattices, steps, options
    for n in names:
        k = kernels[n]
        assert k[".max_flat_workgroup_size"] == 1024 and k[".group_segment_fixed_size"] <= 80 * 1024
        assert k[".sgpr_count"] <= 80 and k[".vgpr_count"] <= 64 and k[".private_segment_fixed_size"] == 0, n
