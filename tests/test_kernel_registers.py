"""What the compiler wrote into the built library about its kernels: none of them may use scratch memory (a spilled vector register is a
store and a load of 256 bytes per wave, in kernels that are laid out to fit the register file).  Needs no GPU."""
import os
import struct

import msgpack
import pytest

import paper_2410_12876_amd as ag

MAGIC = b"__CLANG_OFFLOAD_BUNDLE__"


def _metadata(elf):
    """the kernels of one code object: its NT_AMDGPU_METADATA notes"""
    sections, (size, count) = struct.unpack_from("<Q", elf, 40)[0], struct.unpack_from("<HH", elf, 58)
    for i in range(count):
        if struct.unpack_from("<I", elf, sections + i * size + 4)[0] != 7:  # SHT_NOTE
            continue
        at, length = struct.unpack_from("<QQ", elf, sections + i * size + 24)
        end = at + length
        while at < end:
            name_len, data_len, kind = struct.unpack_from("<III", elf, at)
            at += 12 + (name_len + 3) // 4 * 4
            if kind == 32:
                yield from msgpack.unpackb(elf[at:at + data_len])["amdhsa.kernels"]
            at += (data_len + 3) // 4 * 4


@pytest.fixture(scope="module")
def kernels():
    if not os.path.exists(ag.LIB_PATH):
        from paper_2410_12876_amd import build
        build.build()
    data = open(ag.LIB_PATH, "rb").read()
    found, start = [], data.find(MAGIC)
    while start >= 0:
        entries, at = struct.unpack_from("<Q", data, start + 24)[0], start + 32
        for _ in range(entries):
            offset, size, n = struct.unpack_from("<QQQ", data, at)
            triple = data[at + 24:at + 24 + n]
            at += 24 + n
            if b"gfx950" in triple:
                found += _metadata(data[start + offset:start + offset + size])
        start = data.find(MAGIC, start + 1)
    return found


def test_no_kernel_uses_scratch(kernels):
    assert sum("ag_prefill_bf16_kernel" in k[".name"] for k in kernels) >= 12 and len(kernels) > 100
    assert [k[".name"] for k in kernels if k[".private_segment_fixed_size"] or k[".vgpr_spill_count"]] == []
