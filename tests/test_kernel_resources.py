"""No kernel of the library needs scratch memory: the runtime would hold it on the device, beside what a
call's plan counts against its budget and although the allocation-free entry point promises that there is none."""
import os
import struct

import msgpack
import pytest

from paper_2503_04424_amd import lib_path

MAGIC = b"__CLANG_OFFLOAD_BUNDLE__"
SHT_NOTE, NT_AMDGPU_METADATA = 7, 32


def code_objects(lib):
    """The gfx950 code objects in the library's offload bundles."""
    data = open(lib, "rb").read()
    at = data.find(MAGIC)
    while at >= 0:
        count, = struct.unpack_from("<Q", data, at + len(MAGIC))
        entry = at + len(MAGIC) + 8
        for _ in range(count):
            offset, size, length = struct.unpack_from("<QQQ", data, entry)
            if b"gfx950" in data[entry + 24:entry + 24 + length] and size:
                yield data[at + offset:at + offset + size]
            entry += 24 + length
        at = data.find(MAGIC, at + len(MAGIC))


def kernels(elf):
    """The metadata of a code object's kernels, from its notes."""
    sections, = struct.unpack_from("<Q", elf, 0x28)
    entry_size, count = struct.unpack_from("<HH", elf, 0x3A)
    for i in range(count):
        kind, = struct.unpack_from("<I", elf, sections + i * entry_size + 4)
        at, size = struct.unpack_from("<QQ", elf, sections + i * entry_size + 24)
        end = at + size
        while kind == SHT_NOTE and at < end:
            name, length, note = struct.unpack_from("<III", elf, at)
            at += 12 + (name + 3) // 4 * 4
            if note == NT_AMDGPU_METADATA:
                yield from msgpack.unpackb(elf[at:at + length])["amdhsa.kernels"]
            at += (length + 3) // 4 * 4


def test_no_kernel_needs_scratch_memory():
    if not os.path.exists(lib_path()):
        pytest.skip("library not built")
    found = [k for elf in code_objects(lib_path()) for k in kernels(elf)]
    assert any("trailing_update_kernel" in k[".name"] for k in found)
    scratch = {k[".name"]: k[".private_segment_fixed_size"] for k in found if k[".private_segment_fixed_size"]}
    assert not scratch
    assert not [k[".name"] for k in found if k.get(".vgpr_spill_count", 0)]
