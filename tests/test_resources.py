"""What the compiler gave the kernels of the built library: the notes that it leaves in the code objects."""
import struct

import msgpack
import pytest


def _notes(elf):
    """The AMDGPU metadata notes of a code object (64-bit ELF)."""
    table, = struct.unpack_from("<Q", elf, 40)
    size, number = struct.unpack_from("<HH", elf, 58)
    for i in range(number):
        _, kind, _, _, at, length = struct.unpack_from("<IIQQQQ", elf, table + i * size)
        end = at + length
        while kind == 7 and at < end:  # SHT_NOTE
            name, description, note = struct.unpack_from("<III", elf, at)
            at += 12 + (name + 3 & ~3)
            if note == 32:  # NT_AMDGPU_METADATA
                yield msgpack.unpackb(elf[at:at + description])
            at += description + 3 & ~3


@pytest.fixture(scope="module")
def kernels():
    import os
    from paper_2002_11082_amd import binding, build
    if not os.path.exists(binding.LIB_PATH):
        build.build()
    data, magic, found = open(binding.LIB_PATH, "rb").read(), b"__CLANG_OFFLOAD_BUNDLE__", {}
    at = data.find(magic)
    while at >= 0:
        number, = struct.unpack_from("<Q", data, at + len(magic))
        entry = at + len(magic) + 8
        for _ in range(number):
            offset, size, name = struct.unpack_from("<QQQ", data, entry)
            if b"gfx950" in data[entry + 24:entry + 24 + name]:
                for note in _notes(data[at + offset:at + offset + size]):
                    found.update((kernel[".name"], kernel) for kernel in note["amdhsa.kernels"])
            entry += 24 + name
        at = data.find(magic, at + 1)
    assert len(found) > 400
    return found


@pytest.mark.parametrize("kernel", ["orq_team_kernel", "orq_pool_kernel", "orq_rows_kernel", "orq_gather_kernel", "orq_quantize_kernel"])
def test_no_scratch_memory(kernels, kernel):
    """Registers that spill cost a trip to memory in every bucket."""
    mine = {name: k[".private_segment_fixed_size"] for name, k in kernels.items() if kernel in name}
    assert mine and {name: size for name, size in mine.items() if size} == {}
