"""No kernel of the library keeps registers in scratch memory: the reloads are waited for in order with everything that the kernel has
asked for ahead.  Read from what the compiler wrote beside the code."""
import struct

import msgpack

from paper_2405_16256_amd import build

BUNDLE = b"__CLANG_OFFLOAD_BUNDLE__"


def code_objects(data):
    """The device code in a library: bundles of (offset, size, target) entries."""
    at = data.find(BUNDLE)
    while at >= 0:
        count, = struct.unpack_from("<Q", data, at + len(BUNDLE))
        p = at + len(BUNDLE) + 8
        for _ in range(count):
            offset, size, name = struct.unpack_from("<QQQ", data, p)
            if b"gfx950" in data[p + 24:p + 24 + name] and size:
                yield data[at + offset:at + offset + size]
            p += 24 + name
        at = data.find(BUNDLE, at + 1)


def kernels(elf):
    """The compiler's description of the kernels of an ELF64 file, from its AMDGPU note."""
    sections, = struct.unpack_from("<Q", elf, 40)
    size, count = struct.unpack_from("<HH", elf, 58)
    for i in range(count):
        kind, = struct.unpack_from("<I", elf, sections + i * size + 4)
        p, n = struct.unpack_from("<QQ", elf, sections + i * size + 24)
        end = p + n
        while kind == 7 and p < end:   # notes
            name, desc, what = struct.unpack_from("<III", elf, p)
            body = p + 12 + (name + 3) // 4 * 4
            if what == 32 and elf[p + 12:p + 18] == b"AMDGPU":
                yield from msgpack.unpackb(elf[body:body + desc])["amdhsa.kernels"]
            p = body + (desc + 3) // 4 * 4


def in_scratch(path):
    with open(path, "rb") as f:
        found = [k for elf in code_objects(f.read()) for k in kernels(elf)]
    assert len(found) > 100
    return [k[".name"] for k in found if k[".private_segment_fixed_size"] or k[".vgpr_spill_count"]]


def test_no_kernel_uses_scratch_memory():
    assert in_scratch(build.LIB) == []
