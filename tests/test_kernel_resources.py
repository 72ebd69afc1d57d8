"""What the built library's kernels ask for, from the code objects' own metadata: none of them keeps anything in scratch memory (a
function that was not inlined had the kernel copy its parameters there: 40.8 us for a head of 38323 rows of 599 instead of 31.5)."""
import os
import struct

import msgpack
import pytest

import paper_2412_00061_amd as pkg

LIB = os.path.join(os.path.dirname(os.path.abspath(pkg.__file__)), "libctcspec.so")
MAGIC = b"__CLANG_OFFLOAD_BUNDLE__"


def _notes(elf):
    """The AMDGPU metadata notes (type 32) of a 64-bit little-endian ELF."""
    phoff, = struct.unpack_from("<Q", elf, 32)
    phentsize, phnum = struct.unpack_from("<HH", elf, 54)
    for i in range(phnum):
        kind, _, offset, _, _, size = struct.unpack_from("<IIQQQQ", elf, phoff + i * phentsize)
        at, end = offset, offset + size
        while kind == 4 and at + 12 <= end:  # PT_NOTE
            name, desc, what = struct.unpack_from("<III", elf, at)
            body = at + 12 + (name + 3) // 4 * 4
            if what == 32:
                yield msgpack.unpackb(elf[body:body + desc])
            at = body + (desc + 3) // 4 * 4


def _kernels():
    with open(LIB, "rb") as f:
        data = f.read()
    at = data.find(MAGIC)
    while at >= 0:
        count, = struct.unpack_from("<Q", data, at + len(MAGIC))
        entry = at + len(MAGIC) + 8
        for _ in range(count):
            offset, size, length = struct.unpack_from("<QQQ", data, entry)
            triple = data[entry + 24:entry + 24 + length]
            entry += 24 + length
            if b"gfx950" in triple and size:
                for note in _notes(data[at + offset:at + offset + size]):
                    yield from note["amdhsa.kernels"]
        at = data.find(MAGIC, at + 1)


def test_no_kernel_uses_scratch():
    if not os.path.exists(LIB):
        pytest.skip("the library is not built")
    kernels = list(_kernels())
    assert len(kernels) > 100
    assert not [(k[".name"], k[".private_segment_fixed_size"]) for k in kernels if k[".private_segment_fixed_size"]]
    assert not [k[".name"] for k in kernels if k.get(".vgpr_spill_count")]
