"""Resources of the compiled kernels, from the metadata of the code objects in
libspfel.so: no kernel may need scratch memory (spilled registers, or a private
array indexed by a value the compiler does not know, which costs every launch
of the kernel, also where the array is not reached)."""
import os
import struct

import msgpack
import pytest

from paper_2109_05339_amd import LIB_PATH

MAGIC = b"__CLANG_OFFLOAD_BUNDLE__"


def code_objects(blob):
    """The gfx950 ELF images of every offload bundle in a shared library."""
    at = blob.find(MAGIC)
    while at >= 0:
        count, = struct.unpack_from("<Q", blob, at + len(MAGIC))
        p = at + len(MAGIC) + 8
        for _ in range(count):
            off, size, n = struct.unpack_from("<QQQ", blob, p)
            name = blob[p + 24:p + 24 + n].decode()
            p += 24 + n
            if "gfx950" in name and size:
                yield blob[at + off:at + off + size]
        at = blob.find(MAGIC, at + len(MAGIC))


def kernels(elf):
    """The kernel records of an AMDGPU ELF image's metadata note."""
    shoff, = struct.unpack_from("<Q", elf, 0x28)
    shentsize, shnum = struct.unpack_from("<HH", elf, 0x3A)
    for k in range(shnum):
        sh = shoff + k * shentsize
        kind, = struct.unpack_from("<I", elf, sh + 4)
        off, size = struct.unpack_from("<QQ", elf, sh + 0x18)
        p = off
        while kind == 7 and p < off + size:   # SHT_NOTE
            namesz, descsz, note = struct.unpack_from("<III", elf, p)
            name = elf[p + 12:p + 12 + namesz]
            p += 12 + (namesz + 3) // 4 * 4
            if note == 32 and name.startswith(b"AMDGPU"):   # NT_AMDGPU_METADATA
                yield from msgpack.unpackb(elf[p:p + descsz], strict_map_key=False)["amdhsa.kernels"]
            p += (descsz + 3) // 4 * 4


@pytest.mark.skipif(not os.path.exists(LIB_PATH), reason="library not built")
def test_no_kernel_needs_scratch():
    with open(LIB_PATH, "rb") as f:
        found = [k for elf in code_objects(f.read()) for k in kernels(elf)]
    assert len(found) > 100
    scratch = {k[".name"]: k[".private_segment_fixed_size"] for k in found if k[".private_segment_fixed_size"]}
    assert not scratch
