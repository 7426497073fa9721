"""Registers and scratch of the library's kernels, from the metadata of the code
objects in libcfd.so (the note that the compiler writes beside each kernel)."""
import struct

import msgpack

EM_AMDGPU, SHT_NOTE, NT_AMDGPU_METADATA = 224, 7, 32


def kernels(path):
    """{mangled name: (vector registers, scratch bytes a lane)}"""
    with open(path, "rb") as f:
        b = f.read()
    out = {}
    at = b.find(b"\x7fELF\x02", 4)  # the library is an ELF file itself; the code objects lie inside it
    while at >= 0:
        if struct.unpack_from("<H", b, at + 18)[0] == EM_AMDGPU:
            table = at + struct.unpack_from("<Q", b, at + 40)[0]
            size, count = struct.unpack_from("<HH", b, at + 58)
            for i in range(count):
                _, kind, _, _, offset, length = struct.unpack_from("<IIQQQQ", b, table + i * size)
                p, end = at + offset, at + offset + length
                while kind == SHT_NOTE and p < end:
                    name, desc, note = struct.unpack_from("<III", b, p)
                    p += 12 + (name + 3) // 4 * 4
                    if note == NT_AMDGPU_METADATA:
                        for k in msgpack.unpackb(b[p:p + desc])["amdhsa.kernels"]:
                            out[k[".name"]] = (k[".vgpr_count"], k[".private_segment_fixed_size"])
                    p += (desc + 3) // 4 * 4
        at = b.find(b"\x7fELF\x02", at + 4)
    return out
