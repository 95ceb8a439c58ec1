"""What the compiler gave each kernel of libqe.so: registers, spills, scratch.

The library's `.hip_fatbin` holds one offload bundle per source file, each with a gfx950 ELF whose
NT_AMDGPU_METADATA note (MessagePack) lists its kernels.
"""
import struct

import msgpack

_MAGIC = b"__CLANG_OFFLOAD_BUNDLE__"


def _notes(elf):
    """The descriptor of every note of type 32 (AMDGPU metadata) of a 64-bit little-endian ELF."""
    shoff, = struct.unpack_from("<Q", elf, 0x28)
    shentsize, shnum = struct.unpack_from("<HH", elf, 0x3A)
    for i in range(shnum):
        _, kind, _, _, off, size = struct.unpack_from("<IIQQQQ", elf, shoff + i * shentsize)
        if kind != 7:  # SHT_NOTE
            continue
        at, end = off, off + size
        while at + 12 <= end:
            namesz, descsz, ntype = struct.unpack_from("<III", elf, at)
            desc = at + 12 + (namesz + 3) // 4 * 4
            if ntype == 32:
                yield elf[desc:desc + descsz]
            at = desc + (descsz + 3) // 4 * 4


def kernels(lib_path):
    """{mangled kernel name: its metadata} of every gfx950 kernel in the library."""
    blob = open(lib_path, "rb").read()
    found, at = {}, blob.find(_MAGIC)
    while at >= 0:
        count, = struct.unpack_from("<Q", blob, at + len(_MAGIC))
        pos = at + len(_MAGIC) + 8
        for _ in range(count):
            off, size, idlen = struct.unpack_from("<QQQ", blob, pos)
            target = blob[pos + 24:pos + 24 + idlen]
            pos += 24 + idlen
            if size and b"gfx950" in target:
                for desc in _notes(blob[at + off:at + off + size]):
                    for k in msgpack.unpackb(desc, strict_map_key=False)["amdhsa.kernels"]:
                        found[k[".name"]] = k
        at = blob.find(_MAGIC, at + 1)
    return found
