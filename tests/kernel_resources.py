"""What the compiler gave each kernel of the built library: static LDS, private
memory and registers, from the metadata notes of its gfx950 code objects."""
import os
import re
import struct

import msgpack

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LIB = os.path.join(ROOT, "paper_1804_07250_amd", "libtilings.so")
LDS_BYTES = 160 * 1024   # of a compute unit


def _notes(elf):
    """Descriptors of the metadata notes (type 32) of one code object."""
    shoff, = struct.unpack_from("<Q", elf, 0x28)
    shentsize, shnum = struct.unpack_from("<HH", elf, 0x3A)
    for i in range(shnum):
        sh = shoff + i * shentsize
        kind, = struct.unpack_from("<I", elf, sh + 4)
        off, size = struct.unpack_from("<QQ", elf, sh + 24)
        if kind != 7:   # SHT_NOTE
            continue
        at, end = off, off + size
        while at < end:
            namesz, descsz, typ = struct.unpack_from("<III", elf, at)
            desc = at + 12 + (namesz + 3) // 4 * 4
            if typ == 32:
                yield elf[desc:desc + descsz]
            at = desc + (descsz + 3) // 4 * 4


def kernels():
    """{demangled-enough name: metadata} of every kernel of the library."""
    data = open(LIB, "rb").read()
    out = {}
    for m in re.finditer(b"__CLANG_OFFLOAD_BUNDLE__", data):
        base = m.start()
        count, = struct.unpack_from("<Q", data, base + 24)
        at = base + 32
        for _ in range(count):
            off, size, idlen = struct.unpack_from("<QQQ", data, at)
            name = data[at + 24:at + 24 + idlen]
            at += 24 + idlen
            if b"gfx950" not in name or size == 0:
                continue
            for desc in _notes(data[base + off:base + off + size]):
                for k in msgpack.unpackb(desc, strict_map_key=False).get("amdhsa.kernels", []):
                    out[k[".name"]] = k
    return out
