"""Registers of the kernels of the built library, from the metadata that the
compiler leaves in its code objects."""
import re
import struct

import msgpack


def _code_objects(data):
    at = data.find(b"__CLANG_OFFLOAD_BUNDLE__")
    while at >= 0:
        (n,) = struct.unpack_from("<Q", data, at + 24)
        o = at + 32
        for _ in range(n):
            off, size, ln = struct.unpack_from("<QQQ", data, o)
            name = data[o + 24:o + 24 + ln]
            o += 24 + ln
            if name.startswith(b"hip") and size:
                yield data[at + off:at + off + size]
        at = data.find(b"__CLANG_OFFLOAD_BUNDLE__", at + 24)


def _metadata(elf):
    shoff, = struct.unpack_from("<Q", elf, 0x28)
    shentsize, shnum = struct.unpack_from("<HH", elf, 0x3A)
    for i in range(shnum):
        kind, _, _, off, size = struct.unpack_from("<IQQQQ", elf, shoff + i * shentsize + 4)
        o, end = off, off + size
        while kind == 7 and o < end:  # SHT_NOTE
            namesz, descsz, typ = struct.unpack_from("<III", elf, o)
            name = elf[o + 12:o + 12 + namesz].rstrip(b"\0")
            d = o + 12 + (namesz + 3) // 4 * 4
            if name == b"AMDGPU" and typ == 32:
                yield msgpack.unpackb(elf[d:d + descsz], strict_map_key=False)
            o = d + (descsz + 3) // 4 * 4


def kernels(path):
    """{mangled name: vector registers} of every kernel of the library."""
    out = {}
    with open(path, "rb") as f:
        data = f.read()
    for elf in _code_objects(data):
        for md in _metadata(elf):
            for k in md["amdhsa.kernels"]:
                out[k[".name"]] = k[".vgpr_count"] + k.get(".agpr_count", 0)
    return out


def wavefronts(vgprs):
    """Wavefronts that a SIMD's 512 registers a lane hold (blocks of 8, at most 8 wavefronts)."""
    return min(8, 512 // (-(-max(vgprs, 1) // 8) * 8))


def find(table, name, args):
    """Registers of the kernel `name` with the mangled template arguments `args`."""
    hits = [v for k, v in table.items() if re.search(r"\d%sI%sE" % (name, args), k)]
    assert len(hits) >= 1, (name, args)
    return max(hits)
