"""Resource figures of the kernels in a built library, from the metadata notes
of its code objects (test infrastructure)."""
from __future__ import annotations

import struct

import msgpack

_MAGIC = b"__CLANG_OFFLOAD_BUNDLE__"


def _sections(elf):
    """(name, type, bytes) of every section of a 64-bit ELF image."""
    shoff, = struct.unpack_from("<Q", elf, 0x28)
    size, num, names = struct.unpack_from("<HHH", elf, 0x3A)
    head = [struct.unpack_from("<IIQQQQ", elf, shoff + i * size) for i in range(num)]
    table = head[names][4]
    for name, kind, _, _, off, length in head:
        end = elf.index(b"\0", table + name)
        yield elf[table + name:end].decode(), kind, elf[off:off + length]


def _device_images(blob):
    at = blob.find(_MAGIC)
    while at >= 0:
        count, = struct.unpack_from("<Q", blob, at + len(_MAGIC))
        pos = at + len(_MAGIC) + 8
        for _ in range(count):
            off, size, n = struct.unpack_from("<QQQ", blob, pos)
            triple = blob[pos + 24:pos + 24 + n]
            pos += 24 + n
            if size and b"amdgcn" in triple:
                yield blob[at + off:at + off + size]
        at = blob.find(_MAGIC, at + len(_MAGIC))


def kernels(path):
    """{mangled name: metadata map} of the library's kernels."""
    with open(path, "rb") as f:
        host = f.read()
    out = {}
    for name, _, blob in _sections(host):
        if name != ".hip_fatbin":
            continue
        for image in _device_images(blob):
            for _, kind, notes in _sections(image):
                at = 0
                while kind == 7 and at + 12 <= len(notes):   # SHT_NOTE
                    n_name, n_desc, n_type = struct.unpack_from("<III", notes, at)
                    desc = at + 12 + (n_name + 3) // 4 * 4
                    if n_type == 32 and notes[at + 12:at + 18] == b"AMDGPU":   # code object metadata
                        for k in msgpack.unpackb(notes[desc:desc + n_desc])["amdhsa.kernels"]:
                            out[k[".name"]] = k
                    at = desc + (n_desc + 3) // 4 * 4
    return out
