"""Registers and LDS of the kernels in the built library, from the metadata notes of its code objects (our own build, read from the
file, nothing is loaded)."""

import functools
import re
import struct
import subprocess
from collections import namedtuple

import msgpack

from paper_2510_18413_amd import build as B

Kernel = namedtuple("Kernel", "vgprs sgprs spilled scratch lds")
BUNDLE = b"__CLANG_OFFLOAD_BUNDLE__"


def _code_objects(blob):
    at = blob.find(BUNDLE)
    while at >= 0:
        n, pos = struct.unpack_from("<Q", blob, at + len(BUNDLE))[0], at + len(BUNDLE) + 8
        for _ in range(n):
            offset, size, name = struct.unpack_from("<QQQ", blob, pos)
            target = blob[pos + 24:pos + 24 + name]
            pos += 24 + name
            if b"gfx950" in target and size:
                yield blob[at + offset:at + offset + size]
        at = blob.find(BUNDLE, at + 1)


def _metadata(elf):
    """The NT_AMDGPU_METADATA note (type 32) of an ELF64 file."""
    table, = struct.unpack_from("<Q", elf, 40)
    entry, count = struct.unpack_from("<HH", elf, 58)
    for i in range(count):
        kind, = struct.unpack_from("<I", elf, table + i * entry + 4)
        offset, size = struct.unpack_from("<QQ", elf, table + i * entry + 24)
        pos, end = offset, offset + size
        while kind == 7 and pos < end:      # SHT_NOTE
            name, desc, note = struct.unpack_from("<III", elf, pos)
            pos += 12 + (name + 3) // 4 * 4
            if note == 32:
                return msgpack.unpackb(elf[pos:pos + desc], strict_map_key=False)
            pos += (desc + 3) // 4 * 4
    return {}


@functools.lru_cache(maxsize=1)
def kernels():
    """{"name<arguments>": Kernel} of every kernel, template arguments as the demangler writes them."""
    got = {}
    for elf in _code_objects(B.LIB.read_bytes()):
        for k in _metadata(elf).get("amdhsa.kernels", []):
            got[k[".name"]] = Kernel(k[".vgpr_count"], k[".sgpr_count"], k.get(".vgpr_spill_count", 0) + k.get(".sgpr_spill_count", 0),
                                     k[".private_segment_fixed_size"], k[".group_segment_fixed_size"])
    names = subprocess.run(["c++filt"], input="\n".join(got), capture_output=True, text=True, check=True).stdout.split("\n")
    return {re.sub(r"^void adamas::|\(adamas::.*$", "", n): k for n, k in zip(names, got.values())}


def waves_per_simd(kernel):
    """Waves that the vector registers leave room for: 512 of them per lane, eight at a time."""
    return min(8, 512 // ((kernel.vgprs + 7) // 8 * 8))
