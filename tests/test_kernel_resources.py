"""What the compiled kernels take, read from the code objects' own metadata in the built library: no
kernel launched on its own uses scratch memory (a spill in the per-entry loops of the blend costs every
frame), and the forward blend keeps the registers of seven waves per SIMD."""
import struct

import msgpack

from paper_2510_09997_amd import build

MAGIC = b"__CLANG_OFFLOAD_BUNDLE__"


def code_objects(data):
    """The gfx950 entries of the offload bundles in a file: (offset, size, triple) tables after a magic."""
    at = data.find(MAGIC)
    while at >= 0:
        (count,) = struct.unpack_from("<Q", data, at + len(MAGIC))
        pos = at + len(MAGIC) + 8
        for _ in range(count):
            offset, size, n = struct.unpack_from("<QQQ", data, pos)
            triple = data[pos + 24:pos + 24 + n].decode()
            pos += 24 + n
            if triple.endswith(build.ARCH) and size:
                yield data[at + offset:at + offset + size]
        at = data.find(MAGIC, at + len(MAGIC))


def kernels(elf):
    """amdhsa.kernels of an ELF64 code object: the msgpack note (type 32) of its note sections."""
    (table,) = struct.unpack_from("<Q", elf, 0x28)
    entry, count = struct.unpack_from("<HH", elf, 0x3A)
    for k in range(count):
        head = table + k * entry
        (kind,) = struct.unpack_from("<I", elf, head + 4)
        if kind != 7:   # SHT_NOTE
            continue
        pos, size = struct.unpack_from("<QQ", elf, head + 24)
        end = pos + size
        while pos < end:
            name, desc, note = struct.unpack_from("<III", elf, pos)
            pos += 12 + (name + 3) // 4 * 4
            if note == 32:
                yield from msgpack.unpackb(elf[pos:pos + desc], raw=False)["amdhsa.kernels"]
            pos += (desc + 3) // 4 * 4


def test_no_kernel_spills():
    found = {k[".name"]: k for elf in code_objects(open(build.LIB, "rb").read()) for k in kernels(elf)}
    assert len(found) >= 40 and any("k_blend_fwd" in name for name in found)
    # (The resident server runs every stage in one kernel, at one workgroup per compute unit.)
    scratch = {name: k[".private_segment_fixed_size"] for name, k in found.items()
               if k[".private_segment_fixed_size"] and "k_server" not in name}
    assert scratch == {}
    blend = [k[".vgpr_count"] for name, k in found.items() if "k_blend_fwdILb0" in name]
    assert len(blend) == 1 and blend[0] <= 72
