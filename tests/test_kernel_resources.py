"""What the compiler gave the convolution kernels, from the metadata of the built library's own code objects."""
import re
import struct

import msgpack

import paper_2006_02464_amd as cw
from paper_2006_02464_amd import build

BUNDLE = b"__CLANG_OFFLOAD_BUNDLE__"


def code_objects(data):
    pos = data.find(BUNDLE)
    while pos >= 0:
        n, at = struct.unpack_from("<Q", data, pos + 24)[0], pos + 32
        for _ in range(n):
            off, size, length = struct.unpack_from("<QQQ", data, at)
            if b"gfx950" in data[at + 24:at + 24 + length] and size:
                yield data[pos + off:pos + off + size]
            at += 24 + length
        pos = data.find(BUNDLE, pos + 24)


def kernels(path):
    """Every kernel's metadata by its mangled name: the AMDGPU note (type 32) of each ELF image."""
    out = {}
    for elf in code_objects(open(path, "rb").read()):
        table, = struct.unpack_from("<Q", elf, 0x28)
        entry, count = struct.unpack_from("<HH", elf, 0x3A)
        for i in range(count):
            _, kind, _, _, at, size, _, _, _, _ = struct.unpack_from("<IIQQQQIIQQ", elf, table + i * entry)
            end = at + size
            while kind == 7 and at < end:   # SHT_NOTE
                name, length, note = struct.unpack_from("<III", elf, at)
                desc = at + 12 + (name + 3) // 4 * 4
                if note == 32:
                    out.update((k[".name"], k) for k in msgpack.unpackb(elf[desc:desc + length], strict_map_key=False)["amdhsa.kernels"])
                at = desc + (length + 3) // 4 * 4
    return out


def test_convolution_tiles_need_no_scratch():
    """A tile whose registers do not fit reads and writes memory between the matrix instructions.  256x256 never fitted."""
    cw.lib()
    tile = re.compile(r"conv_dlds_(?:pair_)?kernelI\w*?Li(\d+)ELi(\d+)ELi")
    scratch = {}
    for name, k in kernels(build.LIB).items():
        m = tile.search(name)
        if m:
            scratch.setdefault(tuple(int(v) for v in m.groups()), []).append(k[".private_segment_fixed_size"])
    assert len(scratch) >= 14 and {(256, 128), (128, 256), (256, 256), (64, 64)} <= set(scratch)
    assert [t for t, b in scratch.items() if max(b) > 0] == [(256, 256)]
    assert max(scratch[256, 256]) <= 640   # bytes a lane
