"""What the compiler gave the convolution kernels, from the metadata of the built library's own code objects."""
import re
import struct
import subprocess

import msgpack

import paper_2006_02464_amd as cw
from oracle import topology as T
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


OPS = [T.Op(T.CONV, 3, 64, 7, 7, 2, 3, 1, -1, -1), T.Op(T.CONV, 64, 512, 3, 3, 1, 1, 1, -1, 0), T.Op(T.CONV, 512, 512, 1, 1, 1, 0, 1, -1, 1),
       T.Op(T.CONV, 512, 96, 1, 1, 1, 0, 1, -1, 2), T.Op(T.CONV, 96, 512, 1, 1, 1, 0, 1, -1, 3), T.Op(T.CONV, 512, 512, 3, 3, 1, 1, 1, -1, 4),
       T.Op(T.GAVGPOOL, 512, 512, 0, 0, 1, 0, 0, -1, 5), T.Op(T.FC, 512, 10, 1, 1, 1, 0, 0, -1, 6), T.Op(T.SOFTMAX, 10, 10, 0, 0, 1, 0, 0, -1, 7)]


def test_workgroups_have_the_threads_that_the_plan_tells():
    """block + cw_plan_launch_loaders of every plain form, whole and split K, as its kernel was compiled for."""
    form = re.compile(r"conv_dlds_kernelIDF16_Li(\d+)ELi(\d+)ELi(\d+)ELi(\d+)ELi(\d+)ELi\d+ELi(\d+)ELb([01])ELb0ELi(\d+)ELi(16|32)E")
    compiled = {}
    for name, k in kernels(build.LIB).items():
        m = form.search(name)
        if m:
            bm, bn, wm, wn, bk, mode, split, kg, mt = (int(v) for v in m.groups())
            compiled.setdefault((bm, bn, 64 * wm * wn * kg, bk, mode, split, kg), set()).add(k[".max_flat_workgroup_size"])
    ctx = cw.Context(device=-1)
    seen = set()
    try:
        for name, tile in cw.CONV_TILES.items():
            for split in (1, 2):
                ctx.set_plan_override(tile, split)
                mid = ctx.model_define(OPS, 3, 32, 32, batch_sizes=(1,), dtype="fp16")
                for i, l in enumerate(ctx.plan(mid, 1)):
                    if l["kind"] != 1 or l["grid_z"] > 1:   # tiles in parts: a part's sizes are not reported
                        continue
                    o = OPS[l["op_index"]]
                    mode = 2 if l["op_index"] == 0 else 0 if o.kh > 1 else 1 if o.cin % l["tile_k"] == 0 else 3
                    threads = l["block"] + ctx.plan_launch_loaders(mid, 1, i)
                    assert threads in compiled[l["tile_m"], l["tile_n"], l["block"], l["tile_k"], mode, int(l["split_k"] > 1), l["wave_groups"]], (name, l)
                    seen.add((threads > l["block"], mode, l["split_k"] > 1))
    finally:
        ctx.destroy()
    assert {k for k in seen if k[0]} == {(True, m, False) for m in (0, 1, 3)} and {(False, m, True) for m in range(4)} <= seen


READ_AHEAD = r"""
#include "common.h"
using namespace cw;
// Lines that workgroup `wg` of a launch's `wgs` reads: thread t from wg * readers + t on, every wgs * readers.
constexpr int lines_of(int wg, int wgs, int readers, int lines) {
    int n = 0;
    for (int i = wg * readers; i < lines; i += wgs * readers) n += lines - i < readers ? lines - i : readers;
    return n;
}
constexpr bool even(int lines, int threads) {
    const int wgs = conv_prefetch_wgs(lines), readers = conv_prefetch_threads(threads), each = (lines + wgs - 1) / wgs;
    int all = 0;
    for (int wg = 0; wg < wgs; ++wg) {
        const int n = lines_of(wg, wgs, readers, lines);
        if (n > (each + kPrefetchLines - 1) / kPrefetchLines * kPrefetchLines) return false;
        all += n;
    }
    return all == lines && readers <= threads;
}
constexpr bool even_for(int threads) { return even(2048, threads) && even(9216, threads) && even(9217, threads) && even(16384, threads) && even(18432, threads) && even(36864, threads); }
static_assert(even_for(64) && even_for(128) && even_for(256) && even_for(320) && even_for(384) && even_for(512) && even_for(768) && even_for(1024), "");
"""


def test_reading_ahead_is_spread_over_its_workgroups(tmp_path):
    """However many threads a workgroup has, those that read ahead take 256 lines each (more where 64 of them are too few)."""
    src = tmp_path / "read_ahead.hip"
    src.write_text(READ_AHEAD)
    subprocess.run(["hipcc", "--offload-arch=gfx950", "--offload-host-only", "-std=c++17", "-fsyntax-only", "-I", build.CSRC, str(src)], check=True)
