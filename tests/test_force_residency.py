"""The force kernels' workgroups are all resident at once (no GPU: the built
library's own kernel descriptors).  A block's first work item is the one of its
number, so a launch must not start more blocks than the registers and LDS of
its kernel leave room for: 6 per CU in FP32, 5 in FP64, 3 in FP64 with the
collision branch.  gfx950: 512 VGPRs per lane and SIMD in units of 8, 160 KB of
LDS per CU, a block of 256 threads puts one wave on each SIMD."""
import os
import re
import struct

import msgpack

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LIB = os.path.join(ROOT, "paper_1907_02289_amd", "libbh.so")
MAGIC = b"__CLANG_OFFLOAD_BUNDLE__"


def _code_objects(data):
    """The gfx950 ELF images of the library's offload bundles."""
    at = data.find(MAGIC)
    while at >= 0:
        n = struct.unpack_from("<Q", data, at + len(MAGIC))[0]
        p = at + len(MAGIC) + 8
        for _ in range(n):
            off, size, idlen = struct.unpack_from("<QQQ", data, p)
            name = data[p + 24:p + 24 + idlen]
            p += 24 + idlen
            if b"gfx950" in name and size:
                yield data[at + off:at + off + size]
        at = data.find(MAGIC, at + 1)


def _kernels(elf):
    """Kernel descriptions (AMDGPU metadata note, type 32) of one image."""
    phoff = struct.unpack_from("<Q", elf, 32)[0]
    phsize, phnum = struct.unpack_from("<HH", elf, 54)
    for k in range(phnum):
        kind, _, off, _, _, size = struct.unpack_from("<IIQQQQ", elf, phoff + k * phsize)
        if kind != 4:
            continue
        p = off
        while p < off + size:
            namesz, descsz, note = struct.unpack_from("<III", elf, p)
            p += 12 + (namesz + 3) // 4 * 4
            if note == 32:
                yield from msgpack.unpackb(elf[p:p + descsz], strict_map_key=False)["amdhsa.kernels"]
            p += (descsz + 3) // 4 * 4


def test_every_launched_block_is_resident():
    if not os.path.exists(LIB):
        from paper_1907_02289_amd import build
        build.build()
    data = open(LIB, "rb").read()
    found = {}
    for elf in _code_objects(data):
        for k in _kernels(elf):
            m = re.search(r"k_forceI([fd])Lb([01])ELb([01])ELb([01])ELi(\d+)E", k[".name"])
            if m:
                found[m.groups()] = k
    assert len(found) == 4 * (2 + 1) + 4 * 2          # FP32 tiles 512 and 256 and collisions, FP64 and collisions
    for (real, _, _, coll, tile), k in found.items():
        want = 6 if real == "f" else 3 if coll == "1" else 5
        vgprs = (k[".vgpr_count"] + 7) // 8 * 8
        lds = k[".group_segment_fixed_size"]
        assert min(512 // vgprs, 160 * 1024 // lds) >= want, (k[".name"], vgprs, lds)
