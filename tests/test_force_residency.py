"""The force kernels' workgroups are all resident at once (no GPU: the built
library's own kernel descriptors).  A block's first work item is the one of its
number, so a launch must not start more blocks than the registers and LDS of
its kernel leave room for: 6 per CU in FP32, 5 in FP64, 3 in FP64 with the
collision branch.  The same for the two blocks of the bucket sort.  gfx950: 512 VGPRs per lane and SIMD in units of 8, 160 KB of
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


def _built(pattern):
    """The library's kernels whose name matches, by the match's groups."""
    if not os.path.exists(LIB):
        from paper_1907_02289_amd import build
        build.build()
    found = {}
    for elf in _code_objects(open(LIB, "rb").read()):
        for k in _kernels(elf):
            m = re.search(pattern, k[".name"])
            if m:
                found[m.groups()] = k
    return found


def _resident(k, waves_per_simd):
    """Blocks of a kernel that fit a CU, with that many of a block's waves on each SIMD."""
    vgprs = (k[".vgpr_count"] + 7) // 8 * 8
    return min(512 // vgprs // waves_per_simd, 160 * 1024 // k[".group_segment_fixed_size"])


def test_every_launched_block_is_resident():
    found = _built(r"k_forceI([fd])Lb([01])ELb([01])ELb([01])ELi(\d+)E")
    assert len(found) == 4 * (2 + 1) + 4 * 2          # FP32 tiles 512 and 256 and collisions, FP64 and collisions
    for (real, _, _, coll, _), k in found.items():
        want = 6 if real == "f" else 3 if coll == "1" else 5
        assert _resident(k, 1) >= want, (k[".name"], k[".vgpr_count"], k[".group_segment_fixed_size"])


def test_two_blocks_of_the_bucket_sort_fit_a_cu():
    """The sample sort's bucket capacities are chosen for two blocks (of 512 threads) per CU."""
    found = _built(r"k_ss_sortILi(\d+)ELb([01])E")
    assert len(found) == 4
    for k in found.values():
        assert _resident(k, 2) >= 2, (k[".name"], k[".vgpr_count"], k[".group_segment_fixed_size"])
