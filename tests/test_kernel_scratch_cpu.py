"""Register allocation of the built slice GEMM kernels, from the metadata of the library's gfx950
code objects: no kernel that forms C spills vector registers to scratch memory."""
import os
import re
import struct

import msgpack

import paper_2603_29975_amd as oz

MAGIC = b"__CLANG_OFFLOAD_BUNDLE__"


def _code_objects(blob):
    """The gfx950 ELF images of every offload bundle in the file."""
    at = blob.find(MAGIC)
    while at >= 0:
        count, = struct.unpack_from("<Q", blob, at + len(MAGIC))
        p = at + len(MAGIC) + 8
        for _ in range(count):
            off, size, n = struct.unpack_from("<QQQ", blob, p)
            name = blob[p + 24:p + 24 + n]
            p += 24 + n
            if b"gfx950" in name and size:
                yield blob[at + off:at + off + size]
        at = blob.find(MAGIC, at + 1)


def _kernels(elf):
    """The kernels' metadata (the note of type 32 of an AMDGPU code object)."""
    shoff, = struct.unpack_from("<Q", elf, 40)
    shentsize, shnum = struct.unpack_from("<HH", elf, 58)
    for i in range(shnum):
        kind, = struct.unpack_from("<I", elf, shoff + i * shentsize + 4)
        if kind != 7:  # SHT_NOTE
            continue
        off, size = struct.unpack_from("<QQ", elf, shoff + i * shentsize + 24)
        namesz, descsz, ntype = struct.unpack_from("<III", elf, off)
        if ntype == 32:
            start = off + 12 + (namesz + 3) // 4 * 4
            return msgpack.unpackb(elf[start:start + descsz], strict_map_key=False)["amdhsa.kernels"]
    return []


def test_slice_gemm_kernels_keep_their_accumulators_in_registers():
    with open(oz.library_path, "rb") as f:
        blob = f.read()
    seen, spilled = 0, []
    for elf in _code_objects(blob):
        for k in _kernels(elf):
            # k_ozgemm<S, WJ, WI, IB, WPS, RING, LA, RAW, MODE>; RAW (debug output) may spill
            m = re.search(r"k_ozgemmILi(\d+)E.*ELb0ELi([012])EE", k[".name"])
            if m is None:
                continue
            seen += 1
            if k[".private_segment_fixed_size"] or k[".vgpr_spill_count"]:
                spilled.append((k[".name"], k[".private_segment_fixed_size"]))
    assert seen >= 100
    assert not spilled, spilled
