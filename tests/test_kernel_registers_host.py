"""Registers of the logit tile kernels as built, from the metadata of the code objects in the library: two workgroups of 128 tiles or
one of 256 fit a compute unit only at 256 registers a lane, nothing is spilled to memory, and no accumulator lives in the
accumulation file, between which and the vector registers the compiler then copies in every K-step."""
import re
import struct

import msgpack

import paper_2304_08480_amd as dl


def _code_objects(blob):
    for m in re.finditer(b"__CLANG_OFFLOAD_BUNDLE__", blob):
        at = m.end()
        count, = struct.unpack_from("<Q", blob, at)
        at += 8
        for _ in range(count):
            offset, size, name_len = struct.unpack_from("<QQQ", blob, at)
            name = blob[at + 24:at + 24 + name_len]
            at += 24 + name_len
            if b"gfx950" in name:
                yield blob[m.start() + offset:m.start() + offset + size]


def _kernels(elf):
    """The entries of amdhsa.kernels in the ELF's note of AMD's code object metadata (type 32)."""
    shoff, = struct.unpack_from("<Q", elf, 40)
    shentsize, shnum = struct.unpack_from("<HH", elf, 58)
    for i in range(shnum):
        kind, = struct.unpack_from("<I", elf, shoff + i * shentsize + 4)
        offset, size = struct.unpack_from("<QQ", elf, shoff + i * shentsize + 24)
        at = offset
        while kind == 7 and at < offset + size:                       # SHT_NOTE
            name_len, desc_len, note = struct.unpack_from("<III", elf, at)
            desc = at + 12 + (name_len + 3) // 4 * 4
            if note == 32:
                yield from msgpack.unpackb(elf[desc:desc + desc_len])["amdhsa.kernels"]
            at = desc + (desc_len + 3) // 4 * 4


def test_logit_tile_kernels_keep_their_accumulators_in_vector_registers():
    with open(dl.library_path(), "rb") as f:
        blob = f.read()
    tiles = {k[".name"]: k for elf in _code_objects(blob) for k in _kernels(elf) if "k_logit_tiles" in k[".name"]}
    assert len(tiles) == 20                                           # 128 and 256; see TileKernels<T>::raise_lds
    for name, k in tiles.items():
        assert k[".agpr_count"] == 0 and k[".vgpr_spill_count"] == 0 and k[".vgpr_count"] <= 256, (name, k[".agpr_count"], k[".vgpr_spill_count"], k[".vgpr_count"])
