"""What the built kernels of libaps.so ask of the GPU, from the metadata the
compiler writes beside them (CPU; no GPU needed)."""
from __future__ import annotations

import os
import struct

import pytest

from paper_1911_08907_amd import aps as A

MAGIC = b"__CLANG_OFFLOAD_BUNDLE__"


def _code_objects(blob: bytes):
    """The gfx950 ELF images of every offload bundle in a host library."""
    at = blob.find(MAGIC)
    while at >= 0:
        pos = at + len(MAGIC)
        count, = struct.unpack_from("<Q", blob, pos)
        pos += 8
        for _ in range(count):
            off, size, idlen = struct.unpack_from("<QQQ", blob, pos)
            pos += 24
            if b"gfx950" in blob[pos:pos + idlen]:
                yield blob[at + off:at + off + size]
            pos += idlen
        at = blob.find(MAGIC, pos)


def _kernels(elf: bytes, msgpack):
    """The kernels' metadata maps (note type 32, name AMDGPU) of one ELF image."""
    shoff, = struct.unpack_from("<Q", elf, 0x28)
    shentsize, shnum = struct.unpack_from("<HH", elf, 0x3A)
    for i in range(shnum):
        sh = shoff + i * shentsize
        if struct.unpack_from("<I", elf, sh + 4)[0] != 7:  # SHT_NOTE
            continue
        off, size = struct.unpack_from("<QQ", elf, sh + 0x18)
        namesz, descsz, kind = struct.unpack_from("<III", elf, off)
        desc = off + 12 + (namesz + 3) // 4 * 4
        if kind == 32:
            yield from msgpack.unpackb(elf[desc:desc + descsz])["amdhsa.kernels"]


def test_ordered_reduce_keeps_its_row_walk_in_registers():
    """No instance of the ordered sum's kernel takes more than a few registers'
    worth of scratch: with a second copy of the row walk held to the same 128
    registers the m = 0 formats' took 224 bytes a lane, within the walk, and
    ran up to 1.18 times slower."""
    msgpack = pytest.importorskip("msgpack")
    if not os.path.exists(A.LIB_PATH):
        pytest.skip("libaps.so is not built")
    blob = open(A.LIB_PATH, "rb").read()
    scratch = {k[".name"]: k[".private_segment_fixed_size"]
               for elf in _code_objects(blob) for k in _kernels(elf, msgpack)}
    ex = {n: s for n, s in scratch.items() if "15k_sim_reduce_ex" in n}
    assert len(ex) >= 20
    assert max(ex.values()) <= 48, {n: s for n, s in ex.items() if s > 48}
