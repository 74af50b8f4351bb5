"""What the built kernels ask of a CU, from the metadata of the library's own code objects.

The front end of a prefill batch runs while the shared experts' gate/up launch starts on another stream.  That launch's
blocks (four waves of up to 224 registers per lane, 64 KB of LDS) have to fit on a CU beside a block of the front end, or
they wait for it."""
import os
import struct

import msgpack
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LIB = os.path.join(ROOT, "paper_2504_05897_amd", "libhmoe.so")
MAGIC = b"__CLANG_OFFLOAD_BUNDLE__"


def code_objects(data):
    """The gfx950 ELF images of the offload bundles in a shared library (one bundle per source file)."""
    at = data.find(MAGIC)
    while at >= 0:
        n, = struct.unpack_from("<Q", data, at + 24)
        pos = at + 32
        for _ in range(n):
            offset, size, id_len = struct.unpack_from("<QQQ", data, pos)
            target = data[pos + 24:pos + 24 + id_len].decode()
            pos += 24 + id_len
            if "gfx950" in target and size:
                yield data[at + offset:at + offset + size]
        at = data.find(MAGIC, at + 24)


def kernels_of(elf):
    """name -> metadata, from the note section an AMDGPU code object carries."""
    shoff, = struct.unpack_from("<Q", elf, 0x28)
    shentsize, shnum = struct.unpack_from("<HH", elf, 0x3A)
    for i in range(shnum):
        header = struct.unpack_from("<IIQQQQ", elf, shoff + i * shentsize)
        if header[1] != 7:  # SHT_NOTE
            continue
        pos, end = header[4], header[4] + header[5]
        while pos < end:
            name_size, size, kind = struct.unpack_from("<III", elf, pos)
            body = pos + 12 + (name_size + 3) // 4 * 4
            if kind == 32:  # the metadata of the kernels
                for k in msgpack.unpackb(elf[body:body + size])["amdhsa.kernels"]:
                    yield k[".name"], k
            pos = body + (size + 3) // 4 * 4


@pytest.fixture(scope="module")
def kernels():
    with open(LIB, "rb") as f:
        data = f.read()
    found = {name: k for elf in code_objects(data) for name, k in kernels_of(elf)}
    assert len(found) > 50
    return found


def test_front_end_blocks_leave_room_for_the_shared_experts(kernels):
    """Blocks of up to 16 tokens, 128 experts (larger ones take no more than half of the CUs until those are full anyway;
    more experts keep sixteen waves: there w_g is what the batch waits for)."""
    shared = kernels["_ZN4hmoe19ffn_tile_fit_kernelILb1ELi4ELb0EEEvNS_8TiledCtxEPKtPt"]
    blocks = {n: k for n, k in kernels.items() if "front_tokens_kernel" in n and "RouterShapeILi1E" in n and "ILi64ELi4E" not in n}
    assert len(blocks) == 5
    for name, k in blocks.items():
        waves = k[".max_flat_workgroup_size"] // 64
        registers = (k[".vgpr_count"] + 7) // 8 * 8 * waves // 4  # per lane of a SIMD, four SIMDs
        assert registers + (shared[".vgpr_count"] + 7) // 8 * 8 <= 512, (name, waves, k[".vgpr_count"])
        assert k[".group_segment_fixed_size"] + shared[".group_segment_fixed_size"] <= 160 * 1024, name
