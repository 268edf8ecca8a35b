"""Registers of the kernels whose speed hangs on the waves they leave resident
on a SIMD (512 vector registers, handed out by 8), read from the metadata of
the built library's gfx950 code objects."""
import os
import struct

import msgpack
import pytest

LIB = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_1804_00695_amd",
                   "libmlspgemm.so")


def code_objects(data):
    at = data.find(b"__CLANG_OFFLOAD_BUNDLE__")
    while at >= 0:
        n, pos = struct.unpack_from("<Q", data, at + 24)[0], at + 32
        for _ in range(n):
            off, size, idlen = struct.unpack_from("<QQQ", data, pos)
            name = data[pos + 24:pos + 24 + idlen]
            pos += 24 + idlen
            if b"gfx950" in name:
                yield data[at + off:at + off + size]
        at = data.find(b"__CLANG_OFFLOAD_BUNDLE__", at + 24)


def metadata(elf):
    """The code object's AMDGPU metadata note (type 32, MessagePack)."""
    shoff, = struct.unpack_from("<Q", elf, 0x28)
    shentsize, shnum = struct.unpack_from("<HH", elf, 0x3a)
    for i in range(shnum):
        _, kind, _, _, off, size = struct.unpack_from("<IIQQQQ", elf, shoff + i * shentsize)
        if kind != 7:   # SHT_NOTE
            continue
        namesz, descsz, ntype = struct.unpack_from("<III", elf, off)
        desc = off + 12 + (namesz + 3) // 4 * 4
        if ntype == 32:
            return msgpack.unpackb(elf[desc:desc + descsz], raw=False)
    return {}


@pytest.fixture(scope="module")
def kernels():
    if not os.path.exists(LIB):
        pytest.skip("library not built")
    with open(LIB, "rb") as f:
        data = f.read()
    return {k[".name"]: k for elf in code_objects(data) for k in metadata(elf).get("amdhsa.kernels", [])}


def waves(vgprs):
    return min(8, 512 // ((vgprs + 7) // 8 * 8))


# the count pass of the 256-slot class with 32 lanes per row: 6 waves per SIMD
# for one product, 5 for batches; of the 64-slot class in batches, 5; and
# nothing in scratch memory
@pytest.mark.parametrize("lanes,slots,multi,resident", [(32, 256, 0, 6), (32, 256, 1, 5), (8, 64, 1, 5)])
def test_count_kernel(kernels, lanes, slots, multi, resident):
    k = kernels[f"_ZN3mls9k_sym_ldsILi{lanes}ELi{slots}ELb0ELb{multi}ELi4EEEvNS_5BatchENS_5SchedEi"]
    assert waves(k[".vgpr_count"]) >= resident and k[".vgpr_spill_count"] == 0


# and no batch takes one that leaves fewer
def test_count_kernels_of_batches(kernels):
    ks = [k for n, k in kernels.items() if n.startswith("_ZN3mls9k_sym_ldsILi8ELi64ELb0ELb1E")]
    assert ks and all(waves(k[".vgpr_count"]) >= 5 for k in ks)
