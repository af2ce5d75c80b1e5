"""What the compiler gave the kernels of the built library, read from the code objects inside it: no kernel keeps
private memory, and the kernels whose comments count on a number of wavefronts per SIMD have the registers for it."""
import os
import struct

import msgpack
import pytest

from paper_2408_02937_amd import build

MAGIC = b"__CLANG_OFFLOAD_BUNDLE__"


def code_objects(blob):
    """The gfx950 ELF images of every offload bundle in the library."""
    at = blob.find(MAGIC)
    while at >= 0:
        (count,) = struct.unpack_from("<Q", blob, at + len(MAGIC))
        p = at + len(MAGIC) + 8
        for _ in range(count):
            off, size, n = struct.unpack_from("<QQQ", blob, p)
            name = blob[p + 24:p + 24 + n]
            p += 24 + n
            if b"gfx950" in name and size:
                yield blob[at + off:at + off + size]
        at = blob.find(MAGIC, at + 1)


def kernels(elf):
    """The kernel records of the metadata note of one ELF image."""
    shoff, = struct.unpack_from("<Q", elf, 0x28)
    entsize, num = struct.unpack_from("<HH", elf, 0x3A)
    for i in range(num):
        _, kind = struct.unpack_from("<II", elf, shoff + i * entsize)
        if kind != 7:  # SHT_NOTE
            continue
        p, size = struct.unpack_from("<QQ", elf, shoff + i * entsize + 0x18)
        end = p + size
        while p + 12 <= end:
            nsz, dsz, ntype = struct.unpack_from("<III", elf, p)
            desc = p + 12 + (nsz + 3) // 4 * 4
            if ntype == 32 and elf[p + 12:p + 18] == b"AMDGPU":
                yield from msgpack.unpackb(elf[desc:desc + dsz]).get("amdhsa.kernels", [])
            p = desc + (dsz + 3) // 4 * 4


@pytest.fixture(scope="module")
def records():
    if not os.path.exists(build.LIB):
        build.build()
    with open(build.LIB, "rb") as f:
        blob = f.read()
    out = {k[".name"]: k for e in code_objects(blob) for k in kernels(e)}
    assert len(out) > 40, "the code objects of the library could not be read"
    return out


def test_no_kernel_keeps_private_memory(records):
    assert {n: k[".private_segment_fixed_size"] for n, k in records.items() if k[".private_segment_fixed_size"]} == {}


def test_the_selection_runs_two_workgroups_to_a_compute_unit(records):
    mine = {n: k for n, k in records.items() if "k_select" in n}
    assert len(mine) == 3
    for n, k in mine.items():
        # 8 wavefronts of 512 threads, two workgroups on 4 SIMDs: four wavefronts a SIMD, of 512 registers
        assert k[".vgpr_count"] <= 128, n
        assert 2 * k[".group_segment_fixed_size"] <= 160 * 1024, n
