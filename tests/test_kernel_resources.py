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


# Kernels whose comments count on so many workgroups to a compute unit: four SIMDs of 512 registers (taken by the lane, in
# eights) and 160 KiB of LDS.  Name, kernels of that name, wavefronts of a workgroup, workgroups, dynamic LDS of a workgroup.
# The scan: four wavefronts to a SIMD in short scans but of inner products of floats, three elsewhere (LDS by the tile).
@pytest.mark.parametrize("name,count,waves,groups,lds", [
    ("8k_select", 3, 8, 2, 0),
    ("15k_select_halves", 3, 8, 2, 0),
    ("7k_group", 1, 8, 2, 0),
    ("13k_plan_halves", 1, 8, 2, 0),
    ("13k_scan_halves", 4, 4, 6, 26368),            # steps, staging, and 16 queries of 96 dimensions
    ("13k_scan_halves", 4, 4, 4, 40320),            # 32 of 256
    ("9k_pq_scan", 1, 8, 4, 16 * 1024),             # 16 codes to a vector
    ("10k_pq_bound", 1, 16, 1, 64 * 1024),          # 64
    ("13k_coarse_mfmaILi4", 2, 4, 2, 3 * 384 * 64),
    ("13k_coarse_mfmaILi2", 2, 4, 2, 3 * 256 * 64),
    ("15k_assign_refine", 1, 4, 4, 0),
    ("9k_scan_mmILi0ELb0ELi0ELb0", 1, 4, 4, 0),
    ("9k_scan_mmILi0ELb0ELi1ELb0", 1, 4, 4, 0),
    ("9k_scan_mmILi0ELb0ELi2ELb0", 1, 4, 4, 0),
    ("9k_scan_mmILi1ELb0ELi1ELb0", 1, 4, 4, 0),
    ("9k_scan_mmILi1ELb0ELi2ELb0", 1, 4, 4, 0),
    ("9k_scan_mmILi", 16, 4, 3, 0),
])
def test_as_many_workgroups_to_a_compute_unit_as_the_comments_say(records, name, count, waves, groups, lds):
    mine = {n: k for n, k in records.items() if name in n}
    assert len(mine) == count
    for n, k in mine.items():
        wavefronts_to_a_simd = (waves * groups + 3) // 4
        assert (k[".vgpr_count"] + 7) // 8 * 8 * wavefronts_to_a_simd <= 512, n
        assert groups * (k[".group_segment_fixed_size"] + lds) <= 160 * 1024, n
