"""The items of a scan of halves: the word the plan writes says how far an item goes, so that the scan need not ask how long a list
is by then.  The functions are those the kernels use, compiled for the host."""
import ctypes
import os
import subprocess

import pytest

from paper_2408_02937_amd import build

SHIM = """
#define __host__
#define __device__
#include "halves.h"
extern "C" {
uint32_t word(uint32_t pairs, uint32_t len, uint32_t segment, uint32_t seg) { return rtams::half_item_word(pairs, len, segment, seg); }
uint32_t pairs(uint32_t word) { return rtams::half_item_pairs(word); }
uint32_t units(uint32_t word) { return rtams::half_item_units(word); }
}
"""


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    at = tmp_path_factory.mktemp("items")
    (at / "shim.cpp").write_text(SHIM)
    subprocess.run(["g++", "-std=c++17", "-O1", "-shared", "-fPIC", "-I", build.CSRC, str(at / "shim.cpp"), "-o", str(at / "shim.so")], check=True)
    L = ctypes.CDLL(os.fspath(at / "shim.so"))
    for f in (L.word, L.pairs, L.units):
        f.restype, f.argtypes = ctypes.c_uint32, [ctypes.c_uint32] * (4 if f is L.word else 1)
    return L


# the plan's segments are a power of two of groups of 64 vectors, 2^16 at most; lengths of 0, 1, and around units, groups and segments
@pytest.mark.parametrize("seg", [2, 4, 64, 256, 1 << 16])
def test_the_units_of_a_lists_items_are_those_of_its_planned_length(lib, seg):
    per = 64 * seg
    lengths = {0, 1, 31, 32, 33, 63, 64, 65, per - 1, per, per + 1, 5 * per + 40, 2**31, 2**32 - 1}
    for n in lengths:
        segments = max(1, -(-n // per))
        for sg in range(segments) if segments < 2000 else (0, 1, segments // 2, segments - 2, segments - 1):
            for p in (1, 16, 31, 32):
                w = lib.word(p, n, sg, seg)
                begin, end = sg * per, min((sg + 1) * per, n)
                assert lib.pairs(w) == p and w != 0
                assert lib.units(w) == -(-max(end - begin, 0) // 32), (n, sg)
