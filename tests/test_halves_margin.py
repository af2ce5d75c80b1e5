"""The margins of the scan of halves, the kernels' own functions compiled for the host, against scores emulated with additions
that cut instead of rounding: squared distances from halves and the direct form lie within halves_reach of each other whichever is
taken for the limit; the least an inner product's negative can be from halves is no more than the direct one; and the bound from
a sample of halves is no less than the direct score of what it was taken from."""
import ctypes
import os
import subprocess

import numpy as np
import pytest

from paper_2408_02937_amd import build

F = np.float32
SHIM = """
#define __host__
#define __device__
#include "halves.h"
using namespace rtams;
extern "C" {
float scale(double nsq) { return half_query_scale(nsq); }
void query(float inv, float qsq, float norm, float left, int d, int metric, float ixs, HalfQuery *m) { *m = half_query_of(inv, qsq, norm, left, d, metric, ixs); }
float reach(float v, int d, const HalfQuery *m) { return halves_reach(v, d, *m); }
float reach_ip(float v, const HalfQuery *m) { return halves_reach_ip(v, *m); }
float sampled(float v, int d, const HalfQuery *m) { return halves_sampled(v, d, *m); }
float over(float norm, int exact, int d) { return halves_over(norm, exact != 0, d); }
}
"""


class HalfQuery(ctypes.Structure):
    _fields_ = [(n, ctypes.c_float) for n in ("unscale", "a", "norm", "e", "u")]


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    at = tmp_path_factory.mktemp("margins")
    (at / "shim.cpp").write_text(SHIM)
    subprocess.run(["g++", "-std=c++17", "-O1", "-shared", "-fPIC", "-I", build.CSRC, str(at / "shim.cpp"), "-o", str(at / "shim.so")], check=True)
    L = ctypes.CDLL(os.fspath(at / "shim.so"))
    f, i, q = ctypes.c_float, ctypes.c_int, ctypes.POINTER(HalfQuery)
    for fn, res, args in ((L.scale, f, [ctypes.c_double]), (L.query, None, [f, f, f, f, i, i, f, q]), (L.reach, f, [f, i, q]),
                          (L.reach_ip, f, [f, q]), (L.sampled, f, [f, i, q]), (L.over, f, [f, i, i])):
        fn.restype, fn.argtypes = res, args
    return L


def cut_add(a, b):
    """a + b in 32 bits, cut towards zero: the worst an adder without rounding does."""
    s = float(a) + float(b)
    r = F(s)
    return np.nextafter(r, F(0)) if abs(float(r)) > abs(s) else r


def halves(v, scale):
    w = (v * scale).astype(F)
    w = np.where(np.abs(w) < 6.1035156e-5, F(0), w)
    return w.astype(np.float16).astype(F)


def scan_sums(xh, qh):
    """The sum of products in pieces of 64 coordinates, and the vector's square in lanes' sums of a quarter each."""
    total = F(0)
    for lo in range(0, len(xh), 64):
        acc = F(0)
        for a, b in zip(xh[lo:lo + 64], qh[lo:lo + 64]):
            acc = cut_add(acc, float(a) * float(b))
        total = F(total + acc)
    parts = []
    for lane in range(4):
        acc = F(0)
        for j in range(len(xh)):
            if j // 8 % 4 == lane:
                acc = cut_add(acc, float(xh[j]) ** 2)
        parts.append(acc)
    return total, F(F(parts[0] + parts[1]) + F(parts[2] + parts[3]))


def sample_score(x, q, metric):
    """A sample's score: four lanes, a chunk of eight coordinates to each in turn."""
    parts = []
    for lane in range(4):
        acc = F(0)
        for j in range(len(x)):
            if j // 8 % 4 == lane:
                acc = cut_add(acc, float(F(x[j] - q[j])) ** 2 if metric == "l2" else float(x[j]) * float(q[j]))
        parts.append(acc)
    return F(F(parts[0] + parts[1]) + F(parts[2] + parts[3]))


def direct(x, q, metric):
    acc = F(0)
    for a, b in zip(x, q):
        acc = F(float(acc) + float(F(a - b)) ** 2) if metric == "l2" else F(float(acc) + float(a) * float(b))
    return acc


@pytest.mark.parametrize("d", [4, 32, 100, 256, 768])
@pytest.mark.parametrize("kind", ["near", "far", "offset", "tiny", "mixed", "whole", "whole offset", "whole beside fractions"])
def test_scores_from_halves_stay_within_their_margins(d, kind, lib):
    rng = np.random.default_rng(7 * d + len(kind))
    for _ in range(6 if d > 200 else 20):
        x = {"near": rng.standard_normal(d), "far": 300 * rng.standard_normal(d), "offset": 200 + rng.standard_normal(d),
             "tiny": 1e-7 * rng.standard_normal(d), "mixed": rng.standard_normal(d) * 10.0 ** rng.uniform(-7, 1, d),
             "whole": np.rint(100 * rng.standard_normal(d)),
             # (sums past 2^24; the second's queries are no halves, and far enough for that to weigh more than the sums)
             "whole offset": np.rint(900 + 20 * rng.standard_normal(d)), "whole beside fractions": np.rint(900 + 20 * rng.standard_normal(d))}[kind].astype(F)
        q = (x + {"far": 300, "tiny": 1e-8, "whole": 3, "whole offset": 1, "whole beside fractions": 700}.get(kind, 0.01) * rng.standard_normal(d)).astype(F)
        exact = kind.startswith("whole")  # of the vectors
        if kind in ("whole", "whole offset"):
            q = np.rint(q).astype(F)
        top = {"far": 1500.0, "offset": 204.0, "whole": 400.0, "whole offset": 1000.0, "whole beside fractions": 1000.0, "mixed": 20.0}.get(kind, 4.0)
        xs = F(2.0 ** (8 - int(np.floor(np.log2(top)))))  # the scale of an index whose centroids' largest coordinate is `top`
        xh, qs = halves(x, xs), F(lib.scale(float(np.sum(q.astype(np.float64) ** 2))))
        qh = halves(q, qs)
        if exact:
            assert np.array_equal(xh / xs, x)
        qt, xt = qh.astype(np.float64) / float(qs), xh.astype(np.float64) / float(xs)
        q64 = q.astype(np.float64)
        norm = F(max(np.linalg.norm(q64), np.linalg.norm(qt)) * 1.00001)
        left = F(np.linalg.norm(q64 - qt) * 1.00001)
        inv = F(1) / qs
        m, mi = HalfQuery(), HalfQuery()
        lib.query(-inv if exact else inv, np.sum(qt ** 2), norm, left, d, 0, 1 / xs, m)
        lib.query(-inv if exact else inv, np.sum(qt ** 2), norm, left, d, 1, 1 / xs, mi)
        dot, square = scan_sums(xh, qh)
        # squared distances, as the scan makes them of the sums
        a = F(float(F(-2 * m.unscale)) * float(dot) + float(F(F(m.a) + F(float(square) / float(xs) ** 2))))
        v = direct(x, q, "l2")
        assert a <= lib.reach(v, d, m) and v <= lib.reach(a, d, m), (kind, d, float(a), float(v))
        # ... and the bound from a sample: of the query against what the halves hold
        assert v <= lib.sampled(sample_score(xt.astype(F), q, "l2"), d, m)
        # inner products
        nx = np.sqrt(square) / xs
        least = F(float(F(-mi.unscale)) * float(dot) - float(F(mi.a) * nx))
        w = -direct(x, q, "ip")
        assert least <= lib.reach_ip(w, mi), (kind, d, float(least), float(w))
        assert w <= F(F(lib.over(norm, exact, d)) * nx - sample_score(xt.astype(F), q, "ip")) + F(mi.e)
