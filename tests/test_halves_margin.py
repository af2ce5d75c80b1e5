"""The margins of the scan of halves, emulated on the CPU with additions that cut instead of rounding: squared distances from
halves and the direct form lie within halves_reach of each other whichever is taken for the limit; the least an inner product's
negative can be from halves is no more than the direct one; and the bound from a sample of halves is no less than the direct
score of what it was taken from.  Nothing here touches the HIP library."""
import numpy as np
import pytest

F = np.float32
U = 4.888e-4


def cut_add(a, b):
    """a + b in 32 bits, cut towards zero: the worst an adder without rounding does."""
    s = float(a) + float(b)
    r = F(s)
    return np.nextafter(r, F(0)) if abs(float(r)) > abs(s) else r


def halves(v, scale):
    w = (v * scale).astype(F)
    w = np.where(np.abs(w) < 6.1035156e-5, F(0), w)
    return w.astype(np.float16).astype(F)


def piece_scale(qn):
    if not (0 < qn < np.inf):
        return F(1)
    e = int((F(qn).view(np.uint32) >> 23) & 255) - 127
    return F(2.0 ** max(-100, min(100, 14 - ((e + 2) >> 1))))


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


def direct(x, q, metric):
    acc = F(0)
    for a, b in zip(x, q):
        acc = F(float(acc) + float(F(a - b)) ** 2) if metric == "l2" else F(float(acc) + float(a) * float(b))
    return acc


def reach(v, d, norm, e, u):
    slack = F((2 * (128 + d // 64 + 1) + 16 * ((d + 31) // 32) + 8) * 6.0e-8)
    r0 = np.sqrt(F(max(v, 0)))
    p = F(1.01) * (norm + r0) + e
    fp = slack * p * p
    r = np.sqrt(r0 * r0 * F(1 + (d + 8) * 6.0e-8) + fp) * F(1.000001)
    r += u * (norm + r) + e
    return F((r * r + fp) * 1.000001 + 1e-30)


@pytest.mark.parametrize("d", [4, 32, 100, 256, 768])
@pytest.mark.parametrize("kind", ["near", "far", "offset", "tiny", "mixed", "whole"])
def test_scores_from_halves_stay_within_their_margins(d, kind):
    rng = np.random.default_rng(7 * d + len(kind))
    for _ in range(6 if d > 200 else 20):
        x = {"near": rng.standard_normal(d), "far": 300 * rng.standard_normal(d), "offset": 200 + rng.standard_normal(d),
             "tiny": 1e-7 * rng.standard_normal(d), "mixed": rng.standard_normal(d) * 10.0 ** rng.uniform(-7, 1, d),
             "whole": np.rint(100 * rng.standard_normal(d))}[kind].astype(F)
        q = (x + {"far": 300, "tiny": 1e-8, "whole": 3}.get(kind, 0.01) * rng.standard_normal(d)).astype(F)
        if kind == "whole":
            q = np.rint(q).astype(F)
        top = {"far": 1500.0, "offset": 204.0, "whole": 400.0, "mixed": 20.0}.get(kind, 4.0)
        xs = F(2.0 ** (8 - int(np.floor(np.log2(top)))))  # the scale of an index whose centroids' largest coordinate is `top`
        exact = kind == "whole"
        xh, qs = halves(x, xs), piece_scale(F(np.sum(q.astype(np.float64) ** 2)))
        qh = halves(q, qs)
        if exact:
            assert np.array_equal(xh / xs, x)
        qt, xt = qh.astype(np.float64) / float(qs), xh.astype(np.float64) / float(xs)
        q64 = q.astype(np.float64)
        norm = F(max(np.linalg.norm(q64), np.linalg.norm(qt)) * 1.00001)
        s = F(np.linalg.norm(q64 - qt) * 1.00001)
        t = F(0 if exact else 6.11e-5 * np.sqrt(d) / float(xs))
        u = F(0 if exact else U)
        dot, square = scan_sums(xh, qh)
        unscale = F(1 / (float(qs) * float(xs)))
        # squared distances
        a = F(float(F(-2 * unscale)) * float(dot) + float(F(F(np.sum(qt ** 2)) + F(float(square) / float(xs) ** 2))))
        v = direct(x, q, "l2")
        assert a <= reach(v, d, norm, s + t, u) and v <= reach(a, d, norm, s + t, u), (kind, d, float(a), float(v))
        # ... and the bound from a sample: of the query against what the halves hold
        r = np.sqrt(direct(xt.astype(F), q, "l2")) * F(1 + (d + 8) * 6.0e-8)
        r += u * (norm + r) + s + t
        assert v <= F(r * r * 1.000001)
        # inner products
        nx = np.sqrt(square) / xs
        fp = F((d + d // 64 + 140) * 6.0e-8)
        least = F(float(-unscale) * float(dot) - float(F(1.002) * (s + norm * (u + fp)) * nx))
        e = F(1.002) * t * norm + F(1e-30)
        w = -direct(x, q, "ip")
        assert least <= w + e + (abs(w) + e) * F(2.4e-7), (kind, d, float(least), float(w))
        over = norm * ((F(0) if exact else F(4.9e-4)) + F((2 * d + 8) * 6.0e-8))
        assert w <= F(over * nx - direct(xt.astype(F), q, "ip")) + e
