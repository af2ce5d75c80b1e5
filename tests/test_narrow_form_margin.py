"""The margin of the scan of halves and bytes on 16-bit matrix instructions: the query in three pieces of the operand's
type, their exact products with the stored coordinates added up in 32 bits (the first piece's for themselves), and the
norm form around the sum.  |norm form - direct form| <= slack (2 v + 3 |q|^2) with slack = 1.01 (4 d + 8) 2^-24, as for the
scan in floats, for v either of the two values.  Checked on the CPU against emulations whose additions cut instead of rounding, in several orders; and the pieces add up to
the query to the last bit (bytes) or to 2^-33 of its length (halves).  Nothing here touches the HIP library."""
import numpy as np
import pytest

F = np.float32


def cut_add(a, b):
    """a + b in 32 bits, cut towards zero: the worst an adder without rounding does."""
    s = float(a) + float(b)
    r = F(s)
    return np.nextafter(r, F(0)) if abs(float(r)) > abs(s) else r


def piece_scale(qn):
    if not (0 < qn < np.inf):
        return F(1)
    e = int((F(qn).view(np.uint32) >> 23) & 255) - 127
    return F(2.0 ** max(-100, min(100, 14 - ((e + 2) >> 1))))


def pieces(q, storage, qn):
    scale = piece_scale(qn) if storage == "f16" else F(1)
    w, out = (q * scale).astype(F), []
    for _ in range(3):
        if storage == "f16":
            h = w.astype(np.float16).astype(F)
        else:
            h = (w.view(np.uint32) & np.uint32(0xffff0000)).view(F)
        out.append(h)
        w = (w - h).astype(F)
    return out, scale


def direct_form(x, q):
    acc = F(0)
    for a, b in zip(x, q):
        t = F(a - b)
        acc = F(acc + F(t * t))
    return acc


def norm_form(x, q, storage, order):
    qn = F(np.sum(q.astype(np.float64) ** 2))
    ps, scale = pieces(q, storage, qn)
    acc, low, xn = F(0), F(0), F(0)
    for j in order:
        acc = cut_add(acc, float(x[j]) * float(ps[0][j]))
        for p in ps[1:]:
            low = cut_add(low, float(x[j]) * float(p[j]))
        xn = cut_add(xn, float(x[j]) ** 2)
    return F(F(F(-2) * F(F(1) / scale)) * F(acc + low) + F(xn + qn)), qn


@pytest.mark.parametrize("storage", ["f16", "u8"])
@pytest.mark.parametrize("d", [16, 128, 640])
@pytest.mark.parametrize("kind", ["near", "far", "offset", "tiny"])
def test_the_narrow_norm_form_stays_within_its_margin(storage, d, kind):
    rng = np.random.default_rng(31 * d + len(kind))
    slack = 1.01 * (4 * d + 8) * 2.0 ** -24
    for _ in range(6):
        if storage == "u8":
            x = rng.integers(0, 256, d).astype(F)
            q = {"near": x + 0.3 * rng.standard_normal(d), "far": 255 * rng.random(d), "offset": 1000 + x,
                 "tiny": 1e-6 * rng.standard_normal(d)}[kind].astype(F)
        else:
            x = {"near": rng.standard_normal(d), "far": 300 * rng.standard_normal(d), "offset": 50 + rng.standard_normal(d),
                 "tiny": 1e-6 * rng.standard_normal(d)}[kind].astype(np.float16).astype(F)  # (tiny: subnormal halves)
            q = (x + (0.01 if kind != "far" else 300) * rng.standard_normal(d)).astype(F)
        dv = float(direct_form(x, q))
        for order in (np.arange(d), rng.permutation(d)):
            nv, qn = (float(v) for v in norm_form(x, q, storage, order))
            for v in (dv, max(nv, 0.0)):
                assert abs(nv - dv) <= slack * (2 * v + 3 * qn), f"{storage} {kind} d={d}: {nv} against {dv}"


@pytest.mark.parametrize("size", [1e-30, 1e-6, 1.0, 255.0, 1e9, 1e18])
def test_the_pieces_hold_the_query(size):
    rng = np.random.default_rng(5)
    q = (size * rng.standard_normal(200) * 10.0 ** rng.uniform(-6, 0, 200)).astype(F)
    qn = F(np.sum(q.astype(np.float64) ** 2))
    for storage in ("f16", "u8"):
        ps, scale = pieces(q, storage, qn)
        assert all(np.all(np.isfinite(p)) for p in ps)
        back = np.sum([p.astype(np.float64) for p in ps], axis=0) / float(scale)
        if storage == "u8":
            # exact, down to what is no normal number any more: 2 x 640 x 255 x 2^-126 is under the margin's floor of 1e-30
            assert np.max(np.abs(back - q)) <= (0.0 if np.min(np.abs(q)) > 2.0 ** -100 else 2.0 ** -126)
        elif size > 1e-20:  # (below, the scale is capped and |q| far under the margin's own floor)
            assert np.max(np.abs(back - q)) <= 2.0 ** -33 * np.sqrt(float(qn))
