"""The error bound the matrix-core coarse filter relies on, checked on the CPU against an emulation of what the
matrix instruction is fed: vectors and centroids less the mean of the centroids, scaled by a power of two, as
halves (nearest even, subnormal halves dropped), products added in fp32.  The GPU path decides nothing from these
scores; it only assumes that up to a term common to all centroids they are within E of the exact ones, with
E = g (r_y n_c + (n_y + r_y) r_c + d 2^-23 (n_y + r_y) (n_c + r_c)) + 2^-22 (max |b| + g n_y n_c + m)."""
import numpy as np
import pytest


def scale_of(top):
    return np.float32(1.0) if not (0 < top < np.inf) else np.float32(2.0 ** (13 - np.floor(np.log2(float(top)))))


def halves(x, scale):
    x = (x * scale).astype(np.float32)
    x = np.where(np.abs(x) < 2.0 ** -14, np.float32(0), x)
    return x.astype(np.float16).astype(np.float32)


def filter_scores(y, C, metric, order):
    """(approximate scores, bound) of one vector against all centroids."""
    d, g = C.shape[1], (2.0 if metric == "l2" else 1.0)
    mu = C.astype(np.float64).mean(axis=0).astype(np.float32)
    Cc, yc = (C - mu).astype(np.float32), (y - mu).astype(np.float32)
    b = ((Cc.astype(np.float64) ** 2).sum(1) if metric == "l2" else -(Cc.astype(np.float64) @ mu.astype(np.float64)))
    b = b.astype(np.float32)
    sc, sy = scale_of(np.abs(Cc).max()), scale_of(np.abs(yc).max())
    Ch, yh = halves(Cc, sc), halves(yc, sy)
    acc = np.zeros(len(C), np.float32)
    for j in order:
        acc = (acc + Ch[:, j] * yh[j]).astype(np.float32)  # the product of two halves is exact
    s = np.float32(g / (float(sc) * float(sy)))
    approx = (b.astype(np.float64) - float(s) * acc).astype(np.float32)  # one fused multiply-add
    nrm = lambda v: float(np.sqrt((v.astype(np.float64) ** 2).sum(-1)).max())
    ny, ry = nrm(yc), nrm(yc.astype(np.float64) - yh / float(sy))
    nc, rc = nrm(Cc), nrm(Cc.astype(np.float64) - Ch / float(sc))
    m = (ny + nc) ** 2 if metric == "l2" else nc * (nrm(mu) + 2 * ny)
    E = g * (ry * nc + (ny + ry) * rc + d * 2.0 ** -23 * (ny + ry) * (nc + rc))
    return approx, E + 2.0 ** -22 * (np.abs(b).max() + g * ny * nc + m)


@pytest.mark.parametrize("metric", ["l2", "ip"])
@pytest.mark.parametrize("d", [4, 36, 128, 260])
@pytest.mark.parametrize("kind", ["gauss", "offset", "mixed-scales", "bytes", "tiny", "one-far"])
def test_half_contraction_stays_inside_the_band(metric, d, kind):
    rng = np.random.default_rng(d * 11 + len(kind))
    C = rng.standard_normal((64, d))
    y = C[3] + 0.01 * rng.standard_normal(d)
    if kind == "offset":
        C, y = C + 1000.0, y + 1000.0
    elif kind == "mixed-scales":
        f = 10.0 ** rng.uniform(-6, 3, d)
        C, y = C * f, y * f
    elif kind == "bytes":
        C, y = np.clip(np.rint(60 + 30 * C), 0, 255), np.clip(np.rint(60 + 30 * y), 0, 255)
    elif kind == "tiny":
        C, y = C * 1e-9, y * 1e-9
    elif kind == "one-far":
        C[7] *= 1e5
    C, y = C.astype(np.float32), y.astype(np.float32)
    y64, C64 = y.astype(np.float64), C.astype(np.float64)
    exact = ((C64 - y64) ** 2).sum(1) if metric == "l2" else -(C64 @ y64)
    for order in (np.arange(d), np.arange(d)[::-1], rng.permutation(d)):
        approx, E = filter_scores(y, C, metric, order)
        diff = approx.astype(np.float64) - exact
        # up to a term common to all centroids: the spread of the differences is at most 2 E
        assert diff.max() - diff.min() <= 2 * E
        # what the filter concludes from it: the exact best is among the candidates
        assert approx[np.argmin(exact)] <= approx.min() + 2 * E
