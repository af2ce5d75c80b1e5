"""What the matrix-core coarse filter tells its refinement of a vector, a scale and a band, computed on the CPU in the
float arithmetic of the kernels that prepare centroids and vectors: scales clamped, norms of what the halves leave out,
the limits below and above which the band says nothing.  Where the band is finite it holds twice the error of every
score, so the exact best is within it of the smallest score; where it is not, every score is a finite number and every
centroid is a candidate.  test_coarse_half_bound.py checks the bound itself; nothing here touches the HIP library."""
import numpy as np
import pytest

f32 = np.float32
INF = f32(np.inf)


def half_scale(top):
    if not (top > 0) or not (top < INF):
        return f32(1)
    e = int((np.asarray(top, f32).view(np.uint32) >> 23) & 255) - 127
    return f32(2.0 ** min(100, max(-114, 13 - e)))


def halves(x):
    h = np.where(np.abs(x) < 2.0 ** -14, f32(0), x).astype(np.float16).astype(f32)
    return h, (x - h).astype(f32)


def norm(x):
    return np.sqrt(np.sum(x * x, axis=-1, dtype=f32))


def prepared_centroids(C, metric):
    with np.errstate(all="ignore"):
        mu = C.astype(np.float64).mean(axis=0).astype(f32)
        mu = np.where(np.isfinite(mu), mu, f32(0))
        x = (C - mu).astype(f32)
        bad = not (np.abs(x) < 1e17).all() or not (np.abs(mu) < 1e17).all()
        scale = half_scale(np.fmax.reduce(np.abs(x), axis=None))
        x64 = x.astype(np.float64)
        b = (x64 * x64).sum(1) if metric == "l2" else -(x64 @ mu.astype(np.float64))
        xs = np.zeros_like(x) if bad else (x * scale).astype(f32)
        b = np.zeros(len(C), f32) if bad else b.astype(f32)
        h, r = halves(xs)
    return {"mu": mu, "bad": bad, "scale": scale, "half": h, "bias": b, "n": norm(xs).max(), "r": norm(r).max(),
            "b": np.abs(b).max(), "mean": f32(np.sqrt((mu.astype(np.float64) ** 2).sum()))}


def scores(y, c, metric):
    """(scores, band) of one vector."""
    d = len(y)
    with np.errstate(all="ignore"):
        x = (y - c["mu"]).astype(f32)
        top = np.fmax.reduce(np.abs(x))
        scale = half_scale(top)
        bad = not (top < INF)
        xs = np.where(bad & (x == x), f32(0), (x * scale).astype(f32))
        h, r = halves(xs)
        g, iy, ic = f32(2 if metric == "l2" else 1), f32(1) / scale, f32(1) / c["scale"]
        ny, ry, nc, rc = norm(xs), norm(r), c["n"], c["r"]
        s = f32(f32(g * iy) * ic)
        e = s * (ry * nc + (ny + ry) * rc + f32(d) * f32(1.1920929e-7) * (ny + ry) * (nc + rc))
        uy, uc = ny * iy, nc * ic
        m = (uy + uc) * (uy + uc) if metric == "l2" else uc * (c["mean"] + f32(2) * uy)
        band = f32(2) * (f32(1.01) * e + f32(2.3841858e-7) * f32(1.01) * (c["b"] + s * ny * nc + m)) * f32(1.01)
        if bad or c["bad"] or not (band > 1e-34) or not (band < 1e37) or not (s >= f32(1.17549435e-38)):
            band, s = INF, f32(0)
        acc = np.zeros(len(c["half"]), f32)
        for j in range(d):
            acc = (acc + c["half"][:, j] * h[j]).astype(f32)
        return (c["bias"].astype(np.float64) - float(s) * acc.astype(np.float64)).astype(f32), f32(band)


def case(kind, d):
    rng = np.random.default_rng(d * 7 + len(kind))
    C = rng.standard_normal((64, d))
    Y = C[rng.integers(0, 64, 6)] + 0.05 * rng.standard_normal((6, d))
    if kind == "offset":
        C, Y = C + 100.0, Y + 100.0
    elif kind == "mixed-scales":
        f = 10.0 ** rng.integers(-3, 4, size=d)
        C, Y = C * f, Y * f
    elif kind == "all-positive":
        C, Y = np.abs(C) + 0.5, np.abs(Y) + 0.5
    elif kind == "bytes":
        C, Y = np.clip(np.rint(90 + 40 * C), 0, 255), np.clip(np.rint(90 + 40 * Y), 0, 255)
    elif kind == "one-far":
        C[7] *= 1e5
    elif kind in ("1e-13", "1e-20", "1e16", "1e30"):
        C, Y = C * float(kind), Y * float(kind)
    elif kind == "far-vectors":
        C, Y = C * 1e16, Y * 1e22
    elif kind == "outlier":
        C[5, d // 2] = 1e27
    elif kind == "nan-centroid":
        C[5, d // 2] = np.nan
    elif kind == "opposite":
        C[5, d // 2], C[6, d // 2] = np.inf, -np.inf
    elif kind == "infinite-vector":
        Y[1, 0] = np.inf
    return C.astype(f32), Y.astype(f32)


@pytest.mark.parametrize("metric", ["l2", "ip"])
@pytest.mark.parametrize("d", [4, 36, 128, 260])
@pytest.mark.parametrize("kind", ["gauss", "offset", "mixed-scales", "all-positive", "bytes", "one-far", "1e-13", "1e16"])
def test_the_band_holds_twice_the_error(metric, d, kind):
    C, Y = case(kind, d)
    c = prepared_centroids(C, metric)
    C64 = C.astype(np.float64)
    for y in Y:
        approx, band = scores(y, c, metric)
        assert band < INF, "the filter should tell these apart"
        y64 = y.astype(np.float64)
        exact = ((C64 - y64) ** 2).sum(1) if metric == "l2" else -(C64 @ y64)
        diff = approx.astype(np.float64) - exact
        assert diff.max() - diff.min() <= band, f"{kind} d={d} {metric}"
        assert approx[np.argmin(exact)] <= f32(approx.min() + band)


@pytest.mark.parametrize("metric", ["l2", "ip"])
@pytest.mark.parametrize("d", [4, 128])
@pytest.mark.parametrize("kind", ["1e-20", "1e30", "far-vectors", "outlier", "nan-centroid", "opposite", "infinite-vector"])
def test_where_the_band_says_nothing_every_centroid_is_a_candidate(metric, d, kind):
    C, Y = case(kind, d)
    c = prepared_centroids(C, metric)
    seen = 0
    for y in Y:
        approx, band = scores(y, c, metric)
        if band < INF:
            continue
        seen += 1
        limit = f32(approx.min() + band)
        assert np.isfinite(approx).all() and (approx <= limit).all()
    assert seen >= (1 if kind == "infinite-vector" else len(Y))
