"""The matrix-core filter where it can say nothing: centroids that are infinite, not a number or far outside the range
of the others, vectors that are, and products that overflow.  What it decides has to be what the exact kernel decides
(and the oracle, where the exact scores are numbers): such rows are scored against every centroid, none is dropped."""
import numpy as np
import pytest
import torch

from paper_2408_02937_amd import synth
from tests.gpu_common import dev, make_pair

pytestmark = pytest.mark.gpu


def case(kind, nlist, d, rows):
    rng = np.random.default_rng(nlist + len(kind))
    C = rng.standard_normal((nlist, d)).astype(np.float32)
    if kind == "overflow":  # every centroid below what counts as too large, every vector finite: the products are not
        C *= np.float32(1.5e16)
    y = C[rng.integers(0, nlist, rows)] + (0.05 * rng.standard_normal((rows, d))).astype(np.float32)
    if kind == "outlier":
        C[17, 5] = 1e27
    elif kind == "nan-centroid":
        C[17, 5] = np.nan
    elif kind == "infinite":
        C[17, 5] = np.inf
    elif kind == "opposite":
        C[17, 5], C[nlist // 2, 5] = np.inf, -np.inf
    elif kind == "overflow":
        y[::3] = (1e22 * rng.standard_normal((len(y[::3]), d))).astype(np.float32)
        y[1] = (1e30 * rng.standard_normal(d)).astype(np.float32)
    elif kind == "far-vectors":
        y[::3] *= np.float32(1e35)
        y[1, 2], y[4, 2] = np.inf, -np.inf
    return C, y.astype(np.float32)


# lists: up to what the probe selection scores from its candidates, and more; tiles of 128 and 256 centroids
@pytest.mark.parametrize("metric", ["l2", "ip"])
@pytest.mark.parametrize("kind,nlist,d,rows", [
    (kind, *shape) for kind in ("outlier", "nan-centroid", "infinite", "opposite", "overflow", "far-vectors")
    for shape in ((10, 4, 40), (700, 36, 333), (1500, 68, 40_000))
    if shape[0] > 20 or kind in ("overflow", "far-vectors")])  # the odd centroid is number 17
def test_the_filter_decides_as_the_exact_kernel(kind, metric, nlist, d, rows):
    print(f"[case] filter {kind} {metric} {nlist} x {d}, {rows} rows", flush=True)
    C, y = case(kind, nlist, d, rows)
    w = synth.Workload("odd", metric, d, nlist, 64, 8, 10, np.zeros((0, d), np.float32), C,
                       np.zeros((0, d), np.float32), np.zeros((0, d), np.float32), 1, 0)
    g, o = make_pair(w, pool_blocks=64, candidates_per_query=1024)
    y[-1, 3] = np.nan  # a vector with a NaN beside them goes to the first list
    yd, q = dev(y), dev(y[:64])
    got, probed = {}, {}
    for mode in (2, 0):
        g.set_param("use_mfma", mode)
        got[mode] = g.assign(yd).cpu().numpy()
        probed[mode] = g.probe(q[:40], 8).cpu().numpy()
    assert np.array_equal(got[2], got[0])
    assert got[2][-1] == 0
    assert np.array_equal(probed[2], probed[0])
    some = np.flatnonzero(np.isfinite(y).all(axis=1))[:300]
    assert np.array_equal(got[2][some], o.assign(y[some]))
    torch.cuda.synchronize()
    g.close()


@pytest.mark.parametrize("metric", ["l2", "ip"])
def test_tiny_numbers_stay_in_the_filter(metric):
    """The same vectors and centroids times 2^-46 (norms of 1e-13): the same lists, and not an exact score for every
    centroid, which takes more than ten times as long."""
    rng = np.random.default_rng(46)
    d, nlist, rows = 64, 4096, 65_536
    C = rng.standard_normal((nlist, d)).astype(np.float32)
    y = (C[rng.integers(0, nlist, rows)] + 0.1 * rng.standard_normal((rows, d))).astype(np.float32)
    got, ms = [], []
    for f in (1.0, 2.0 ** -46):
        w = synth.Workload("tiny", metric, d, nlist, 64, 8, 10, np.zeros((0, d), np.float32), C * np.float32(f),
                           np.zeros((0, d), np.float32), np.zeros((0, d), np.float32), 1, 0)
        g, _ = make_pair(w, pool_blocks=64, candidates_per_query=1024)
        yd = dev(y * np.float32(f))
        for _ in range(3):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            out = g.assign(yd)
            b.record()
            torch.cuda.synchronize()
            t = a.elapsed_time(b)
        got.append(out.cpu().numpy()); ms.append(t)
        g.close()
    print(f"[case] tiny {metric}: {ms} ms", flush=True)
    assert np.array_equal(got[0], got[1])
    assert ms[1] < 3 * ms[0]
