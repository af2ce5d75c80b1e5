"""Insertion of batches that go through one workgroup behind the coarse scores, and of those just too large for it:
lists bit for bit against the oracle, block structure, counters, allocator reports."""
import numpy as np
import pytest
import torch

from oracle.oracle import OracleIndex
from paper_2408_02937_amd import rtams, synth
from tests.gpu_common import assert_lists_equal, dev, make_pair

pytestmark = pytest.mark.gpu


# one vector; a wavefront and one more; the most one workgroup takes and one more; with d 68 about 960 vectors are the
# most it also moves
@pytest.mark.parametrize("batches", [[1, 1, 1], [63, 64, 65], [959, 964, 1023], [1024, 1025, 1], [3000, 7, 1024]])
@pytest.mark.parametrize("hot", [False, True])
@pytest.mark.parametrize("mfma,ordered", [(0, 0), (2, 0), (1, 1)])
def test_batches_around_the_limits(batches, hot, mfma, ordered):
    """`hot`: every vector falls into one list, which opens sixteen blocks and more (and table segments) at once."""
    rng = np.random.default_rng(sum(batches) + mfma)
    d, nlist = 68, 300
    C = rng.standard_normal((nlist, d)).astype(np.float32)
    print(f"[case] insert batches {batches} hot={hot} use_mfma={mfma} ordered={ordered}", flush=True)
    w = synth.Workload("tail", "l2", d, nlist, 64, 8, 10, np.zeros((0, d), np.float32), C,
                       np.zeros((0, d), np.float32), np.zeros((0, d), np.float32), 1, 0)
    g, o = make_pair(w, pool_blocks=2000, candidates_per_query=8192)
    g.set_param("use_mfma", mfma)
    g.set_param("ordered_add", ordered)
    bounds = []
    for m in batches:
        at = np.full(m, 5) if hot else rng.integers(0, nlist, m)
        y = (C[at] + 0.05 * rng.standard_normal((m, d))).astype(np.float32)
        bounds.append(o.ntotal)
        g.add(dev(y)); o.add(y)
    g.validate()
    assert_lists_equal(g, o, np.array(bounds[1:]))
    assert g.poll_error() == 0
    q = (C[:33] + 0.05 * rng.standard_normal((33, d))).astype(np.float32)
    dd, ii = g.search(dev(q), 10, 8)
    rd, ri = o.search(q, 10, 8)
    assert np.allclose(dd.cpu().numpy(), rd, rtol=1e-4, atol=1e-6)
    g.close()


@pytest.mark.parametrize("storage,pq_m", [("f16", 0), ("u8", 0), ("f32", 8)])
def test_small_batches_of_narrow_and_coded_lists(storage, pq_m):
    """The same vectors in one add of thousands and in batches of 50: the same lists."""
    rng = np.random.default_rng(3)
    d, nlist, n = 64, 40, 4000
    C = np.rint(rng.uniform(0, 255, (nlist, d))).astype(np.float32)
    y = np.clip(np.rint(C[rng.integers(0, nlist, n)] + 9 * rng.standard_normal((n, d))), 0, 255).astype(np.float32)
    held = []
    for step in (n, 50):
        g = rtams.Index(d, nlist, "l2", 64, pool_blocks=600, storage=storage, pq_m=pq_m, candidates_per_query=4096)
        g.set_centroids(dev(C))
        if pq_m:
            g.set_codebooks(dev(synth.codebooks_from_rows(1, y, pq_m)))
        g.set_param("ordered_add", 1)
        for lo in range(0, n, step):
            g.add(dev(y[lo:lo + step]), dev(np.arange(lo, min(n, lo + step), dtype=np.int64)))
        g.validate()
        out = [(g.list_export_codes(k) if pq_m else g.list_export(k)) for k in range(nlist)]
        held.append([(i.cpu().numpy(), v.cpu().numpy()) for i, v in out])
        torch.cuda.synchronize()
        g.close()
    for (ia, va), (ib, vb) in zip(*held):
        assert np.array_equal(ia, ib) and np.array_equal(va, vb)
