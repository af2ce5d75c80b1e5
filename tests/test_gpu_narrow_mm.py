"""Lists of halves and bytes scanned on the matrix cores: against the oracle and against the vector-unit scan, at
dimensions around the chunks a register set holds, tiles of every size, and values that overflow a half."""
import numpy as np
import pytest
import torch

from paper_2408_02937_amd import synth
from tests.gpu_common import assert_lists_equal, dev, make_pair, scan_modes
from tests.helpers import assert_topk_matches, RTOL

pytestmark = pytest.mark.gpu


def loaded(storage, metric, d, nlist=24, n=9000, k=20, seed=0, scale=1.0):
    rng = np.random.default_rng(1000 * d + seed)
    C = rng.standard_normal((nlist, d)) * scale
    if storage == "u8":
        C = np.clip(120 + 40 * C, 0, 255)
    C = C.astype(np.float32)
    w = synth.Workload("narrow-mm", metric, d, nlist, 128, 6, k, np.zeros((0, d), np.float32), C,
                       np.zeros((0, d), np.float32), np.zeros((0, d), np.float32), 1, 0)
    g, o = make_pair(w, pool_blocks=400, max_k=128, candidates_per_query=n, storage=storage)
    draw = lambda m: (C[rng.integers(0, nlist, m)] + (9.0 if storage == "u8" else 0.2 * scale) *
                      rng.standard_normal((m, d))).astype(np.float32)
    y = draw(n)
    g.add(dev(y)); o.add(y)
    return g, o, draw


@pytest.mark.parametrize("metric", ["l2", "ip"])
# chunks of a vector: 1, 2, 7, 8, 9, 17 (a register set holds four, two sets go round)
@pytest.mark.parametrize("storage,d", [("f16", 8), ("f16", 56), ("f16", 64), ("f16", 136), ("u8", 16), ("u8", 32),
                                       ("u8", 112), ("u8", 128), ("u8", 144), ("u8", 272)])
def test_both_scans_give_the_oracle_s_answers(storage, d, metric):
    print(f"[case] narrow scan {storage} d={d} {metric}", flush=True)
    g, o, draw = loaded(storage, metric, d)
    assert_lists_equal(g, o)
    for nq, nprobe, k in ((1, 24, 20), (5, 6, 1), (33, 6, 20), (131, 24, 100), (256, 3, 20)):
        q = draw(nq)
        rd, ri = o.search(q, k, nprobe)
        for mode in scan_modes(g, (1, 2, 0)):
            dd, ii = g.search(dev(q), k, nprobe)
            assert_topk_matches(metric, dd.cpu().numpy(), ii.cpu().numpy(), rd, ri, rtol=RTOL, atol=1e-5,
                                what=f"scan_mfma {mode}, {nq} queries, k {k}")
    g.close()


def test_values_that_overflow_a_half_are_infinitely_far_in_both_scans():
    """Vectors with a coordinate beyond the largest half are kept as infinities; a search that asks for more than the
    finite ones gets them last, at an infinite distance, whichever unit scans."""
    g, o, draw = loaded("f16", "l2", 32, nlist=2, n=60)
    y = draw(40)
    y[::2, 3] = 1e6
    y[1::4, 5] = -1e6
    g.add(dev(y)); o.add(y)
    q = draw(70)
    rd, _ = o.search(q, 100, 2)
    for mode in scan_modes(g, (2, 0)):
        dd, ii = g.search(dev(q), 100, 2)
        dd, ii = dd.cpu().numpy(), ii.cpu().numpy()
        assert np.array_equal(np.isinf(dd), np.isinf(rd)), f"scan_mfma {mode}"
        assert np.allclose(dd[~np.isinf(rd)], rd[~np.isinf(rd)], rtol=1e-4)
        assert np.all(np.sort(ii, axis=1) == np.arange(100)), f"scan_mfma {mode}: every vector is returned once"
    g.close()
