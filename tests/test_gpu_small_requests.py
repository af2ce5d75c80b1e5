"""Small requests over short lists, whose scan walks them one at a time and whose selection takes the survivor records
as they come: against the oracle, at every storage and at numbers of chunks around a register set's, and at numbers of
survivors around what the selection holds."""
import numpy as np
import pytest

from paper_2408_02937_amd import synth
from tests.gpu_common import assert_lists_equal, dev, make_pair
from tests.helpers import assert_topk_matches, RTOL

pytestmark = pytest.mark.gpu


def loaded(storage, metric, d, n, nlist=24, k=20, candidates=None):
    rng = np.random.default_rng(7 * d + n)
    C = rng.standard_normal((nlist, d))
    if storage == "u8":
        C = np.clip(120 + 40 * C, 0, 255)
    C = C.astype(np.float32)
    w = synth.Workload("small", metric, d, nlist, 128, 6, k, np.zeros((0, d), np.float32), C,
                       np.zeros((0, d), np.float32), np.zeros((0, d), np.float32), 1, 0)
    g, o = make_pair(w, pool_blocks=400, max_k=1024, candidates_per_query=candidates or n, storage=storage)
    draw = lambda m: (C[rng.integers(0, nlist, m)] +
                      (9.0 if storage == "u8" else 0.2) * rng.standard_normal((m, d))).astype(np.float32)
    y = draw(n)
    g.add(dev(y)); o.add(y)
    return g, o, draw


@pytest.mark.parametrize("metric", ["l2", "ip"])
# chunks of a vector: less than a set, two sets exactly, one more; of floats also two sets of eight, once and twice
@pytest.mark.parametrize("storage,d", [("f32", 4), ("f32", 28), ("f32", 32), ("f32", 36), ("f32", 64), ("f32", 68),
                                       ("f32", 128), ("f16", 24), ("f16", 64), ("f16", 72), ("u8", 48), ("u8", 128),
                                       ("u8", 144)])
def test_one_group_at_a_time_gives_the_oracle_s_answers(storage, d, metric):
    print(f"[case] small requests {storage} d={d} {metric}", flush=True)
    g, o, draw = loaded(storage, metric, d, 5000)  # 208 vectors a list: 4 groups, so 2048 groups are 512 pairs
    assert_lists_equal(g, o)
    g.set_param("scan_mfma", 0)
    for nq, nprobe, k in ((1, 1, 20), (1, 24, 1), (9, 24, 100), (21, 24, 20), (22, 24, 20)):
        q = draw(nq)
        rd, ri = o.search(q, k, nprobe)
        dd, ii = g.search(dev(q), k, nprobe)
        assert_topk_matches(metric, dd.cpu().numpy(), ii.cpu().numpy(), rd, ri, rtol=RTOL, atol=1e-5,
                            what=f"{nq} queries, {nprobe} probes, k {k}")
    g.close()


@pytest.mark.parametrize("n", [1, 63, 1024, 1025, 4095, 4096, 4097, 6000])
def test_all_vectors_survive(n):
    """k near the number of vectors keeps every record: as many as the selection takes directly, and one more."""
    g, o, draw = loaded("f32", "l2", 16, n, nlist=3)
    q = draw(5)
    for k in (1, min(n, 1024), 1024):
        rd, ri = o.search(q, k, 3)
        dd, ii = g.search(dev(q), k, 3)
        assert_topk_matches("l2", dd.cpu().numpy(), ii.cpu().numpy(), rd, ri, rtol=RTOL, atol=1e-5, what=f"k {k}")
    g.close()
