"""Small batches that are assigned, opened, filled and published in one launch, and large ones that are filled list by
list: lists bit for bit against the oracle, block structure and counters, at the sizes where the paths begin and end."""
import numpy as np
import pytest

from paper_2408_02937_amd import synth
from tests.gpu_common import assert_lists_equal, dev, make_pair

pytestmark = pytest.mark.gpu


def run(batches, d, nlist, metric, hot, storage="f32", pool_blocks=3000):
    rng = np.random.default_rng(sum(batches) + d + nlist)
    C = rng.standard_normal((nlist, d)).astype(np.float32)
    if storage == "u8":
        C = np.rint(100 + 30 * C)
    w = synth.Workload("paths", metric, d, nlist, 64, min(8, nlist), 10, np.zeros((0, d), np.float32), C.astype(np.float32),
                       np.zeros((0, d), np.float32), np.zeros((0, d), np.float32), 1, 0)
    g, o = make_pair(w, pool_blocks=pool_blocks, candidates_per_query=16384, storage=storage)
    bounds = []
    for m in batches:
        at = np.full(m, nlist // 2) if hot else rng.integers(0, nlist, m)
        y = (C[at] + 0.05 * rng.standard_normal((m, d))).astype(np.float32)
        if storage == "u8":
            y = np.clip(np.rint(y), 0, 255).astype(np.float32)
        bounds.append(o.ntotal)
        g.add(dev(y)); o.add(y)
    g.validate()
    assert_lists_equal(g, o, np.array(bounds[1:]))
    assert g.ntotal == o.ntotal and g.poll_error() == 0
    g.close()


# one launch: up to 256 vectors of up to 4,096 chunks of 16 bytes in all (256 x 64, 240 x 68, 16 x 1,024)
@pytest.mark.parametrize("batches", [[1, 2, 1, 63, 64, 65], [255, 256, 257, 256], [240, 241, 16, 17, 100]])
@pytest.mark.parametrize("d,nlist,metric", [(4, 1, "l2"), (64, 3, "ip"), (68, 300, "l2"), (32, 2100, "ip"), (1024, 20, "l2")])
@pytest.mark.parametrize("hot", [False, True])
def test_batches_of_one_launch(batches, d, nlist, metric, hot):
    print(f"[case] one launch {batches} d={d} nlist={nlist} {metric} hot={hot}", flush=True)
    run(batches, d, nlist, metric, hot)


@pytest.mark.parametrize("storage,d", [("f16", 8), ("f16", 136), ("u8", 16), ("u8", 144)])
def test_batches_of_one_launch_into_narrow_lists(storage, d):
    print(f"[case] one launch {storage} d={d}", flush=True)
    run([1, 65, 256, 257], d, 30, "l2", False, storage)


# list by list from 8,192 vectors, or from 2^18 chunks above 1,024; a workgroup moves 64 vectors x 16 chunks: 1, 15, 16, 17, 33
# chunks of a vector.  1,025 narrow vectors go vector by vector
@pytest.mark.parametrize("n", [1025, 8191, 8192, 8257])
@pytest.mark.parametrize("storage,d", [("f32", 4), ("f32", 60), ("f32", 64), ("f32", 68), ("f32", 132), ("f16", 136), ("u8", 272)])
@pytest.mark.parametrize("nlist,hot", [(1, True), (7, False), (2500, False)])
def test_large_batches_list_by_list(n, storage, d, nlist, hot):
    print(f"[case] list by list {n} {storage} d={d} nlist={nlist}", flush=True)
    run([70, n, 3, n], d, nlist, "l2", hot, storage, pool_blocks=9000)


# 192 and 64 chunks of a vector: 2^18 of them are 1,366 and 4,096 vectors
@pytest.mark.parametrize("d,n", [(768, 1365), (768, 1366), (768, 2049), (256, 4095), (256, 4096), (256, 4200), (1024, 1025)])
def test_fewer_vectors_list_by_list_where_they_are_wide(d, n):
    print(f"[case] list by list, wide: {n} x {d}", flush=True)
    run([70, n, 3, n], d, 300, "l2", False, "f32", pool_blocks=2000)


def test_rounds_and_ids_of_the_caller_list_by_list():
    """One call of three rounds (8,192, 8,192 and 3,616 vectors, the last by vector) with ids of its own, beside one without."""
    print("[case] list by list, rounds and ids", flush=True)
    rng = np.random.default_rng(12)
    d, nlist, n = 36, 90, 20_000
    C = rng.standard_normal((nlist, d)).astype(np.float32)
    w = synth.Workload("rounds", "l2", d, nlist, 64, 8, 10, np.zeros((0, d), np.float32), C, np.zeros((0, d), np.float32),
                       np.zeros((0, d), np.float32), 1, 0)
    g, o = make_pair(w, pool_blocks=2000, candidates_per_query=16384, max_add_batch=8192)
    for ids in (None, rng.permutation(10 * n)[:n].astype(np.int64) + (1 << 40)):
        y = (C[rng.integers(0, nlist, n)] + 0.05 * rng.standard_normal((n, d))).astype(np.float32)
        g.add(dev(y), None if ids is None else dev(ids)); o.add(y, ids)
    g.validate()
    assert_lists_equal(g, o)
    assert g.ntotal == o.ntotal and g.poll_error() == 0
    g.close()


def test_a_vector_with_a_nan_joins_the_first_list_in_one_launch():
    print("[case] one launch, a NaN", flush=True)
    rng = np.random.default_rng(9)
    C = rng.standard_normal((40, 16)).astype(np.float32)
    w = synth.Workload("nan", "l2", 16, 40, 64, 8, 10, np.zeros((0, 16), np.float32), C, np.zeros((0, 16), np.float32),
                       np.zeros((0, 16), np.float32), 1, 0)
    g, o = make_pair(w, pool_blocks=200, candidates_per_query=1024)
    y = C[rng.integers(0, 40, 20)].copy()
    y[7, 3] = np.nan
    g.add(dev(y)); o.add(y)
    assert np.array_equal(g.list_sizes(), o.list_sizes())
    g.validate()
    g.close()
