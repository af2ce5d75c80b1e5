"""Squared distances to lists of halves and bytes on the 16-bit matrix instructions, where that scan can go wrong: the
narrowest and widest vectors it takes and the next ones, chunks past the vector's end, tiles of 16, 17 and 32 queries, queries that need
one, two and three pieces side by side, subnormal halves, and lengths far from one."""
import numpy as np
import pytest
import torch

from paper_2408_02937_amd import synth
from tests.gpu_common import assert_lists_equal, dev, make_pair, scan_modes
from tests.helpers import assert_topk_matches, RTOL

pytestmark = pytest.mark.gpu


def pair(storage, C, n, d, k=20):
    nlist = len(C)
    w = synth.Workload("narrow-pieces", "l2", d, nlist, 128, nlist, k, np.zeros((0, d), np.float32), C,
                       np.zeros((0, d), np.float32), np.zeros((0, d), np.float32), 1, 0)
    return make_pair(w, pool_blocks=n // 128 + 4 * nlist + 8, max_k=128, candidates_per_query=n + 64, storage=storage)


def check(g, o, q, k, nprobe, what, atol=1e-5):
    rd, ri = o.search(q, k, nprobe)
    for mode in scan_modes(g):
        dd, ii = g.search(dev(q), k, nprobe)
        assert_topk_matches("l2", dd.cpu().numpy(), ii.cpu().numpy(), rd, ri, rtol=RTOL, atol=atol, what=f"{what}, scan_mfma {mode}")


# whole fours of chunks and one, two or three past them; the first and the last width that is taken, and their neighbours
@pytest.mark.parametrize("storage,d", [("f16", 24), ("f16", 32), ("f16", 40), ("f16", 72), ("f16", 120), ("f16", 632), ("f16", 640),
                                       ("f16", 648), ("u8", 48), ("u8", 64), ("u8", 80), ("u8", 112), ("u8", 624), ("u8", 640),
                                       ("u8", 656)])
def test_widths_and_tiles(storage, d):
    print(f"[case] narrow pieces {storage} d={d}", flush=True)
    rng = np.random.default_rng(d)
    C = (np.clip(120 + 40 * rng.standard_normal((4, d)), 0, 255) if storage == "u8" else rng.standard_normal((4, d))).astype(np.float32)
    n = 2600
    g, o = pair(storage, C, n, d)
    noise = 9.0 if storage == "u8" else 0.2
    draw = lambda m: (C[rng.integers(0, 4, m)] + noise * rng.standard_normal((m, d))).astype(np.float32)
    y = draw(n)
    g.add(dev(y)); o.add(y)
    assert_lists_equal(g, o)
    for nq in (15, 16, 17, 32, 33, 70):  # every list has all queries: tiles of 16, one more, 32, ...
        q = draw(nq)
        if nq == 17:
            q = np.rint(q)  # one piece (bytes)
        if nq == 32:
            q[::2] = np.rint(q[::2])
            q[1::4] = q[1::4].astype(np.float16)  # one or two pieces beside three
        check(g, o, q.astype(np.float32), 20, 4, f"{storage} d={d}, {nq} queries")
    g.close()


@pytest.mark.parametrize("size", [1e-6, 1e-3, 200.0, 2e4])
def test_halves_of_every_length(size):
    """1e-6: every stored coordinate is a subnormal half; 2e4: near the largest."""
    print(f"[case] narrow pieces, halves of size {size}", flush=True)
    rng = np.random.default_rng(3)
    d, n = 72, 3000
    C = (size * rng.uniform(-1, 1, (6, d))).astype(np.float32)
    g, o = pair("f16", C, n, d)
    y = (C[rng.integers(0, 6, n)] + size * 0.3 * rng.standard_normal((n, d))).astype(np.float32)
    g.add(dev(y)); o.add(y)
    q = (C[rng.integers(0, 6, 90)] + size * 0.3 * rng.standard_normal((90, d))).astype(np.float32)
    q[0] = 0.0  # no length: no scale
    q[1] *= 1e4  # far outside of what the lists hold
    check(g, o, q, 20, 6, f"halves of size {size}", atol=1e-5 * size * size * d)
    g.close()
