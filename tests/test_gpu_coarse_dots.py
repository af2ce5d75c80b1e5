"""Probes by inner product at the edges of the double-precision matrix tiles (16 vectors, 16 centroids, 64 to a workgroup, 16
and 32 chunks of a row): the lists of the fixed arithmetic, one fused multiply-add per coordinate, in order.  The centroids
are permutations of one another and the vectors hold one value each, so all scores of a vector are the same number but
for the rounding of sums in different orders: any other order of the arithmetic chooses other lists."""
import numpy as np
import pytest
import torch

from oracle import oracle as orc
from paper_2408_02937_amd import rtams

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,nlist,d", [
    (8, 1, 4), (15, 16, 8), (16, 17, 60), (17, 63, 64), (33, 65, 68), (31, 300, 124), (64, 1000, 128),
    (100, 1400, 132), (256, 512, 196), (12, 4096, 768), (24, 4100, 260), (128, 1030, 2048)])
def test_the_lists_of_the_chain(n, nlist, d):
    print(f"[case] dots {n} x {nlist} x {d}", flush=True)
    rng = np.random.default_rng(n + nlist + d)
    row = rng.standard_normal(d).astype(np.float32) * np.exp2(rng.integers(-12, 12, d)).astype(np.float32)
    C = np.stack([rng.permutation(row) for _ in range(nlist)])
    q = np.repeat(rng.standard_normal((n, 1)).astype(np.float32), d, axis=1)
    nprobe = min(nlist, 8)
    o = orc.OracleIndex(d, nlist, "ip", 64, pool_blocks=8)
    o.set_centroids(C)
    g = rtams.Index(d, nlist, "ip", 64, pool_blocks=nlist + 8, n_resources=2, max_batch=256, max_k=8, max_nprobe=nprobe,
                    candidates_per_query=1024)
    g.set_param("use_mfma", 0)  # the exact scores alone
    g.set_centroids(torch.from_numpy(C).cuda())
    got = g.probe(torch.from_numpy(q).cuda(), nprobe)
    torch.cuda.synchronize()
    assert np.array_equal(got.cpu().numpy(), o.probe(q, nprobe))
    g.close()
