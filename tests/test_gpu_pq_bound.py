"""The bound of a request over quantised lists, taken from a table in LDS and from codes read ahead: 4 to 64 codes to a
vector (one, several and not a whole number of the words read ahead), nearest lists of fewer groups than the workgroup has
wavefronts and of more, and empty ones."""
import numpy as np
import pytest
import torch

from paper_2408_02937_amd import synth
from tests.gpu_common import dev
from tests.helpers import assert_topk_matches, ATOL_PQ, RTOL
from tests.test_gpu_pq import make_pq_pair

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("metric", ["l2", "ip"])
@pytest.mark.parametrize("M,d", [(4, 32), (8, 24), (20, 40), (36, 36), (64, 128)])
def test_samples_of_every_width(M, d, metric):
    print(f"[case] pq bound M={M} d={d} {metric}", flush=True)
    rng = np.random.default_rng(M)
    nlist = 24
    C = (rng.standard_normal((nlist, d)) * 4).astype(np.float32)
    C[5] = C[6] = 1e4  # the nearest lists of a query there are empty
    if metric == "ip":
        C /= np.linalg.norm(C, axis=1, keepdims=True)
    share = np.r_[np.full(20, 400), 2200, 130, 0, 0]  # one list of 35 groups, one of three
    lists = [i for i in range(nlist) if i not in (5, 6)] + [5, 6]
    at = np.repeat(lists, share)
    y = (C[at] + 0.3 * rng.standard_normal((len(at), d))).astype(np.float32)
    cb = (rng.standard_normal((M, 256, d // M)) * 2).astype(np.float32)
    w = synth.Workload("pq-bound", metric, d, nlist, 64, nlist, 20, y, C, np.zeros((0, d), np.float32),
                       np.zeros((0, d), np.float32), 1, 0)
    g, o = make_pq_pair(w, M, cb, pool_blocks=len(y) // 64 + 3 * nlist)
    g.add(dev(y)); o.add(y)
    q = (C[rng.integers(0, nlist, 60)] + 0.3 * rng.standard_normal((60, d))).astype(np.float32)
    q[:3] = C[5]
    for k, nprobe in ((1, nlist), (20, nlist), (100, 12)):
        rd, ri = o.search(q, k, nprobe)
        dd, ii = g.search(dev(q), k, nprobe)
        torch.cuda.synchronize()
        assert g.poll_error() == 0
        # fp32 sums of M entries: M 2^-24 of the sum of their sizes at most, which by Cauchy-Schwarz is the query's length times
        # that of the longest reconstruction (squared distances: terms of one sign, the relative tolerance holds them)
        longest = np.sqrt((np.linalg.norm(cb, axis=2).max(axis=1) ** 2).sum()) * np.linalg.norm(q, axis=1).max()
        assert_topk_matches(metric, dd.cpu().numpy(), ii.cpu().numpy(), rd, ri, rtol=RTOL,
                            atol=max(ATOL_PQ, (M + d // M) * 2.0 ** -24 * longest if metric == "ip" else 0.0),
                            what=f"M {M}, k {k}, {nprobe} probes")
    g.close()
