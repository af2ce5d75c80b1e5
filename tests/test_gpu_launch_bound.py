"""What the host knows of the lists when it launches a search, and what it makes of it: the longest list, which picks
the scan's unit and bounds the work items a scan is launched for."""
import numpy as np
import pytest
import torch

from paper_2408_02937_amd import rtams

pytestmark = pytest.mark.gpu


def lists_of(lengths, d, seed, **kw):
    """An index with one centroid per list and vectors that join them in random order: (index, vectors)."""
    rng = np.random.default_rng(seed)
    nlist = len(lengths)
    C = (100.0 * rng.standard_normal((nlist, d))).astype(np.float32)
    at = rng.permutation(np.repeat(np.arange(nlist), lengths))
    y = torch.from_numpy(C).cuda()[torch.from_numpy(at).cuda()]
    y += torch.randn(y.shape, device="cuda:0", generator=torch.Generator("cuda:0").manual_seed(seed))
    kw = {"block_vecs": 64, "max_nprobe": min(64, nlist), "max_k": 16, "max_batch": 256, "n_resources": 2,
          "pool_blocks": int(sum(lengths)) // 64 + 2 * nlist + 8, "candidates_per_query": 65536, **kw}
    g = rtams.Index(d, nlist, "l2", **kw)
    g.set_centroids(torch.from_numpy(C).cuda())
    return g, y


def test_the_host_learns_the_longest_list_of_a_publication():
    """Lists of growing length published by many wavefronts at once, one of them 16 times the average: requests of 64
    queries with few pairs then scan on the matrix cores.  (A host word written by every wavefront that found a longer
    list kept a smaller length now and then: this fails without the mend on some loads only.)"""
    nlist = 4096
    lengths = np.linspace(1, 28, nlist).astype(int)
    lengths[-1] = 400
    for seed in range(25):
        g, y = lists_of(lengths, 4, seed)
        g.add(y)
        torch.cuda.synchronize()
        g.set_param("profile_scan", 1)
        g.scan_kernels(reset=True)
        g.search(y[:64].contiguous(), 5, 1)
        torch.cuda.synchronize()
        assert g.scan_kernels()["k_scan_mm"] == 1, f"load {seed}"
        g.close()
