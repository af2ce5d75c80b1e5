"""Assignment where the centroids come in clusters much tighter than the whole: the band of a vector holds tens of its
cluster's centroids, and tiles hold more of them than they can keep."""
import numpy as np
import pytest
import torch

from paper_2408_02937_amd import rtams

pytestmark = pytest.mark.gpu


def index(clusters, nlist, d, rows):
    gen = torch.Generator("cuda:0").manual_seed(nlist + d + clusters)
    heads = torch.randn(clusters, d, device="cuda:0", generator=gen)
    draw = lambda n: (heads[torch.randint(clusters, (n,), device="cuda:0", generator=gen)] +
                      0.1 * torch.randn(n, d, device="cuda:0", generator=gen))
    g = rtams.Index(d, nlist, "l2", 64, pool_blocks=64, n_resources=1, max_batch=8, max_k=8, max_nprobe=8,
                    candidates_per_query=1024)
    g.set_centroids(draw(nlist))
    return g, draw(rows)


# few rows to a workgroup of the refinement and many, rows with tens of candidates and with whole tiles
@pytest.mark.parametrize("clusters,nlist,d,rows", [(100, 2048, 24, 300), (100, 8192, 256, 2048), (10, 1000, 128, 9000),
                                                   (3, 777, 36, 70_000), (1, 300, 64, 5000)])
def test_clustered_centroids_decide_as_the_exact_kernel(clusters, nlist, d, rows):
    print(f"[case] {clusters} clusters of {nlist} centroids x {d}, {rows} rows", flush=True)
    g, y = index(clusters, nlist, d, rows)
    got = []
    for mode in (2, 0):
        g.set_param("use_mfma", mode)
        got.append(g.assign(y).cpu().numpy())
    assert np.array_equal(*got)
    g.close()


def test_clusters_cost_little_more_than_none():
    """131,072 vectors x 256 against 8,192 centroids: 1.8 ms where they come in 100 clusters and 1.1 where they do not (5.0
    ms when a tile kept four columns and rows with more than sixteen candidates were scored by a wavefront each)."""
    ms = []
    for clusters in (100, 8192):
        g, y = index(clusters, 8192, 256, 131_072)
        t = []
        for _ in range(5):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            g.assign(y)
            b.record()
            torch.cuda.synchronize()
            t.append(a.elapsed_time(b))
        ms.append(min(t))
        g.close()
    print(f"[case] clustered, spread: {ms} ms", flush=True)
    assert ms[0] < 2.5 * ms[1]
