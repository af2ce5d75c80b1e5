"""The matrix-core filter at the edges of its tiles: one, two, three and more steps of 32 coordinates, rows and centroids
around the multiples a tile takes, lanes that hold several candidates and tiles that hold more than they keep.  Whatever the
filter narrows down is decided by the exact arithmetic, so every list is the one the exact kernel gives."""
import pytest
import torch

from paper_2408_02937_amd import rtams

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("metric", ["l2", "ip"])
@pytest.mark.parametrize("m,nlist,d,clusters", [
    (32, 1, 4, 1), (33, 63, 32, 63), (127, 64, 36, 64), (128, 65, 64, 65), (129, 255, 68, 255), (300, 256, 96, 256),
    (1000, 257, 100, 257), (1000, 1000, 260, 1000), (2100, 8200, 128, 8200), (700, 520, 772, 520),
    # centroids in clusters far tighter than the whole: several candidates to a lane, and more than a tile keeps
    (400, 512, 64, 100), (400, 520, 100, 40), (400, 1000, 32, 12), (260, 300, 128, 2)])
def test_the_filter_gives_the_lists_of_the_exact_kernel(m, nlist, d, clusters, metric):
    print(f"[case] filter tiles {m} x {nlist} x {d} in {clusters} clusters {metric}", flush=True)
    gen = torch.Generator("cuda:0").manual_seed(m + nlist + d)
    centres = torch.randn(clusters, d, device="cuda:0", generator=gen)
    C = centres[torch.arange(nlist, device="cuda:0") % clusters]
    if clusters < nlist:
        C = C + 1e-4 * torch.randn(nlist, d, device="cuda:0", generator=gen)
    y = C[torch.randint(nlist, (m,), device="cuda:0", generator=gen)] + 0.2 * torch.randn(m, d, device="cuda:0", generator=gen)
    C, y = C.contiguous(), y.contiguous()
    g = rtams.Index(d, nlist, metric, 64, pool_blocks=2 * nlist + m // 64 + 64, n_resources=2, max_batch=256, max_k=8,
                    max_nprobe=min(nlist, 8), max_add_batch=4096, candidates_per_query=4096)
    g.set_centroids(C)
    got, probes = {}, {}
    for mode in (0, 2):
        g.set_param("use_mfma", mode)
        got[mode] = g.assign(y)
        probes[mode] = g.probe(y[:256].contiguous(), min(nlist, 8))
    torch.cuda.synchronize()
    assert torch.equal(got[0], got[2])
    assert torch.equal(probes[0], probes[2])
    g.close()
