"""Which unit scans a request, on both sides of the lines of the rule, and that the answers are the same either way."""
import numpy as np
import pytest
import torch

from paper_2408_02937_amd import rtams

pytestmark = pytest.mark.gpu


# metric, storage, d, lists, vectors of a list, of the last one, queries, probes, the unit that takes it
@pytest.mark.parametrize("metric,storage,d,nlist,length,last,nq,nprobe,unit", [
    ("ip", "f32", 768, 64, 300, 300, 256, 64, "k_scan_mm"),      # 1.4 to 1.9 times faster there
    ("ip", "f32", 512, 128, 300, 300, 128, 1, "k_scan_mm"),      # one pair to a list
    ("ip", "f32", 512, 129, 300, 300, 128, 1, "k_scan"),
    ("ip", "f32", 256, 64, 2000, 2000, 256, 64, "k_scan_mm"),    # 8.4 G products
    ("ip", "f32", 256, 64, 1800, 1800, 256, 64, "k_scan"),       # 7.6 G
    ("ip", "f32", 96, 64, 800, 800, 256, 64, "k_scan_mm"),       # 1.3 G
    ("ip", "f32", 96, 64, 500, 500, 256, 64, "k_scan"),          # 0.8 G
    ("ip", "f32", 256, 256, 50, 30_000, 256, 256, "k_scan_mm"),  # a hot list: 2.9 G
    ("ip", "f32", 256, 256, 50, 12_000, 256, 64, "k_scan"),      # 0.5 G
    ("ip", "f16", 512, 256, 20, 20, 64, 1, "k_scan_mm"),         # always from there
    ("ip", "f16", 128, 64, 600, 600, 64, 64, "k_scan_mm"),       # 0.3 G
    ("ip", "f16", 128, 64, 500, 500, 256, 64, "k_scan"),         # lists of fewer than 512
    ("ip", "u8", 128, 64, 600, 600, 64, 32, "k_scan"),           # 0.16 G
    ("l2", "f16", 512, 64, 600, 600, 128, 4, "k_scan_mm"),       # eight pairs to a list
    ("l2", "f16", 512, 64, 600, 600, 128, 3, "k_scan"),
    ("l2", "f16", 256, 64, 600, 600, 128, 2, "k_scan_mm"),       # four
    ("l2", "f32", 32, 128, 20, 20, 64, 1, "k_scan"),
])
def test_the_unit_that_scans(metric, storage, d, nlist, length, last, nq, nprobe, unit):
    print(f"[case] unit {metric} {storage} d={d} {nlist} x {length}, longest {last}, {nq} x {nprobe}", flush=True)
    gen = torch.Generator("cuda:0").manual_seed(d + nlist)
    # centroids of one length, so that every vector's nearest is its own under both metrics
    C = torch.randn(nlist, d, device="cuda:0", generator=gen)
    C *= 8.0 * d ** 0.5 / C.norm(dim=1, keepdim=True)
    if storage == "u8":
        C = (C + 60.0).clamp_(0.0, 255.0)
    at = torch.repeat_interleave(torch.arange(nlist, device="cuda:0"),
                                 torch.tensor([length] * (nlist - 1) + [last], device="cuda:0"))
    at = at[torch.randperm(len(at), device="cuda:0", generator=gen)]
    y = C[at] + 0.5 * torch.randn(len(at), d, device="cuda:0", generator=gen)
    g = rtams.Index(d, nlist, metric, 64, pool_blocks=len(y) // 64 + 2 * nlist + 8, n_resources=1, max_batch=256,
                    max_k=16, max_nprobe=nprobe, candidates_per_query=len(y), storage=storage)
    g.set_centroids(C)
    g.add(y)
    sizes = g.list_sizes()
    if storage != "u8":
        assert list(sizes) == [length] * (nlist - 1) + [last]
    q = y[:nq].contiguous()
    g.set_param("profile_scan", 1)
    out = {}
    for mode in (1, 0, 2):
        g.set_param("scan_mfma", mode)
        g.scan_kernels(reset=True)
        dist, ids = g.search(q, 10, nprobe)
        torch.cuda.synchronize()
        assert g.poll_error() == 0
        out[mode] = dist.cpu().numpy()
        if mode == 1:
            assert g.scan_kernels()[unit] == 1
    # fp32 sums of d terms in two orders: an inner product differs by 2 d 2^-24 of the norms' product (66 d) at most, a
    # squared distance by as much of itself
    for mode in (1, 0):
        assert np.allclose(out[mode], out[2], rtol=2 * d * 2.0 ** -24, atol=2 * d * 2.0 ** -24 * 66 * d if metric == "ip" else 0)
    g.close()
