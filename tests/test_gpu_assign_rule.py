"""Insertion batches on both sides of the line from which assignments go through the matrix-core filter take the path
that is faster, and the vectors join the lists the other path gives."""
import numpy as np
import pytest
import torch

from paper_2408_02937_amd import rtams

pytestmark = pytest.mark.gpu


# measured, exact / filter: 40 / 55, 47 / 60, 35 / 48, 65 / 61, 144 / 67, 47 / 38, 30 / 37 us a batch
@pytest.mark.parametrize("m,nlist,d", [(256, 420, 688), (256, 1024, 768), (256, 420, 512), (256, 2048, 768),
                                       (512, 4096, 768), (3725, 306, 32), (1024, 1024, 32)])
def test_a_batch_takes_the_faster_path(m, nlist, d):
    print(f"[case] assign rule {m} x {nlist} x {d}", flush=True)
    gen = torch.Generator("cuda:0").manual_seed(m + d)
    C = torch.randn(nlist, d, device="cuda:0", generator=gen)
    y = C[torch.randint(nlist, (m,), device="cuda:0", generator=gen)]
    # unit vectors far from their centroid: several centroids are candidates, as at the borders of cells
    C /= C.norm(dim=1, keepdim=True)
    y = y / y.norm(dim=1, keepdim=True) + 0.3 * torch.randn(m, d, device="cuda:0", generator=gen)
    y /= y.norm(dim=1, keepdim=True)
    g = rtams.Index(d, nlist, "ip", 64, pool_blocks=40 * nlist + 1000 * m // 64, n_resources=1, max_batch=8, max_k=8,
                    max_nprobe=8, candidates_per_query=1024)
    g.set_centroids(C)
    ms, lists = {}, {}
    for mode in (0, 2, 1) * 4:  # the shortest of four turns each
        g.set_param("use_mfma", mode)
        lists[mode] = g.assign(y).cpu().numpy()
        for _ in range(5):
            g.add(y)
        torch.cuda.synchronize()
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record()
        for _ in range(40):
            g.add(y)
        b.record()
        torch.cuda.synchronize()
        ms[mode] = min(ms.get(mode, 1e9), a.elapsed_time(b) / 40)
    print(f"[case] exact, rule, filter: {ms[0]:.4f} {ms[1]:.4f} {ms[2]:.4f} ms", flush=True)
    assert np.array_equal(lists[0], lists[2]) and np.array_equal(lists[0], lists[1])
    assert ms[1] < 1.18 * min(ms[0], ms[2])
    g.close()
