"""A sample read by several workgroups (requests of few queries, wide vectors or long lists) gives the answers that one
workgroup's gives: the same queries inside a request of 256, where every query has one workgroup, answer bit for bit alike;
on a slice, on the static array, recorded, and with small requests in between, which share the counters."""
import pytest
import torch

from paper_2408_02937_amd import rtams

pytestmark = pytest.mark.gpu


def build(n, d, nlist, metric, storage="f32", hot=0):
    gen = torch.Generator("cuda:0").manual_seed(n + d)
    C = torch.randn(nlist, d, device="cuda:0", generator=gen) * 20 + 100
    if metric == "ip":
        C = C - 100
    at = torch.randint(nlist, (n,), device="cuda:0", generator=gen)
    at[:hot] = 3
    y = C[at] + 8 * torch.randn(n, d, device="cuda:0", generator=gen)
    g = rtams.Index(d, nlist, metric, 64, pool_blocks=n // 64 + 2 * nlist + 64, n_resources=3, max_batch=256, max_k=128,
                    max_nprobe=64, candidates_per_query=n, storage=storage)
    g.set_centroids(C)
    g.add(y)
    q = C[torch.randint(nlist, (256,), device="cuda:0", generator=gen)] + 8 * torch.randn(256, d, device="cuda:0", generator=gen)
    if hot:
        q[::3] = C[3] + 8 * torch.randn(86, d, device="cuda:0", generator=gen)
    return g, q.contiguous()


# samples of 512 vectors (8 groups, fewer than the wavefronts of four workgroups), of a long list's quarter, and more keys
# than the query's row has room for (600 lists: one workgroup again); inner products without a bound below 32 d candidates
@pytest.mark.parametrize("metric", ["l2", "ip"])
@pytest.mark.parametrize("storage,d,nlist,hot,n", [("f32", 256, 512, 0, 80_000), ("f32", 260, 1030, 5000, 220_000),
                                                   ("f32", 256, 600, 12000, 130_000), ("f16", 512, 512, 4000, 160_000),
                                                   ("u8", 1024, 640, 0, 360_000)])
def test_parts_of_a_sample(storage, d, nlist, hot, n, metric):
    print(f"[case] sample parts {metric} {storage} d={d} {nlist} lists, hot {hot}", flush=True)
    g, q = build(n, d, nlist, metric, storage, hot)
    g.set_param("use_mfma", 0)
    sizes = torch.from_numpy(g.list_sizes()).cuda()
    for mode in (0, 2) if metric == "ip" else (0,):
        g.set_param("scan_mfma", mode)
        for k, nprobe in ((10, 64), (128, 64), (1, 60)):
            total = sizes[g.probe(q, nprobe).long()].sum(1).cpu()
            bounded = total > (4096 if metric == "l2" else max(4096, 32 * d))
            assert int(bounded.sum()) > 240
            want_d, want_i = g.search(q, k, nprobe)
            for nq in (1, 3, 63, 64, 128, 200):
                small = g.search(q[:1].contiguous(), 5, 2)  # leaves the counters as it finds them
                torch.cuda.synchronize()
                got_d, got_i = g.search(q[:nq].contiguous(), k, nprobe)
                torch.cuda.synchronize()
                assert g.poll_error() == 0
                assert torch.equal(got_d, want_d[:nq]) and torch.equal(got_i, want_i[:nq]), f"{nq} queries, k {k}, unit {mode}"
                assert (small[1] >= 0).any()
                keys, kept, path = g.request_trace(nq)
                assert path == ("k_scan_mm" if mode else path) and path in ("k_scan", "k_scan_small", "k_scan_mm")
                assert torch.equal(keys.to(torch.int64) != 0xFFFFFFFF, bounded[:nq]), f"{nq} queries, k {k}, unit {mode}"
                assert (kept.to(torch.int64)[bounded[:nq]] < total[:nq][bounded[:nq]]).all()
    g.set_param("scan_mfma", 0)
    out_d, out_i = torch.empty(9, 10, device="cuda:0"), torch.empty(9, 10, dtype=torch.int64, device="cuda:0")
    want_d, want_i = g.search(q, 10, 64)
    q9 = q[:9].contiguous()
    torch.cuda.synchronize()
    for _ in range(3):
        g.search_noalloc(q9, 10, 64, out_d, out_i)
        torch.cuda.synchronize()
        assert torch.equal(out_d, want_d[:9]) and torch.equal(out_i, want_i[:9])
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        g.search_noalloc(q9, 10, 64, out_d, out_i)
    for _ in range(4):
        out_d.zero_()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(out_d, want_d[:9]) and torch.equal(out_i, want_i[:9])
        g.search(q[:40].contiguous(), 10, 64)
        torch.cuda.synchronize()
    assert g.poll_error() == 0
    g.close()
