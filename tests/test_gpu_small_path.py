"""Small requests go without a plan (three launches); the same requests through the plan give the same answers bit for bit:
number of lists around what a workgroup takes, few and many probes, empty lists, fewer candidates than k, every kind of
list, requests of different sizes in turn on the same slices.  Which way a request went is read back every time."""
import pytest
import torch

from paper_2408_02937_amd import rtams

pytestmark = pytest.mark.gpu


def build(n, d, nlist, metric, storage, T=64, hot=False, n_resources=2):
    gen = torch.Generator("cuda:0").manual_seed(n + d + nlist)
    C = torch.randn(nlist, d, device="cuda:0", generator=gen) * 20 + 100
    at = torch.randint(max(1, nlist // (4 if n < nlist else 1)), (n,), device="cuda:0", generator=gen)
    if hot:
        at[: n // 2] = 3
    y = (C[at] + 8 * torch.randn(n, d, device="cuda:0", generator=gen)).round().clamp(0, 255)
    g = rtams.Index(d, nlist, metric, T, pool_blocks=n // T + 2 * nlist + 64, n_resources=n_resources, max_batch=64, max_k=128,
                    max_nprobe=min(nlist, 64), candidates_per_query=n + 64, storage=storage)
    g.set_centroids(C)
    if n:
        g.add(y)
    q = (C[torch.randint(nlist, (40,), device="cuda:0", generator=gen)] + 8 * torch.randn(40, d, device="cuda:0", generator=gen)).contiguous()
    return g, q


def goes_small(g, n, longest, nq, nprobe):
    """The rule: vectors of a workgroup's coarse tile, bytes the queries read, and how wide vectors may be."""
    blocks = (g.nlist + 255) // 256
    vt = 8 if g.d <= 768 else 4
    while vt > 1 and (nq + vt - 1) // vt * blocks < 256:
        vt //= 2
    if not 32 <= g.nlist <= 4096 or nprobe > 64 or vt > 1:
        return False
    avg = n // g.nlist + 1
    chunks = g.d // {"f32": 4, "f16": 8, "u8": 16}[g.storage]
    if nq * (nprobe * avg + longest) * chunks * 16 > 32e6:
        return False
    short, narrow = avg // 64 + 1 <= 4, g.storage != "f32"
    wide = (1024 if narrow else 768) if short else (768 if narrow else 512)
    if g.d > wide and g.nlist > 256 and not (short and (nq >= 16 or nq * nprobe >= (100 if narrow else 400) * (2 if g.d > 1536 else 1))):
        return False
    return short or nprobe * avg <= (4096 if g.metric == rtams.L2 else max(4096, 32 * g.d)) or (chunks < 96 and g.d <= 512)


def both(g, q, k, nprobe):
    sizes = g.list_sizes()
    torch.cuda.synchronize()
    small = goes_small(g, int(sizes.sum()), int(sizes.max()), q.shape[0], nprobe)
    out = []
    for on in (1, 0, 1):
        g.set_param("small_requests", on)
        out.append(g.search(q, k, nprobe))
        torch.cuda.synchronize()
        assert g.request_trace(q.shape[0])[2] == ("k_scan_small" if on and small else "k_scan"), f"{q.shape[0]} x {nprobe}"
    assert torch.equal(out[0][0], out[1][0]) and torch.equal(out[0][1], out[1][1])
    assert torch.equal(out[0][0], out[2][0]) and torch.equal(out[0][1], out[2][1])
    assert g.poll_error() == 0
    return small


@pytest.mark.parametrize("metric", ["l2", "ip"])
@pytest.mark.parametrize("nlist,d,n", [(32, 4, 500), (33, 32, 9000), (511, 64, 30000), (513, 128, 30000), (1025, 96, 40000),
                                       (2049, 36, 30000), (4096, 64, 60000), (4097, 64, 60000), (700, 1536, 3000),
                                       (700, 768, 3000), (700, 772, 3000), (64, 512, 30000), (64, 384, 30000), (64, 380, 30000)])
def test_small_requests_answer_like_planned_ones(nlist, d, n, metric):
    print(f"[case] small path {metric} {n} x {d} into {nlist}", flush=True)
    g, q = build(n, d, nlist, metric, "f32")
    took = [both(g, q[:nq].contiguous(), k, nprobe)
            for nq, k, nprobe in ((1, 100, 32), (10, 10, 8), (3, 1, 1), (7, 128, min(64, nlist)), (1, 50, min(63, nlist)), (33, 5, 2))]
    assert any(took) == (nlist <= 4096)
    g.close()


@pytest.mark.parametrize("metric", ["l2", "ip"])
@pytest.mark.parametrize("storage,d", [("f16", 72), ("u8", 80), ("u8", 1024), ("f16", 1032), ("u8", 1040)])
@pytest.mark.parametrize("n,hot", [(20, False), (6000, False), (20000, True)])
def test_small_requests_over_narrow_empty_and_hot_lists(storage, d, n, hot, metric):
    print(f"[case] small path {metric} {storage} {n} hot={hot}", flush=True)
    g, q = build(n, d, 200, metric, storage, hot=hot)
    for nq, k, nprobe in ((1, 100, 32), (9, 10, 64), (2, 128, 1)):
        took = both(g, q[:nq].contiguous(), k, nprobe)
        assert took or hot or d > 1000 and nq > 1
    g.close()


def test_an_empty_index_and_a_slice_that_is_too_small():
    print("[case] small path, nothing to find", flush=True)
    g, q = build(0, 32, 64, "l2", "f32")
    d, i = g.search(q[:5].contiguous(), 10, 8)
    assert torch.isinf(d).all() and (i == -1).all()
    g.close()
    g, q = build(8000, 32, 40, "l2", "f32")
    small = rtams.Index(32, 40, "l2", 64, pool_blocks=300, n_resources=1, max_batch=4, max_k=16, max_nprobe=40, candidates_per_query=1000)
    small.set_centroids(torch.randn(40, 32, device="cuda:0"))
    small.add(torch.randn(8000, 32, device="cuda:0"))
    a = small.search(q[:1].contiguous(), 10, 2)
    torch.cuda.synchronize()
    small.search(q[:4].contiguous(), 10, 40)  # 8,000 candidates to each of four queries: the slice holds 4,000
    torch.cuda.synchronize()
    assert small.poll_error() == -6
    small.clear_error()
    b = small.search(q[:1].contiguous(), 10, 2)
    torch.cuda.synchronize()
    assert small.poll_error() == 0 and torch.equal(a[0], b[0]) and torch.equal(a[1], b[1])
    small.close()
    g.close()


def test_requests_of_all_kinds_in_turn_on_several_streams():
    print("[case] small path, streams", flush=True)
    g, q = build(40000, 64, 300, "l2", "f32", n_resources=6)
    sizes = [(1, 10, 4), (40, 20, 32), (5, 100, 64), (40, 3, 1), (2, 128, 16)]
    assert [both(g, q[:nq].contiguous(), k, nprobe) for nq, k, nprobe in sizes] == [True, False, True, True, True]
    g.set_param("small_requests", 0)
    want = []
    for nq, k, nprobe in sizes:
        want.append(g.search(q[:nq].contiguous(), k, nprobe))
        torch.cuda.synchronize()
    g.set_param("small_requests", 1)
    streams = [torch.cuda.Stream() for _ in range(4)]
    for turn in range(6):
        got = []
        for j, (nq, k, nprobe) in enumerate(sizes):
            s = streams[(turn + j) % 4]
            with torch.cuda.stream(s):
                got.append(g.search(q[:nq], k, nprobe))
        torch.cuda.synchronize()
        for (a, b), (c, e) in zip(got, want):
            assert torch.equal(a, c) and torch.equal(b, e)
    g.close()
