"""The scan of the halves beside float lists says which vectors are scored, never what is returned: the same bits as the
request has without it, whichever unit that takes.  The halves' memory starts as NaNs."""
import pytest
import torch

from paper_2408_02937_amd import rtams

pytestmark = pytest.mark.gpu

DEV = "cuda:0"


def index(d, nlist, metric, block_vecs, n, nprobe, monkeypatch, threshold=0, resources=1):
    monkeypatch.setattr(rtams, "HALVES_LEAST", 1)
    g = rtams.Index(d, nlist, metric, block_vecs, pool_blocks=n // block_vecs + 3 * nlist + 64, n_resources=resources, max_batch=256, max_k=1024,
                    max_nprobe=nprobe, candidates_per_query=n, rearrange_threshold=threshold)
    assert g.halves is not None
    g.halves.fill_(0xFF)
    return g


def both(g, q, k, nprobe):
    g.set_param("small_requests", 0)
    g.set_param("scan_halves", 0)
    want = g.search(q, k, nprobe)
    torch.cuda.synchronize()
    g.set_param("scan_halves", 2)
    got = g.search(q, k, nprobe)
    torch.cuda.synchronize()
    assert g.poll_error() == 0
    path = g.request_trace(q.shape[0])[2]
    assert path == "k_scan_halves"
    return want, got


def same(want, got, finite_only=False):
    (d0, i0), (d1, i1) = want, got
    if finite_only:  # (the order of infinitely far ones and of NaNs is left open)
        ok = torch.isfinite(d0)
        assert torch.equal(ok, torch.isfinite(d1))
        assert torch.equal(d0[ok], d1[ok]) and torch.equal(i0[ok], i1[ok])
        return
    assert torch.equal(d0.view(torch.int32), d1.view(torch.int32))
    assert torch.equal(i0, i1)


# dimensions: one chunk of halves, a chunk half filled, whole steps and a rest of one to three chunks, 64 coordinates and their
# neighbours, the widest; tiles of 16 and 32 queries and one more; k of one, and more than the sample's first size
@pytest.mark.parametrize("metric", ["l2", "ip"])
@pytest.mark.parametrize("d,nlist,block_vecs,nq,nprobe,k", [
    (4, 16, 64, 1, 16, 1), (12, 17, 128, 16, 5, 10), (32, 64, 64, 17, 8, 100), (36, 33, 192, 33, 33, 128), (64, 64, 128, 256, 64, 50),
    (100, 40, 64, 64, 20, 1000), (128, 64, 256, 256, 32, 100), (260, 20, 64, 7, 20, 600), (768, 100, 128, 64, 8, 10), (2048, 16, 64, 40, 16, 100)])
@pytest.mark.parametrize("whole", [False, True])
def test_the_same_bits_as_the_floats_alone(metric, d, nlist, block_vecs, nq, nprobe, k, whole, monkeypatch):
    print(f"[case] halves {metric} d {d}, {nq} x {nprobe}, k {k}, whole {whole}", flush=True)
    gen = torch.Generator(DEV).manual_seed(d + nq)
    n = min(60_000, 20_000_000 // d)
    centres = torch.randn(nlist, d, device=DEV, generator=gen)

    def rows(m):
        # a few lists hold one to 70 vectors: ends of units, of groups and of blocks
        at = torch.cat([torch.arange(min(nlist, 8), device=DEV).repeat_interleave(torch.tensor([1, 31, 32, 33, 63, 64, 65, 70][:min(nlist, 8)], device=DEV))[:m],
                        torch.randint(8 if nlist > 16 else 0, nlist, (max(0, m - 359),), device=DEV, generator=gen)])[:m]
        x = centres[at] + 0.2 * torch.randn(len(at), d, device=DEV, generator=gen)
        return (60 * x).round_() if whole else x  # (whole numbers: their halves are their floats)

    g = index(d, nlist, metric, block_vecs, n, nprobe, monkeypatch)
    g.set_centroids((60 * centres).round_() if whole else centres)
    x = rows(n)
    for piece in (x[:1], x[1:70], x[70:2000], x[2000:]):  # the tail, by vector and by lists
        g.add(piece.contiguous())
    q = rows(max(nq, 359))[-nq:].contiguous()
    same(*both(g, q, k, nprobe))
    for steal in (1, 0):  # as a long scan, whose workgroups take other dies' items
        g.set_param("scan_exclusive_pairs", steal)
        g.set_param("scan_exclusive_bytes", 1 if steal else 16 << 30)
        same(*both(g, q, k, nprobe))
    g.close()


# finalists by the thousand and queries whose workgroups share them; vectors that no half can tell apart
@pytest.mark.parametrize("metric", ["l2", "ip"])
@pytest.mark.parametrize("spread,nq,k", [(0.1, 8, 50), (0.1, 128, 100), (0.1, 130, 100), (1e-4, 8, 10), (0.0, 24, 300)])
def test_shared_and_many_finalists(metric, spread, nq, k, monkeypatch):
    print(f"[case] finalists {metric}, spread {spread}, {nq} queries, k {k}", flush=True)
    gen = torch.Generator(DEV).manual_seed(nq)
    d, nlist, n = 512, 16, 40_000
    centres = torch.randn(nlist, d, device=DEV, generator=gen)
    x = centres[torch.randint(nlist, (n,), device=DEV, generator=gen)] + spread * torch.randn(n, d, device=DEV, generator=gen)
    g = index(d, nlist, metric, 128, n, nlist, monkeypatch)
    g.set_centroids(centres)
    g.add(x)
    q = (x[:nq] + spread * torch.randn(nq, d, device=DEV, generator=gen)).contiguous()
    for nprobe in (2, nlist):
        same(*both(g, q, k, nprobe))
    g.close()


@pytest.mark.parametrize("metric", ["l2", "ip"])
def test_what_halves_cannot_hold_is_scored(metric, monkeypatch):
    print(f"[case] infinities and large values, {metric}", flush=True)
    gen = torch.Generator(DEV).manual_seed(3)
    d, nlist, n = 96, 32, 20_000
    centres = torch.randn(nlist, d, device=DEV, generator=gen)
    x = centres[torch.randint(nlist, (n,), device=DEV, generator=gen)] + 0.1 * torch.randn(n, d, device=DEV, generator=gen)
    x[::97] *= 1e4      # past the largest half
    x[1::101] *= 1e-9   # below the smallest
    x[5] = float("inf")
    x[7, 3] = float("nan")
    q = x[100:140].clone()
    q[2] *= 1e25
    q[3] = float("nan")
    q[4] = 0.0
    g = index(d, nlist, metric, 64, n, nlist, monkeypatch)
    g.set_centroids(centres)
    g.add(x)
    same(*both(g, q, 20, nlist), finite_only=True)
    g.close()


def test_the_halves_move_with_their_blocks_and_grow_with_the_lists(monkeypatch):
    print("[case] rearrangement", flush=True)
    gen = torch.Generator(DEV).manual_seed(4)
    d, nlist, n = 100, 24, 30_000
    centres = torch.randn(nlist, d, device=DEV, generator=gen)
    x = centres[torch.randint(nlist, (n,), device=DEV, generator=gen)] + 0.3 * torch.randn(n, d, device=DEV, generator=gen)
    g = index(d, nlist, "l2", 64, n, nlist, monkeypatch, threshold=300)
    g.set_centroids(centres)
    for lo in range(0, n, 777):
        g.add(x[lo:lo + 777].contiguous())
    for _ in range(2):
        same(*both(g, x[:50].contiguous(), 60, 6))
        g.rearrange(-1)
        torch.cuda.synchronize()
        g.validate()
    g.close()


def test_recorded_requests_read_them_too(monkeypatch):
    print("[case] recorded", flush=True)
    gen = torch.Generator(DEV).manual_seed(5)
    d, nlist, n, nq, k = 128, 64, 50_000, 96, 40
    centres = torch.randn(nlist, d, device=DEV, generator=gen)
    x = centres[torch.randint(nlist, (n,), device=DEV, generator=gen)] + 0.2 * torch.randn(n, d, device=DEV, generator=gen)
    g = index(d, nlist, "ip", 128, n, 16, monkeypatch, resources=4)
    g.set_centroids(centres)
    g.add(x)
    q = x[:nq].clone()
    _, want = both(g, q, k, 16)
    od, oi = torch.empty(nq, k, device=DEV), torch.empty(nq, k, dtype=torch.int64, device=DEV)
    torch.cuda.synchronize()
    s = torch.cuda.Stream()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=s):
        g.search(q, k, 16, od, oi)
    for turn in range(4):
        q.copy_(x[turn * 100:turn * 100 + nq])
        want = g.search(q, k, 16)
        torch.cuda.synchronize()
        od.zero_()
        graph.replay()
        torch.cuda.synchronize()
        same(want, (od, oi))
    with pytest.raises(rtams.RtamsError) as e:  # the graph may be launched again
        g.drop_halves()
    assert e.value.code == rtams.ESTATE
    g.close()


# metric, d, lists, vectors of a list, queries, probes, k, which scan takes it
@pytest.mark.parametrize("metric,d,nlist,length,nq,nprobe,k,path", [
    ("l2", 128, 64, 4000, 8, 32, 10, "k_scan_halves"),    # 133 MB of lists, 525 that the pairs meet, of which a fifth: 238 of 133
    ("l2", 128, 64, 4000, 7, 64, 10, "k_scan"),           # fewer than eight queries
    ("l2", 128, 64, 1000, 64, 32, 10, "k_scan_halves"),   # 33 MB, and 1,050 that the pairs meet
    ("l2", 128, 64, 1000, 8, 32, 10, "k_scan"),           # 33 and 131
    ("ip", 128, 64, 6000, 64, 32, 10, "k_scan_halves"),   # 199.7 MB of 199.1
    ("ip", 128, 64, 4000, 64, 32, 10, "k_scan"),          # 133
])
def test_which_requests_read_them(metric, d, nlist, length, nq, nprobe, k, path, monkeypatch):
    monkeypatch.setattr(rtams, "HALVES_LEAST", 1)
    gen = torch.Generator(DEV).manual_seed(6)
    centres = torch.randn(nlist, d, device=DEV, generator=gen)
    centres *= 8.0 * d ** 0.5 / centres.norm(dim=1, keepdim=True)
    x = centres.repeat_interleave(length, 0) + 0.5 * torch.randn(nlist * length, d, device=DEV, generator=gen)
    g = rtams.Index(d, nlist, metric, 128, pool_blocks=len(x) // 128 + 2 * nlist + 8, n_resources=1, max_batch=256, max_k=16, max_nprobe=nprobe,
                    candidates_per_query=len(x))
    g.set_centroids(centres)
    g.add(x)
    q = x[::97][:nq].contiguous()
    g.set_param("small_requests", 0)
    torch.cuda.synchronize()
    g.search(q, k, nprobe)
    torch.cuda.synchronize()
    assert g.request_trace(nq)[2] == path
    g.close()


# Queries so far away that halves cannot tell their candidates apart: the rule leaves the next 1,024 requests to the floats, whatever they ask
def test_halves_that_tell_nothing_get_a_rest(monkeypatch):
    print("[case] a rest", flush=True)
    monkeypatch.setattr(rtams, "HALVES_LEAST", 1)
    gen = torch.Generator(DEV).manual_seed(11)
    d, nlist, length, nq, nprobe = 128, 64, 4000, 8, 32
    centres = torch.randn(nlist, d, device=DEV, generator=gen)
    x = centres.repeat_interleave(length, 0) + 0.3 * torch.randn(nlist * length, d, device=DEV, generator=gen)
    g = rtams.Index(d, nlist, "l2", 128, pool_blocks=len(x) // 128 + 2 * nlist + 8, n_resources=1, max_batch=nq, max_k=16, max_nprobe=nprobe,
                    candidates_per_query=len(x))
    g.set_centroids(centres)
    g.add(x)
    g.set_param("small_requests", 0)
    torch.cuda.synchronize()
    near, far = x[::31999][:nq].contiguous(), 1e3 * x[::31999][:nq].contiguous()

    def search(q):
        out = g.search(q, 10, nprobe)
        torch.cuda.synchronize()
        return g.request_trace(nq)[2], out

    assert [search(near)[0] for _ in range(3)] == ["k_scan_halves"] * 3  # these are told apart
    path, first = search(far)
    assert path == "k_scan_halves" and g.request_trace(nq)[1].to(torch.int64).max() > 2048
    path, again = search(far)
    assert path == "k_scan"
    same(first, again)
    assert {search(near)[0] for _ in range(1023)} == {"k_scan"}
    assert search(near)[0] == "k_scan_halves"
    g.close()


def test_timed_scans_of_halves_are_counted_as_such(monkeypatch):
    gen = torch.Generator(DEV).manual_seed(10)
    d, nlist, n = 64, 16, 5000
    x = torch.randn(n, d, device=DEV, generator=gen)
    g = index(d, nlist, "l2", 64, n, 8, monkeypatch)
    g.set_centroids(x[:nlist].contiguous())
    g.add(x)
    g.set_param("small_requests", 0)
    g.set_param("profile_scan", 1)
    for halves, mfma, name in ((2, 1, "k_scan_halves"), (2, 2, "k_scan_halves"), (0, 2, "k_scan_mm"), (0, 0, "k_scan")):
        g.set_param("scan_halves", halves)
        g.set_param("scan_mfma", mfma)
        for _ in range(2):
            g.search(x[:64].contiguous(), 5, 8)
            torch.cuda.synchronize()
        assert g.scan_kernels()[name] == 2
        got = g.scan_kernels(reset=True)
        assert got.pop(name) == 2 and not any(got.values()), (name, got)
    g.close()


def test_whether_an_index_keeps_halves_is_its_callers_choice(monkeypatch):
    print("[case] kept, declined and given back", flush=True)
    kw = dict(block_vecs=64, pool_blocks=500, n_resources=2, max_batch=64, max_k=10, max_nprobe=8, candidates_per_query=10_000)
    gen = torch.Generator(DEV).manual_seed(12)
    x, q = torch.randn(10_000, 32, device=DEV, generator=gen), torch.randn(64, 32, device=DEV, generator=gen)

    def filled(**more):
        g = rtams.Index(32, 64, "l2", **kw, **more)
        g.set_centroids(x[:64].contiguous())
        g.add(x)
        g.set_param("scan_halves", 2)
        g.set_param("small_requests", 0)
        return g

    def search(g):
        out = g.search(q, 10, 8)
        torch.cuda.synchronize()
        return g.request_trace(64)[2], out

    with pytest.raises(ValueError):
        rtams.Index(32, 64, "l2", **kw, storage="f16", halves=True)
    plain = filled()
    assert plain.halves_bytes == 0  # too few for any scan of them to be long ...
    with pytest.raises(rtams.RtamsError) as e:
        plain.drop_halves()
    assert e.value.code == rtams.ESTATE
    kept = filled(halves=True)      # ... but for whoever wants them
    assert kept.halves_bytes == rtams.lib().rtams_halves_bytes(kept._h) > 0
    monkeypatch.setattr(rtams, "HALVES_LEAST", 1)
    with_rule, declined = filled(), filled(halves=False)
    assert with_rule.halves_bytes == kept.halves_bytes and declined.halves_bytes == 0
    path, want = search(declined)
    assert path == "k_scan_mm"
    same(want, search(plain)[1])
    for g in (kept, with_rule):
        path, got = search(g)
        assert path == "k_scan_halves"
        same(want, got)
    before = torch.cuda.memory_allocated()
    nbytes = kept.halves_bytes
    kept.drop_halves()
    assert kept.halves_bytes == 0 and torch.cuda.memory_allocated() <= before - nbytes
    path, got = search(kept)
    assert path == "k_scan_mm"
    same(want, got)
    more = torch.randn(3000, 32, device=DEV, generator=gen)
    for g in (kept, with_rule):
        g.add(more)
        g.rearrange(-1)
    torch.cuda.synchronize()
    same(search(with_rule)[1], search(kept)[1])
    kept.validate()
    for g in (plain, kept, with_rule, declined):
        g.close()


# (the allocation that fails is made to: nothing here fills the device)
def test_halves_that_nobody_asked_for_make_room_for_an_index(monkeypatch):
    print("[case] room for an index", flush=True)
    monkeypatch.setattr(rtams, "HALVES_LEAST", 1)
    kw = dict(block_vecs=64, pool_blocks=500, n_resources=2, max_batch=64, max_k=10, max_nprobe=8, candidates_per_query=10_000)
    gen = torch.Generator(DEV).manual_seed(13)
    x = torch.randn(10_000, 32, device=DEV, generator=gen)
    q = x[:64].contiguous()

    def filled(**more):
        g = rtams.Index(32, 64, "l2", **kw, **more)
        g.set_centroids(x[:64].contiguous())
        g.add(x)
        g.set_param("scan_halves", 2)
        g.set_param("small_requests", 0)
        torch.cuda.synchronize()
        return g

    by_rule, asked = filled(), filled(halves=True)
    recorded = filled()
    od, oi = torch.empty(64, 10, device=DEV), torch.empty(64, 10, dtype=torch.int64, device=DEV)
    recorded.search(q, 10, 8)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        recorded.search(q, 10, 8, od, oi)
    want = by_rule.search(q, 10, 8)
    torch.cuda.synchronize()
    real, failed = torch.empty, []

    def empty(*a, **k):
        if k.get("dtype") is torch.uint8 and not failed:
            failed.append(a)
            raise torch.OutOfMemoryError("no memory left")
        return real(*a, **k)

    monkeypatch.setattr(rtams.torch, "empty", empty)
    g = rtams.Index(32, 64, "l2", **kw, halves=False)
    monkeypatch.setattr(rtams.torch, "empty", real)
    assert failed and by_rule.halves_bytes == 0 and asked.halves_bytes > 0 and recorded.halves_bytes > 0 and g.halves_bytes == 0
    same(want, by_rule.search(q, 10, 8))
    graph.replay()
    torch.cuda.synchronize()
    same(want, (od, oi))
    for ix in (by_rule, asked, recorded, g):
        ix.close()


def test_who_keeps_halves_and_when_they_are_taken():
    L = rtams.lib()
    kinds = {"f32": (64, {}), "16 lists": (16, {}), "15 lists": (15, {}), "f16": (64, dict(storage="f16")), "u8": (64, dict(storage="u8")), "pq": (64, dict(pq_m=8))}
    for name, (nlist, more) in kinds.items():
        g = rtams.Index(32, nlist, "l2", 64, pool_blocks=200, n_resources=1, max_batch=8, max_k=8, max_nprobe=8, candidates_per_query=1000, **more)
        want = L.rtams_halves_bytes(g._h)
        assert want == (g.pool_stats().blocks_total * 64 * 64 if name in ("f32", "16 lists") else 0), name
        if not want:
            t = torch.empty(1 << 20, dtype=torch.uint8, device=DEV)
            assert L.rtams_set_halves(g._h, t.data_ptr(), 1 << 20) == rtams.ESTATE, name
        g.close()
    g = rtams.Index(32, 64, "l2", 64, pool_blocks=200, n_resources=1, max_batch=8, max_k=8, max_nprobe=8, candidates_per_query=1000)
    assert g.halves is None  # too few for any scan of them to be long
    want = L.rtams_halves_bytes(g._h)
    t = torch.empty(want + 256, dtype=torch.uint8, device=DEV)
    assert L.rtams_set_halves(g._h, None, want) == rtams.EINVAL
    assert L.rtams_set_halves(g._h, t.data_ptr() + 16, want) == rtams.EINVAL
    assert L.rtams_set_halves(g._h, t.data_ptr(), want - 1) == rtams.EINVAL
    x = torch.randn(500, 32, device=DEV)
    g.set_centroids(x[:64].contiguous())
    assert L.rtams_set_halves(g._h, t.data_ptr(), want) == rtams.OK
    g.add(x)
    assert L.rtams_set_halves(g._h, t.data_ptr(), want) == rtams.ESTATE
    torch.cuda.synchronize()
    g.close()


# A query's workgroups take a limit from whichever of its records they come by first, and need not take the same.  Here some 1,060 of the
# first 4,096 records share the first digit of their scores (inner products from 128 to 512), more than the 1,024 that are scored for
# a limit.  The last of them, below 256, decides whether the digits of the next selection are of one or of two: a threshold of 259 or of
# 258, with inner products closer to 259 than halves tell apart, some of them among the 1,000 best, on either side of it.
# (Two of these 64 fail where a workgroup leaves out what lies below its own threshold.)
@pytest.mark.parametrize("sixteen", range(4))
def test_workgroups_of_a_query_with_limits_of_their_own(sixteen, monkeypatch):
    for seed in range(16 * sixteen, 16 * sixteen + 16):
        print(f"[case] limits of their own, seed {seed}", flush=True)
        limits_of_their_own(seed, monkeypatch)


def limits_of_their_own(seed, monkeypatch):
    d, nlist, nq, k, top = 64, 16, 32, 1000, 1200
    gen = torch.Generator(DEV).manual_seed(seed)

    def between(m, lo, hi):
        return lo + (hi - lo) * torch.rand(m, device=DEV, generator=gen)

    x = 0.02 * torch.randn(4700 + 3096, d, device=DEV, generator=gen)
    x[:, :3] = 0.0
    axis = torch.zeros(d, device=DEV)
    axis[3:6] = 3 ** -0.5
    norm = 115.5 * 3 ** 0.5  # of the query, whose halves are its floats
    x -= (x @ axis)[:, None] * axis
    x[:, 0] = 0.3
    margin = 1.002 * norm * (4.888e-4 + (d + d // 64 + 140) * 6.0e-8)  # of a vector of length 1: what a score of halves is below the inner product's negative
    edge = 259 - margin * ((259 / norm) ** 2 + 0.09 + 0.02 ** 2 * 60) ** 0.5
    best = torch.cat([between(950, 300, 400), between(40, 259.2, 262), between(20, edge - 0.02, edge + 0.06), between(8, 258.1, 258.6),
                      between(top - 1019, 256.2, 257.4), between(1, 255.4, 255.5)])[torch.randperm(top, device=DEV, generator=gen)]
    rest, out = between(4700 - top, -20, 100), between(3096, -80, -30)
    near = torch.cat([best[:300], rest[:700], out])  # the nearest list, which the sample is of
    far = torch.cat([best[300:], rest[700:]])
    ips = torch.cat([near[torch.randperm(len(near), device=DEV, generator=gen)], far[torch.randperm(len(far), device=DEV, generator=gen)]])
    x[:len(near), 1], x[:len(near), 0] = 0.3, 0.0
    x += ips[:, None] / norm * axis
    centres = 0.01 * torch.randn(nlist, d, device=DEV, generator=gen)
    centres[0] += axis
    centres[0, 1], centres[1, 0] = 100.0, 100.0
    g = index(d, nlist, "ip", 64, len(x), nlist, monkeypatch)
    g.set_centroids(centres)
    g.add(x)
    q = torch.zeros(nq, d, device=DEV)
    q[:, 3:6] = 115.5
    want, got = both(g, q, k, nlist)
    kept = g.request_trace(nq)[1].to(torch.int64)
    assert kept.min() > 4096 and want[0][:, -1].min() > 258.7, (kept, want[0][:, -1])
    same(want, got)
    g.close()


# Coordinates that vanish under the scale of the halves: one centroid is so large that all others' vectors are zero there
def test_vectors_that_vanish_under_the_scale(monkeypatch):
    print("[case] vectors that vanish under the scale", flush=True)
    gen = torch.Generator(DEV).manual_seed(8)
    d, nlist, n = 64, 16, 4000
    centres = 1e-20 * torch.randn(nlist, d, device=DEV, generator=gen)
    centres[0] = 2.0 ** 100
    x = centres[1 + torch.randint(nlist - 1, (n,), device=DEV, generator=gen)] + 1e-21 * torch.randn(n, d, device=DEV, generator=gen)
    g = index(d, nlist, "ip", 64, n, nlist, monkeypatch)
    g.set_centroids(centres)
    g.add(x)
    q = 1e18 * torch.randn(8, d, device=DEV, generator=gen)
    want, got = both(g, q, 10, nlist)
    assert want[0].abs().min() > 0
    same(want, got)
    g.close()


# Queries so short that their squares, or those of what their halves leave out, are zero in 32 bits
@pytest.mark.parametrize("metric", ["l2", "ip"])
@pytest.mark.parametrize("size", [1e-17, 1e-20, 1e-22, 1e-24, 1e-30])
@pytest.mark.parametrize("whole", [False, True])
def test_short_queries(metric, size, whole, monkeypatch):
    print(f"[case] queries of {size}, {metric}, whole {whole}", flush=True)
    gen = torch.Generator(DEV).manual_seed(9)
    d, nlist, n = 128, 16, 20_000
    centres = 60 * torch.randn(nlist, d, device=DEV, generator=gen)
    x = centres[torch.randint(nlist, (n,), device=DEV, generator=gen)] + 20 * torch.randn(n, d, device=DEV, generator=gen)
    x = x.round_() if whole else x
    g = index(d, nlist, metric, 64, n, nlist, monkeypatch)
    g.set_centroids(centres)
    g.add(x)
    same(*both(g, size * torch.randn(40, d, device=DEV, generator=gen), 100, 8))
    g.close()
