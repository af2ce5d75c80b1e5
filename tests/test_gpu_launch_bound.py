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


def scan_ms(g, q, k, nprobe):
    g.scan_time(reset=True)
    out = g.search(q, k, nprobe)
    torch.cuda.synchronize()
    ms, launches = g.scan_time()
    assert launches == 1
    return ms, out


# 256 queries in 8 tiles a list: segments of 512 groups of 64 vectors are 6 to a list, 528 items in all, two to a compute
# unit and a few more; segments of 256 groups would be more than 1,024 items
LONG = [6 * 512 * 64] * 11


def test_a_search_behind_an_unfinished_load_is_launched_for_its_lists():
    """The first search behind a bulk load that is still running scans as fast as the same search later.  (Launched for
    what the host knew of the empty index it was cut into 1,024 items at most, sixteen times as long as they need be, and took a fifth longer.)"""
    ratios = []
    for seed in range(5):
        g, y = lists_of(LONG, 32, seed, candidates_per_query=sum(LONG), n_resources=1)
        q = y[:256].contiguous()
        g.set_param("profile_scan", 1)
        torch.cuda.synchronize()
        g.add(y)
        behind, first = scan_ms(g, q, 10, len(LONG))
        after = []
        for _ in range(5):
            t, again = scan_ms(g, q, 10, len(LONG))
            after.append(t)
            assert torch.equal(first[0], again[0]) and torch.equal(first[1], again[1])
        ratios.append(behind / np.median(after))
        assert g.poll_error() == 0
        g.close()
    print(f"[case] scan behind the load against later: {ratios}", flush=True)
    # measured 1.00 to 1.02, and 1.12 to 1.17 launched for the empty index
    assert np.median(ratios) < 1.07


def test_a_recorded_search_fits_lists_that_grow_between_its_replays():
    """A request on the library's static scratch recorded into a graph over an index of a few vectors and replayed
    while its lists grow to hundreds of groups: the eager answers every time."""
    g, y = lists_of([13_000] * 64, 32, 5, candidates_per_query=16 * 13_000)
    nq, k, nprobe = 16, 10, 16
    q = y[-nq:].contiguous()
    d = torch.empty((nq, k), dtype=torch.float32, device="cuda:0")
    i = torch.empty((nq, k), dtype=torch.int64, device="cuda:0")
    g.add(y[:2000])
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        g.search_noalloc(q, k, nprobe, d, i)
    at = 2000
    for more in (0, 1, 30_000, len(y)):
        if more:
            g.add(y[at:at + more])
            at += more
        for _ in range(2):
            d.zero_(); i.zero_()
            rd, ri = g.search(q, k, nprobe)
            graph.replay()
            torch.cuda.synchronize()
            assert g.poll_error() == 0
            assert torch.equal(d, rd) and torch.equal(i, ri)
    del graph
    g.close()


@pytest.mark.parametrize("storage", ["f32", "f16", "u8"])
def test_one_group_at_a_time_through_a_list_of_thousands(storage):
    """Lists short enough on average to be walked a group at a time, and one of 31,000 groups among them: its segments
    get longer until they fit, and its queries' neighbours are those of 64-bit arithmetic."""
    d, hot = 16, 2_000_000
    lengths = [20] * 11_999 + [hot]
    rng = np.random.default_rng(3)
    C = rng.uniform(0, 255, (len(lengths), d)).astype(np.float32)
    C[-1] = 128.0
    C[:-1][np.abs(C[:-1] - 128.0).max(axis=1) < 60] = 255.0  # nobody else near the long list's centroid
    cd = torch.from_numpy(C).cuda()
    at = torch.from_numpy(rng.permutation(np.repeat(np.arange(len(lengths)), lengths))).cuda()
    y = cd[at] + torch.randn(len(at), d, device="cuda:0", generator=torch.Generator("cuda:0").manual_seed(3))
    y.round_().clamp_(0.0, 255.0)  # whole numbers: the same in every kind of list, sums exact
    g = rtams.Index(d, len(lengths), "l2", 64, pool_blocks=len(at) // 64 + 2 * len(lengths) + 8, n_resources=1,
                    max_batch=8, max_k=100, max_nprobe=8, candidates_per_query=hot + 100_000, storage=storage)
    g.set_centroids(cd)
    g.add(y)
    mine = torch.nonzero(g.assign(y) == len(lengths) - 1).flatten()
    assert len(mine) > 0.9 * hot
    q = cd[-1:] + torch.tensor([[0.0], [1.0], [2.0], [-3.0]], device="cuda:0")
    for nq, nprobe in ((1, 1), (4, 8), (2, 3)):
        dist, _ = g.search(q[:nq].contiguous(), 100, nprobe)
        want = torch.stack([torch.sort(((y[mine] - x) ** 2).double().sum(1))[0][:100] for x in q[:nq]])
        assert g.poll_error() == 0
        assert torch.equal(dist.double(), want), f"{storage} {nq} x {nprobe}"
    g.close()
