"""The pruning bound of a query is the k-th best score of a sample of its candidates, whatever k: read back after the
request and compared with the sample taken here, in the order of the exported lists.  Scores are small whole numbers, the
same in every form and order.  What decides the size of a sample: 4 k vectors, 512 at least, a quarter of the nearest list,
1 MiB of them at most (but 512 in any case, and under squared distances a quarter more than k).  Several workgroups that share
a sample do without the 4 k.  A sample of more than one turn of the wavefronts that read it is the nearest number of whole
turns, but no fewer than a quarter more than k or that 1 MiB comes to."""
import pytest
import torch

from paper_2408_02937_amd import rtams

pytestmark = pytest.mark.gpu

NO_BOUND = 0xFFFFFFFF


def workgroups(nq, nprobe):
    """Workgroups that may read a query's sample."""
    pairs = nq * nprobe
    scatterers = 1 if pairs <= 2048 else min(8, (pairs + 2047) // 2048)
    room = (511 - scatterers) // nq
    return 1 if room < 3 else min(4, room)


def sample_groups(k, nearest, chunks, nlist, parts, l2):
    """Groups of 64 vectors of the sample of a query whose nearest list holds `nearest` vectors of `chunks` 16-byte chunks."""
    least = max(512, k + k // 4)
    cap = min(max((1 << 20) // (16 * chunks) // 64 * 64, (least + 63) // 64 * 64 if l2 else 512), 4096)
    want = (min(max(4 * k, nearest // 4, 512), cap) + 63) // 64
    if parts > 1 and (want * chunks < 260 or want * 64 > nlist):
        parts = 1
    if parts > 1:
        want = min(want, (max(least, nearest // 4) + 63) // 64)
    turn = 8 * parts  # eight wavefronts to a workgroup, a group to each in turn
    if want > turn:
        want = min(max((want + turn // 2) // turn * turn, min(want, (least + 63) // 64)), 64)
        if parts > 1:
            want = min(want, nlist // 64)
    return want


def score_of_key(key):
    """What the scan compares: squared distances, or negated inner products."""
    bits = key & 0x7FFFFFFF if key & 0x80000000 else ~key & 0xFFFFFFFF
    return torch.tensor([bits], dtype=torch.int64).to(torch.int32).view(torch.float32).item() if bits < 1 << 31 else \
        torch.tensor([bits - (1 << 32)], dtype=torch.int64).to(torch.int32).view(torch.float32).item()


def build(n, d, nlist, metric, storage, max_batch):
    gen = torch.Generator("cuda:0").manual_seed(n + d + nlist)
    C = torch.randint(0, 16, (nlist, d), device="cuda:0", generator=gen).float()
    if metric == "ip" and storage != "u8":
        C -= 8
    lo, hi = C.min().item(), C.max().item()

    def near(m):
        at = torch.randint(nlist, (m,), device="cuda:0", generator=gen)
        return (C[at] + 2 * torch.randn(m, d, device="cuda:0", generator=gen)).round_().clamp_(lo, hi)

    g = rtams.Index(d, nlist, metric, 64, pool_blocks=n // 64 + 2 * nlist + 64, n_resources=1, max_batch=max_batch, max_k=1024,
                    max_nprobe=32, candidates_per_query=min(n, 65536), storage=storage)
    g.set_centroids(C)
    g.add(near(n))
    return g, near(max_batch)


def check(g, q, k, nprobe, chunks, some):
    metric_ip, nlist, nq = g.metric == rtams.IP, g.nlist, q.shape[0]
    probes = g.probe(q, nprobe).cpu()
    g.search(q, k, nprobe)
    torch.cuda.synchronize()
    assert g.poll_error() == 0
    bounds, kept, path = g.request_trace(nq)
    assert path in ("k_scan", "k_scan_mm")
    sizes = g.list_sizes()
    bounded = 0
    for i in some:
        lists = [int(x) for x in probes[i]]
        groups = sample_groups(k, int(sizes[lists[0]]), chunks, nlist, workgroups(nq, nprobe), not metric_ip)
        scores, left = [], groups
        total = sum(int(sizes[l]) for l in lists)
        for l in lists:
            if not left:
                break
            _, x = g.list_export(l)
            take = min((int(sizes[l]) + 63) // 64, left)
            left -= take
            x = x[:take * 64].double()
            y = q[i].double()
            scores.append(-(x @ y) if metric_ip else ((x - y) ** 2).sum(1))
        s = torch.sort(torch.cat(scores))[0]
        key, n_kept = int(bounds[i]), int(kept[i])
        # (the last group of a list holds fewer than 64 vectors)
        if total <= (max(4096, 32 * g.d) if metric_ip else 4096) or k > len(s):
            assert key == NO_BOUND, f"query {i}"
            continue
        assert key != NO_BOUND, f"query {i}: no bound, k {k}, {groups} groups"
        bound = score_of_key(key)
        kth = s[k - 1].item()
        admitted, tied = int((s <= bound).sum()), int((s <= kth).sum())
        assert bound >= kth and admitted <= max(k + k // 16, tied), f"query {i}: bound {bound}, k-th {kth}, admits {admitted}"
        assert k <= n_kept <= total, f"query {i}"
        bounded += 1
    return bounded


# 256 queries (200: two to each would have room): a workgroup to each.  d 400: 640 vectors are 1 MiB, ten groups
@pytest.mark.parametrize("d,ks", [(400, (100, 200, 512, 513, 600, 640, 700)), (348, (513, 700, 705)), (128, (129, 600, 1024))])
def test_one_workgroup_to_a_sample(d, ks):
    print(f"[case] bound of 256 queries, d {d}", flush=True)
    g, q = build(60_000, d, 40, "l2", "f32", 256)
    g.set_param("scan_mfma", 0)
    for k in ks:
        check(g, q, k, 16, d // 4, range(0, 256, 37))
    check(g, q[:200].contiguous(), ks[-2], 16, d // 4, (0, 199))
    g.close()


# 64 and 100 queries: four and five workgroups' worth of room; the row of scores holds 1,100 keys, 17 groups
@pytest.mark.parametrize("metric", ["l2", "ip"])
@pytest.mark.parametrize("storage,d,ks", [("f32", 300, (10, 200, 240, 513, 600, 800, 832, 900)), ("f16", 560, (200, 600, 900)),
                                          ("u8", 1088, (200, 600, 900))])
def test_shared_samples(storage, d, ks, metric):
    print(f"[case] bound of 64 queries, {metric} {storage} d {d}", flush=True)
    g, q = build(1_300_000 if metric == "ip" and storage != "f32" else 500_000, d, 1100, metric, storage, 100)
    chunks = d // {"f32": 4, "f16": 8, "u8": 16}[storage]
    for mode in (0, 2) if metric == "ip" else (0,):
        g.set_param("scan_mfma", mode)
        for k in ks:
            some = range(0, 64, 13)
            assert check(g, q[:64].contiguous(), k, 32, chunks, some) == len(some) or k > 600  # (not past what the sample holds)
        check(g, q, ks[-1], 32, chunks, (0, 99))
    g.close()
