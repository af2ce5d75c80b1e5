"""The selection where a query has about as many records as are sorted without a threshold: k, up to sixteen more, one past
that, at the smallest and the largest k; distances that differ, that tie in pairs, and that are all alike."""
import pytest
import torch

from paper_2408_02937_amd import rtams

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("metric", ["l2", "ip"])
@pytest.mark.parametrize("kind", ["apart", "pairs", "alike"])
@pytest.mark.parametrize("k", [1, 16, 100, 1007, 1008, 1024])
def test_a_few_more_records_than_k(k, kind, metric):
    print(f"[case] selection edges {metric} k={k} {kind}", flush=True)
    d, gen = 16, torch.Generator("cuda:0").manual_seed(k)
    for more in (-1, 0, 1, 15, 16, 17, 18):
        n = k + more
        if n < 1:
            continue
        g = rtams.Index(d, 1, metric, 64, pool_blocks=n // 64 + 4, n_resources=1, max_batch=4, max_k=1024, max_nprobe=1,
                        candidates_per_query=n)
        g.set_centroids(torch.zeros(1, d, device="cuda:0"))
        order = torch.randperm(n, device="cuda:0", generator=gen)
        y = torch.zeros(n, d, device="cuda:0")  # one coordinate: whole numbers, exact in every form
        y[:, 5] = {"apart": order, "pairs": order // 2, "alike": torch.full_like(order, 3)}[kind].float()
        ids = torch.randperm(10 * n, device="cuda:0", generator=gen)[:n] + (1 << 33)
        g.add(y, ids)
        q = torch.zeros(2, d, device="cuda:0")
        q[:, 5] = 0.0 if metric == "l2" else -1.0
        score = (y[:, 5] ** 2 if metric == "l2" else y[:, 5]).double()
        by = sorted(zip(score.tolist(), ids.tolist()))[:k]
        want_ids = [x[1] for x in by] + [-1] * (k - len(by))
        want = [x[0] if metric == "l2" else -x[0] for x in by]
        for mode in (0, 2):
            g.set_param("scan_mfma", mode)
            dist, got = g.search(q, k, 1)
            torch.cuda.synchronize()
            for i in range(2):
                assert got[i].tolist() == want_ids, f"{n} records, unit {mode}"
                assert dist[i, :len(by)].tolist() == want
        g.close()
