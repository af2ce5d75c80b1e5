"""Searches that read the halves beside float lists, on streams of their own while insertions run: they see whole batches only."""
import threading
import time

import pytest
import torch

from paper_2408_02937_amd import rtams, synth
from tests.gpu_common import assert_lists_equal, make_pair, whole_batches_check

pytestmark = pytest.mark.gpu


def pair(w, monkeypatch):
    monkeypatch.setattr(rtams, "HALVES_LEAST", 1)
    g, o = make_pair(w, n_resources=8)
    assert g.halves is not None
    g.halves.fill_(0xFF)
    g.set_param("small_requests", 0)
    g.set_param("scan_halves", 2)
    return g, o


# Lists that grow by a block every other batch, and table segments with them.  An item goes as far as its list did when the request
# was planned: what the block table holds beyond that may be anything to a scan that runs meanwhile.
@pytest.mark.parametrize("steal", [0, 1])
@pytest.mark.parametrize("metric", ["l2", "ip"])
def test_a_scan_goes_no_further_than_its_plan(metric, steal, monkeypatch):
    print(f"[case] inserts beside scans of halves, {metric}, steal {steal}", flush=True)
    make = synth.gaussian_l2 if metric == "l2" else synth.unit_ip
    w = make("beside", 81, d=64, n_base=20_000, nlist=16, block_vecs=64, n_queries=64, n_inserts=8_000, insert_batch=160, nprobe=8)
    g, o = pair(w, monkeypatch)
    if steal:  # as long scans, whose workgroups take other dies' items
        g.set_param("scan_exclusive_pairs", 1)
        g.set_param("scan_exclusive_bytes", 1)
    whole_batches_check(w, g, o, 3)
    assert g.request_trace(64)[2] == "k_scan_halves"
    assert_lists_equal(g, o)
    g.close()


# The first vector that is not whole, in the middle of searches: until then all halves are their floats, and a query's finalists are left
# to one workgroup; afterwards several share them.  Whichever a request finds, every query gets all of its answer, the one of before or
# the one of after.
@pytest.mark.parametrize("metric", ["l2", "ip"])
def test_the_first_inexact_vector_beside_searches(metric, monkeypatch):
    print(f"[case] first inexact vector beside searches, {metric}", flush=True)
    monkeypatch.setattr(rtams, "HALVES_LEAST", 1)
    d, nlist, n, nq, k = 512, 16, 20_000, 8, 100
    for turn in range(6):
        gen = torch.Generator("cuda:0").manual_seed(turn)
        centres = (60 * torch.randn(nlist, d, device="cuda:0", generator=gen)).round_()
        x = centres[torch.randint(nlist, (n,), device="cuda:0", generator=gen)] + (20 * torch.randn(n, d, device="cuda:0", generator=gen)).round_()
        q = x[:nq].clone()
        first = q[:1] + (0.3 if metric == "l2" else 0.1 * q[:1])
        g = rtams.Index(d, nlist, metric, 64, pool_blocks=n // 64 + 3 * nlist, n_resources=4, max_batch=nq, max_k=k, max_nprobe=8, candidates_per_query=n)
        g.set_centroids(centres)
        g.add(x)
        g.set_param("small_requests", 0)
        g.set_param("scan_halves", 2)
        before = g.search(q, k, 8)
        torch.cuda.synchronize()
        got, stop = [], threading.Event()

        def searcher():
            s = torch.cuda.Stream()
            while True:
                last = stop.is_set()
                od, oi = torch.full((nq, k), -7.0, device="cuda:0"), torch.full((nq, k), -7, dtype=torch.int64, device="cuda:0")
                torch.cuda.current_stream().synchronize()
                g.search(q, k, 8, od, oi, stream=s)
                s.synchronize()
                got.append((od, oi))
                if last:
                    return

        threads = [threading.Thread(target=searcher) for _ in range(2)]
        for t in threads:
            t.start()
        while len(got) < 6 and all(t.is_alive() for t in threads):
            time.sleep(1e-4)
        data = torch.cuda.Stream()
        g.add(first.contiguous(), stream=data)
        data.synchronize()
        stop.set()
        for t in threads:
            t.join()
        after = g.search(q, k, 8)
        torch.cuda.synchronize()
        assert g.poll_error() == 0 and g.request_trace(nq)[2] == "k_scan_halves"
        assert not torch.equal(before[1], after[1])
        for od, oi in got:
            for r in range(nq):
                assert any(torch.equal(od[r], w[0][r]) and torch.equal(oi[r], w[1][r]) for w in (before, after)), (turn, r, oi[r])
        g.set_param("scan_halves", 0)
        want = g.search(q, k, 8)
        torch.cuda.synchronize()
        assert torch.equal(want[0], after[0]) and torch.equal(want[1], after[1])
        g.close()
