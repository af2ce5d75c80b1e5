"""Insertion calls on different streams in turn, with nothing but the library's own event between them: every batch finds
what the batches before it left, whatever stream they ran on, also where rearrangements follow."""
import pytest
import torch

from paper_2408_02937_amd import synth
from tests.gpu_common import assert_lists_equal, dev, make_pair
from tests.helpers import assert_topk_matches, RTOL

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("batch,threshold", [(1, 0), (64, 0), (64, 600), (700, 0), (2000, 0)])
def test_batches_from_streams_in_turn(batch, threshold):
    print(f"[case] streams in turn, batches of {batch}, threshold {threshold}", flush=True)
    total = min(60 * batch, 20_000)
    w = synth.gaussian_l2("turn", 5, n_base=3_000, n_queries=32, n_inserts=total, insert_batch=batch, nlist=32, block_vecs=64)
    g, o = make_pair(w, pool_blocks=2_000, rearrange_threshold=threshold)
    y = dev(w.inserts)
    base = dev(w.base)
    torch.cuda.synchronize()
    streams = [torch.cuda.Stream() for _ in range(3)]
    with torch.cuda.stream(streams[2]):
        g.add(base)
    o.add(w.base)
    for i, at in enumerate(range(0, total, batch)):
        with torch.cuda.stream(streams[i % 3]):
            g.add(y[at:at + batch])
        o.add(w.inserts[at:at + batch])
    torch.cuda.synchronize()
    assert g.poll_error() == 0
    g.validate()
    assert_lists_equal(g, o)
    rd, ri = o.search(w.queries, 10, 8)
    dd, ii = g.search(dev(w.queries), 10, 8)
    assert_topk_matches("l2", dd.cpu().numpy(), ii.cpu().numpy(), rd, ri, rtol=RTOL, atol=1e-5)
    g.close()
