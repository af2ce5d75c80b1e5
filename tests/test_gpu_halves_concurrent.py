"""Searches that read the halves beside float lists, on streams of their own while insertions run: they see whole batches only."""
import pytest

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
