"""Probes behind the matrix-core filter right up to what a request may ask for: the lists of the exact arithmetic in its order,
and no fall in speed before the candidates of the filter really are too many for LDS."""
import pytest
import torch

from paper_2408_02937_amd import rtams

pytestmark = pytest.mark.gpu


def build(nlist, d):
    gen = torch.Generator("cuda:0").manual_seed(nlist + d)
    C = torch.rand(nlist, d, device="cuda:0", generator=gen) * 128
    g = rtams.Index(d, nlist, "l2", 64, pool_blocks=nlist, n_resources=8, max_batch=256, max_k=16, max_nprobe=1024,
                    candidates_per_query=1024)
    g.set_centroids(C)
    q = C[torch.randint(nlist, (256,), device="cuda:0", generator=gen)] + 8 * torch.randn(256, d, device="cuda:0", generator=gen)
    return g, q


@pytest.mark.parametrize("nlist,d", [(4096, 128), (16384, 64)])
def test_the_lists_of_many_probes(nlist, d):
    print(f"[case] many probes of {nlist} lists", flush=True)
    g, q = build(nlist, d)
    for nprobe in (455, 456, 910, 980, 1010, 1024):
        got = {}
        for mode in (0, 2):  # without the filter, behind it
            g.set_param("use_mfma", mode)
            got[mode] = g.probe(q, nprobe)
            torch.cuda.synchronize()
        assert torch.equal(got[0], got[2]), nprobe
    g.close()


def test_no_fall_in_speed_short_of_what_fits():
    """980 probes take little longer than 900.  (A threshold that admits an eighth more lists than asked for sent them down
    the path for bands too wide for LDS: 243 us against 105.)"""
    g, q = build(16384, 64)
    g.set_param("use_mfma", 2)

    def shortest(nprobe):
        best = 1e9
        for _ in range(4):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            g.probe(q, nprobe)
            torch.cuda.synchronize()
            a.record()
            for _ in range(5):
                g.probe(q, nprobe)
            b.record()
            torch.cuda.synchronize()
            best = min(best, a.elapsed_time(b) / 5)
        return best

    at_900, at_980 = shortest(900), shortest(980)
    print(f"[case] 900 probes {at_900 * 1e3:.0f} us, 980 {at_980 * 1e3:.0f}", flush=True)
    assert at_980 < 1.4 * at_900
    g.close()
