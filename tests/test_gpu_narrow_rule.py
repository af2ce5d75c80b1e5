"""Which instructions scan a request for squared distances over lists of halves and bytes, on both sides of the lines of the
rule (pairs to a list, bytes of the lists, chunks of a vector), and that the answers are those of the vector unit."""
import pytest
import torch

from paper_2408_02937_amd import rtams

pytestmark = pytest.mark.gpu

WIDE, NARROW = "k_scan_mm", "k_scan_mm narrow"


@pytest.mark.parametrize("storage,d,length,nq,nprobe,path", [
    ("f16", 64, 600, 128, 2, WIDE),       # four pairs to a list, 5 MB of lists
    ("f16", 64, 600, 128, 3, NARROW),     # six
    ("f16", 128, 600, 128, 2, NARROW),    # four, from 128 dimensions
    ("f16", 512, 5000, 64, 8, NARROW),    # eight, 330 MB
    ("f16", 512, 8000, 64, 8, WIDE),      # eight, 520 MB
    ("f16", 512, 8000, 64, 9, NARROW),
    ("u8", 128, 600, 64, 2, WIDE),        # two pairs to a list, 5 MB
    ("u8", 128, 600, 64, 3, NARROW),
    ("u8", 64, 600, 64, 2, WIDE),         # two, 2 MB
    ("u8", 64, 16000, 64, 2, NARROW),     # two, 66 MB of 64 dimensions
    ("u8", 512, 10000, 64, 4, WIDE),      # four, 330 MB
    ("u8", 512, 10000, 64, 5, NARROW),
    ("u8", 192, 600, 64, 2, NARROW),      # two, twelve chunks to a vector
    ("f16", 360, 8000, 64, 4, NARROW),    # four, 370 MB, 45 chunks
    ("u8", 656, 600, 64, 8, WIDE),        # wider than the 16-bit scan takes
])
def test_the_instructions_that_scan(storage, d, length, nq, nprobe, path):
    print(f"[case] narrow rule {storage} d={d} 64 x {length}, {nq} x {nprobe}", flush=True)
    nlist = 64
    gen = torch.Generator("cuda:0").manual_seed(d + length)
    C = torch.randint(0, 16, (nlist, d), device="cuda:0", generator=gen).float()
    near = lambda m: (C[torch.randint(nlist, (m,), device="cuda:0", generator=gen)] +
                      2 * torch.randn(m, d, device="cuda:0", generator=gen)).round_().clamp_(0, 15)
    n = nlist * length
    g = rtams.Index(d, nlist, "l2", 64, pool_blocks=n // 64 + 2 * nlist + 8, n_resources=1, max_batch=nq, max_k=10,
                    max_nprobe=nprobe, candidates_per_query=2 * nprobe * length, storage=storage)
    g.set_centroids(C)
    for at in range(0, n, 65536):
        g.add(near(min(65536, n - at)))
    q = near(nq)
    torch.cuda.synchronize()  # (the rule of the unit asks how long the lists are)
    got = {}
    for mode, took in ((0, "k_scan"), (1, path), (2, NARROW if d <= 640 else WIDE)):  # 2: wherever the kernel can run
        g.set_param("scan_mfma", mode)
        g.set_param("small_requests", 0)
        got[mode] = g.search(q, 10, nprobe)
        torch.cuda.synchronize()
        assert g.poll_error() == 0
        assert g.request_trace(nq)[2] == took, f"scan_mfma {mode}"
    for mode in (1, 2):  # whole numbers: exact in every form
        assert torch.equal(got[mode][0], got[0][0]) and torch.equal(got[mode][1], got[0][1])
    g.close()
