"""Assignment through the matrix-core filter against the oracle and against the exact kernel alone: rows that
have one candidate behind the filter, several, more than a row may list, and tiles that could not keep theirs."""
import numpy as np
import pytest
import torch

from paper_2408_02937_amd import synth
from tests.gpu_common import dev, make_pair

pytestmark = pytest.mark.gpu


def centroids_in_groups(rng, nlist, d, group, spread):
    """Centroids in groups of `group` that differ by `spread` of their norm, scattered over the list numbers."""
    heads = rng.standard_normal(((nlist + group - 1) // group, d))
    c = np.repeat(heads, group, axis=0)[:nlist]
    c = c + spread * rng.standard_normal(c.shape)
    return c[rng.permutation(nlist)].astype(np.float32)


# rows: a wavefront takes one row, two, or sixteen of them; remainders in all of them; more than one sub-round
@pytest.mark.parametrize("rows", [32, 4 * 1024 + 1, 8 * 1024 + 3, 70_001])
@pytest.mark.parametrize("metric", ["l2", "ip"])
# one candidate to a row; several; more than a row lists; whole tiles in the band
@pytest.mark.parametrize("group,spread", [(1, 0.0), (6, 2e-4), (28, 2e-5), (1000, 1e-6)])
def test_filtered_assignment_is_the_exact_one(rows, metric, group, spread):
    rng = np.random.default_rng(rows + group)
    d, nlist = 36, 2000
    C = centroids_in_groups(rng, nlist, d, group, spread)
    print(f"[case] assign rows={rows} {metric} groups of {group}", flush=True)
    w = synth.Workload("assign", metric, d, nlist, 64, 8, 10, np.zeros((0, d), np.float32), C,
                       np.zeros((0, d), np.float32), np.zeros((0, d), np.float32), 1, 0)
    g, o = make_pair(w, pool_blocks=64, candidates_per_query=1024)
    y = (C[rng.integers(0, nlist, rows)] + 0.05 * rng.standard_normal((rows, d))).astype(np.float32)
    y[rows // 2] = C[7]  # a vector that is a centroid
    yd = dev(y)
    g.set_param("use_mfma", 2)
    got = g.assign(yd).cpu().numpy()
    g.set_param("use_mfma", 0)
    assert np.array_equal(got, g.assign(yd).cpu().numpy())
    some = np.r_[:min(rows, 700), max(0, rows - 700):rows]
    assert np.array_equal(got[some], o.assign(y[some]))
    torch.cuda.synchronize()
    g.close()
