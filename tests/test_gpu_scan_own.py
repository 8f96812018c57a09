"""Short rows whose points one workgroup of the scan meets all centroids with: it settles them itself.  Against the oracle
and, to the last bit, against batches small enough that workgroups share their points and a pass of its own settles them."""
import numpy as np
import pytest
import torch

from oracle import cpu as oracle
from paper_2408_01391_amd import binding as ftk, synth
from tests.gpu_util import DEV, check_assign, to_dev

pytestmark = pytest.mark.gpu

# every number of lanes a row has, D % 4 of all kinds, whole and partial last blocks, one and several chunks, both forms
SIZES = [(131073, 5, 800, "f32"), (131072, 8, 1030, "f32"), (140001, 12, 700, "f32"), (139999, 13, 700, "f32"), (131329, 16, 900, "f32"),
         (131327, 17, 300, "f32"), (135000, 24, 300, "f32"), (150001, 25, 330, "f32"), (140032, 32, 400, "f32"),
         (900001, 24, 800, "f32"), (500161, 32, 1000, "f32"), (700001, 27, 900, "f32"), (131585, 6, 700, "f64"), (140001, 11, 700, "f64"),
         (131073, 16, 700, "f64"), (140001, 19, 700, "f64"), (131072, 30, 700, "f64"), (900001, 32, 1500, "f64")]


@pytest.mark.parametrize("N,D,K,dtype", SIZES)
def test_points_settled_by_the_scan_itself(N, D, K, dtype):
    print("own", N, D, K, dtype, flush=True)
    X, C = synth.random_problem(N + D + K, N, D, K, dtype, spread=3.0)
    Xd, Cd = to_dev(X), to_dev(C)
    labels, mind = ftk.kmeans_assign(Xd, Cd)
    rows = np.unique(np.concatenate([np.random.default_rng(N).integers(0, N, 3000), np.arange(300), np.arange(N - 300, N)]))
    lab_h, mind_h = labels.cpu().numpy()[rows], mind.cpu().numpy()[rows]
    check_assign(X[rows], C, lab_h, mind_h, ref=oracle.assign(X[rows], C))
    lab_b, mind_b, _ = ftk.kmeans_step_batched(Xd, Cd.clone(), 2048)
    assert torch.equal(labels, lab_b) and torch.equal(mind, mind_b)
    alone, none = ftk.kmeans_assign(Xd, Cd, want_mindist=False)
    assert none is None and torch.equal(alone, labels)


@pytest.mark.parametrize("N,D,K,dtype", [(131073, 7, 800, "f32"), (140001, 15, 700, "f32"), (600001, 29, 1000, "f32"), (131073, 14, 700, "f64")])
def test_ties_and_values_that_are_not_numbers(N, D, K, dtype):
    X, C = synth.random_problem(D, N, D, K, dtype)
    C[K // 2:] = C[: K - K // 2]  # every point listed
    good, dist = ftk.kmeans_assign(to_dev(X), to_dev(C))
    assert int(good.max()) < K // 2
    bad_rows = [0, 255, 256, 70001, N - 1]
    X[bad_rows[0], 3], X[bad_rows[1]], X[bad_rows[2], 0], X[bad_rows[3]], X[bad_rows[4]] = np.nan, np.inf, -np.inf, np.finfo(X.dtype).max, 0
    bad, bdist = ftk.kmeans_assign(to_dev(X), to_dev(C))
    keep = torch.ones(N, dtype=torch.bool, device=DEV)
    keep[bad_rows] = False
    assert torch.equal(bad[keep], good[keep]) and torch.equal(bdist[keep], dist[keep])
    assert 0 <= int(bad.min()) and int(bad.max()) < K
