"""Small unprotected problems (one launch per assignment and per Lloyd iteration) against the CPU oracle:
compiled widths and their edges, every split of a point's centroids over lanes, more points than one
round of the grid, ragged and unaligned rows, ties, empty clusters, and the fit's objective."""
import numpy as np
import pytest
import torch

from oracle import cpu as oracle
from paper_2408_01391_amd import binding as ftk, synth
from tests.gpu_util import DEV, check_assign, check_centroids, to_dev

pytestmark = pytest.mark.gpu

EPS = {"f32": 2.0 ** -24, "f64": 2.0 ** -53}


@pytest.mark.parametrize("dtype", ["f32", "f64"])
@pytest.mark.parametrize("N,D,K", [(1, 1, 1), (3, 2, 1), (1000, 3, 2), (257, 8, 1000), (777, 9, 65), (513, 16, 33),
                                   (300, 24, 100), (999, 25, 7), (1500, 32, 64), (260, 33, 90), (100, 48, 128),
                                   (1111, 63, 31), (700, 64, 128), (300000, 4, 5), (1000003, 2, 3)])
def test_small_assign_matches_oracle(N, D, K, dtype):
    print("small", N, D, K, dtype, flush=True)
    X, C = synth.random_problem(N + D + K, N, D, K, dtype)
    labels, mind = ftk.kmeans_assign(to_dev(X), to_dev(C))
    torch.cuda.synchronize()
    ref = oracle.assign(X, C)
    labels, mind = labels.cpu().numpy(), mind.cpu().numpy()
    check_assign(X, C, labels, mind, ref=ref)
    # distances are formed in double: one rounding to fp32, or the order of D terms in fp64 (both sides)
    tol = EPS["f32"] if dtype == "f32" else 2 * (D + 4) * EPS["f64"]
    assert np.all(np.abs(mind.astype(np.float64) - ref[1]) <= tol * ref[1] * 1.01)


@pytest.mark.parametrize("N,D,K", [(9429, 39, 70), (20165, 39, 38), (13186, 54, 67), (32803, 48, 17), (11000, 64, 35), (20001, 33, 35)])
def test_small_assign_of_longer_rows(N, D, K):
    """Rows of 33 .. 64 floats where lanes that share a row would have little to do in their last round."""
    print("small, longer rows", N, D, K, flush=True)
    X, C = synth.random_problem(N + D + K, N, D, K, "f32")
    flat = torch.empty(X.size + 1, dtype=torch.float32, device=DEV)
    flat[1:] = to_dev(X).flatten()
    ref = oracle.assign(X, C)
    for x in (to_dev(X), flat[1:].view(N, D)):
        labels, mind = ftk.kmeans_assign(x, to_dev(C))
        labels, mind = labels.cpu().numpy(), mind.cpu().numpy()
        check_assign(X, C, labels, mind, ref=ref)
        assert np.all(np.abs(mind.astype(np.float64) - ref[1]) <= EPS["f32"] * ref[1] * 1.01)


def test_small_assign_ties_offsets_and_values_that_are_not_numbers():
    X, C = synth.random_problem(4, 900, 12, 40, "f32")
    C[20:] = C[:20]
    labels, _ = ftk.kmeans_assign(to_dev(X), to_dev(C))
    assert int(labels.max()) < 20
    flat = torch.empty(X.size + 1, dtype=torch.float32, device=DEV)
    flat[1:] = to_dev(X).flatten()
    off, none = ftk.kmeans_assign(flat[1:].view(X.shape), to_dev(C), want_mindist=False)
    assert none is None and torch.equal(off, labels)
    Xb = X.copy()
    Xb[7, 3] = np.nan
    Xb[8, 0] = np.inf
    bad, _ = ftk.kmeans_assign(to_dev(Xb), to_dev(C))
    keep = np.ones(len(X), bool)
    keep[7:9] = False
    assert np.array_equal(bad.cpu().numpy()[keep], labels.cpu().numpy()[keep])
    assert 0 <= int(bad.min()) and int(bad.max()) < 40


@pytest.mark.parametrize("dtype", ["f32", "f64"])
@pytest.mark.parametrize("N,D,K,iters", [(4096, 16, 8, 10), (1000, 3, 5, 1), (5000, 8, 500, 2), (30000, 17, 30, 3),
                                         (200000, 4, 6, 3), (900, 64, 60, 4), (2, 5, 2, 3)])
def test_small_fit_matches_oracle(N, D, K, iters, dtype):
    print("small fit", N, D, K, iters, dtype, flush=True)
    X, _ = synth.random_problem(3 * N + D + K, N, D, K, dtype)
    C0 = X[np.random.default_rng(N).choice(N, K, replace=False)].copy()
    ref = oracle.fit(X, C0, iters)
    out = ftk.kmeans_fit(to_dev(X), K, iters, C_init=to_dev(C0))
    assert np.array_equal(out["labels"].cpu().numpy(), ref["labels"])
    assert np.array_equal(out["counts"].cpu().numpy(), ref["counts"])
    check_centroids(out["C"].cpu().numpy(), ref["C"])
    assert np.allclose(out["inertia"], ref["inertia"], rtol=1e-6 if dtype == "f32" else 1e-13)


def test_small_fit_keeps_an_empty_cluster_and_repeats_itself():
    X, _ = synth.random_problem(8, 3000, 6, 4, "f32")
    C0 = np.concatenate([X[:4], np.full((1, 6), 1e4, np.float32)])
    a = ftk.kmeans_fit(to_dev(X), 5, 4, C_init=to_dev(C0))
    b = ftk.kmeans_fit(to_dev(X), 5, 4, C_init=to_dev(C0))
    assert int(a["counts"][4]) == 0 and np.array_equal(a["C"][4].cpu().numpy(), C0[4])
    assert torch.equal(a["C"], b["C"]) and torch.equal(a["labels"], b["labels"])


@pytest.mark.parametrize("N,D,K", [(4096, 16, 8), (30000, 17, 300)])
def test_fits_of_either_kind_are_profiled_once_an_iteration(N, D, K):
    X, _ = synth.random_problem(2, N, D, K, "f32")
    Xd, C0 = to_dev(X), to_dev(X[:K])
    ftk.profile_enable(True)
    try:
        ftk.profile_read()
        ftk.kmeans_fit(Xd, K, 5, C_init=C0)
        ms, launches = ftk.profile_read()
    finally:
        ftk.profile_enable(False)
    assert launches == 5 and ms > 0.0
