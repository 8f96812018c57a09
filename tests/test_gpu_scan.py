"""The scan path of the unprotected assignment (bf16 scan, exact settlement) against the CPU oracle at
the sizes where it can go wrong: edges of the compiled widths and tiles, ragged rows, workgroups that
share a block of points, rows too long for its own settlement of ties, exact ties, more candidates than
are noted, scales far from one, values that are not numbers, rows aligned to elements only."""
import numpy as np
import pytest
import torch

from oracle import cpu as oracle
from paper_2408_01391_amd import binding as ftk
from tests.gpu_util import DEV, check_assign, to_dev

pytestmark = pytest.mark.gpu

EPS = {"f32": 2.0 ** -24, "f64": 2.0 ** -53}
NP = {"f32": np.float32, "f64": np.float64}


def blobs(seed, N, D, K, dtype, scale=1.0):
    rng = np.random.default_rng(seed)
    centres = rng.normal(size=(max(2, K // 3), D)) * 3
    X = centres[rng.integers(0, len(centres), N)] + rng.normal(size=(N, D))
    C = X[rng.integers(0, N, K)] + rng.normal(size=(K, D)) * 0.1
    return (X * scale).astype(NP[dtype]), (C * scale).astype(NP[dtype])


def run(X, C, **kw):
    labels, mind = ftk.kmeans_assign(to_dev(X), to_dev(C), **kw)
    torch.cuda.synchronize()
    return labels.cpu().numpy(), mind.cpu().numpy()


def check_direct(X, C, dtype):
    """Labels as everywhere; the distance is the direct-difference one: D terms, each off by at most
    3 roundings (difference, square, sum), in any order - the oracle's own sum included for fp64."""
    labels, mind = run(X, C)
    ref = oracle.assign(X, C)
    check_assign(X, C, labels, mind, ref=ref)
    assert np.all(np.abs(mind.astype(np.float64) - ref[1]) <= 2 * (X.shape[1] + 4) * EPS[dtype] * ref[1])
    return labels


@pytest.mark.parametrize("dtype", ["f32", "f64"])
@pytest.mark.parametrize("N,D,K", [
    (100003, 4, 768), (700, 8, 1000), (3001, 7, 800), (2000, 9, 800),          # one block, three / two pieces
    (5000, 16, 769), (257, 17, 1200), (1000, 31, 800), (100001, 45, 200),      # ragged rows
    (3000, 64, 1023), (900, 65, 800), (255, 97, 777), (1500, 128, 800),        # compiled widths
    (1, 33, 900), (300, 40, 5000),                                             # splits of one block of points
    (1030, 129, 768), (600, 160, 800), (513, 255, 1100), (300, 1021, 800),     # streamed rows, ragged ends
    (200, 1153, 768),                                                          # ties settled by the refine kernel
])
def test_scan_matches_oracle_at_the_edges(N, D, K, dtype):
    print("scan", N, D, K, dtype, flush=True)
    X, C = blobs(N + D + K, N, D, K, dtype)
    check_direct(X, C, dtype)


@pytest.mark.parametrize("N,D,K", [(700, 97, 8), (1001, 111, 33), (300, 337, 9), (513, 867, 20), (300001, 21, 32)])
def test_scan_of_ragged_rows_with_few_centroids(N, D, K):
    print("scan ragged", N, D, K, flush=True)
    X, C = blobs(N + D + K, N, D, K, "f32")
    check_direct(X, C, "f32")


@pytest.mark.parametrize("dtype,scale", [("f32", 1e-15), ("f32", 1e15), ("f64", 1e-120), ("f64", 1e120), ("f64", 1e-25)])
@pytest.mark.parametrize("D", [6, 48, 200])
def test_scan_at_scales_far_from_one(D, dtype, scale):
    X, C = blobs(D, 1500, D, 800, dtype, scale)
    check_direct(X, C, dtype)


@pytest.mark.parametrize("D", [8, 40, 150])
def test_exact_ties_go_to_the_lowest_index_and_crowds_are_settled(D):
    X, C = blobs(D + 1, 2000, D, 800, "f32")
    C[700:] = C[:100]            # two equal candidates
    C[300:320] = C[5]            # more equal candidates than the third pass notes
    X[:50] = C[5]
    labels = check_direct(X, C, "f32")
    assert np.all(labels[:50] == 5)
    assert labels.max() < 700 and not np.any((labels >= 300) & (labels < 320))


@pytest.mark.parametrize("D", [8, 40, 150])
def test_rows_that_are_not_finite_leave_the_others_alone(D):
    X, C = blobs(D + 2, 1500, D, 800, "f32")
    clean, md = run(X, C)
    Xb = X.copy()
    Xb[7, D // 2] = np.nan
    Xb[600, 0] = np.inf
    Xb[1400, D - 1] = 3e38
    labels, mind = run(Xb, C)
    keep = np.ones(len(X), bool)
    keep[[7, 600, 1400]] = False
    assert np.array_equal(labels[keep], clean[keep]) and np.array_equal(mind[keep], md[keep])
    assert labels.min() >= 0 and labels.max() < 800
    Cb = C.copy()
    Cb[17] = np.nan              # a centroid that is not a number never wins
    labels, mind = run(X, Cb)
    far = C.copy()
    far[17] = 1e6
    ref = oracle.assign(X, far)
    assert np.array_equal(labels, ref[0])


@pytest.mark.parametrize("dtype", ["f32", "f64"])
@pytest.mark.parametrize("D", [8, 33, 130])
def test_rows_aligned_to_elements_only_and_no_distance_wanted(D, dtype):
    X, C = blobs(D + 3, 1200, D, 800, dtype)
    ref, _ = run(X, C)
    Xo = torch.empty(X.size + 1, dtype=to_dev(X).dtype, device=DEV)
    Co = torch.empty(C.size + 1, dtype=Xo.dtype, device=DEV)
    Xo[1:] = to_dev(X).flatten()
    Co[1:] = to_dev(C).flatten()
    labels, _ = ftk.kmeans_assign(Xo[1:].view(X.shape), Co[1:].view(C.shape))
    assert np.array_equal(labels.cpu().numpy(), ref)
    bare, none = ftk.kmeans_assign(to_dev(X), to_dev(C), want_mindist=False)
    assert none is None and np.array_equal(bare.cpu().numpy(), ref)


def test_scan_counts_what_it_settles():
    X, C = blobs(5, 3000, 40, 800, "f32")
    C[700:] = C[:100]
    stats = ftk.new_stats(DEV)
    labels, _ = ftk.kmeans_assign(to_dev(X), to_dev(C), stats=stats)
    torch.cuda.synchronize()
    tied = np.isin(labels.cpu().numpy(), np.arange(100)).sum()
    assert ftk.stats_dict(stats)["refined"] >= tied
