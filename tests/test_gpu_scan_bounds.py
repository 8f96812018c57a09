"""The error bounds of the unprotected scan, on operands that reach them and on data that stretches
them: labels are the exact arg-min, whatever two bf16 pieces lose, overflow or leave out of proportion."""
import numpy as np
import pytest
import torch

from oracle import cpu as oracle
from paper_2408_01391_amd import binding as ftk
from tests.bf16_operands import FIRST, adversarial
from tests.gpu_util import check_assign, to_dev

pytestmark = pytest.mark.gpu

NP = {"f32": np.float32, "f64": np.float64}


def run(X, C, **kw):
    labels, mind = ftk.kmeans_assign(to_dev(X), to_dev(C), **kw)
    torch.cuda.synchronize()
    return labels.cpu().numpy(), mind.cpu().numpy()


@pytest.mark.parametrize("moved", [False, True])
@pytest.mark.parametrize("dtype", ["f32", "f64"])
@pytest.mark.parametrize("D", [20, 32, 33, 64, 100, 128, 160])
def test_worst_operands_of_two_pieces_are_settled(D, dtype, moved):
    print("scan bound", D, dtype, moved, flush=True)
    X, C = adversarial(D, 800, 1 / 32, moved=moved)
    labels, _ = run(X.astype(NP[dtype]), C.astype(NP[dtype]))
    assert np.all(labels == FIRST)


@pytest.mark.parametrize("dtype", ["f32", "f64"])
@pytest.mark.parametrize("D,nudge", [(20, 0.001), (32, 0.008), (32, 0.001), (64, 0.001), (128, 0.001)])
def test_points_next_to_a_centroid_with_all_features_at_a_midpoint(D, nudge, dtype):
    """Distances far below the norms: the wrong centroid is thousands of times farther."""
    K = 800
    X = np.full((64, D), 1 + 2.0 ** -8 - 2.0 ** -16, NP[dtype])
    C = np.zeros((K, D), NP[dtype])
    C[K // 2:] = -1
    C[5] = 1 + 2.0 ** -8 - (2.0 ** -17 + 2.0 ** -22)
    C[9] = 1 + 2.0 ** -8 + (2.0 ** -17 + 2.0 ** -22)
    C[9, 0] += nudge
    labels, mind = run(X, C)
    check_assign(X, C, labels, mind)
    assert np.all(labels == 5)


@pytest.mark.parametrize("D,K,dtype", [(97, 8, "f32"), (97, 800, "f32"), (40, 768, "f64"), (12, 800, "f32"), (200, 800, "f64")])
def test_centroids_of_mixed_magnitude_meet_every_candidate(D, K, dtype):
    """Rows whose scaled norms overflow fp32 beside rows that look tiny: no score may be trusted, and the
    few that are numbers are not all there is."""
    rng = np.random.default_rng(D)
    C = rng.normal(size=(K, D)) * 1e-10
    big = np.arange(K) % 8 if K > 8 else np.arange(K) % 2
    C[big % 2 == 1] *= 1e20 if dtype == "f32" else 1e35
    X = np.concatenate([1.01 * C[1:2], 0.99 * C[3:4], C[2:3], 1.5 * C[5:6]])
    X, C = X.astype(NP[dtype]), C.astype(NP[dtype])
    labels, mind = run(X, C)
    ref = oracle.assign(X, C)
    assert np.array_equal(labels, ref[0])
    assert np.allclose(mind, ref[1], rtol=1e-5)


def offset_blobs(seed, N, D, K, offset, dtype):
    rng = np.random.default_rng(seed)
    C = rng.normal(size=(K, D)) * 5
    X = C[rng.integers(0, K, N)] + rng.normal(size=(N, D))
    return (X + offset).astype(NP[dtype]), (C + offset).astype(NP[dtype])


def refined(X, C):
    stats = ftk.new_stats("cuda:0")
    labels, mind = run(X, C, stats=stats)
    check_assign(X, C, labels, mind)
    return ftk.stats_dict(stats)["refined"]


@pytest.mark.parametrize("dtype", ["f32", "f64"])
@pytest.mark.parametrize("D", [8, 16, 32, 128, 200])
def test_an_offset_of_all_data_lists_no_more_points(D, dtype):
    """Distances do not change when everything moves, so neither may what cannot be decided."""
    N, K = 20000, 1024
    at_origin = refined(*offset_blobs(D, N, D, K, 0.0, dtype))
    for offset in (100.0, 1000.0):
        n = refined(*offset_blobs(D, N, D, K, offset, dtype))
        print("listed", D, dtype, offset, at_origin, n, flush=True)
        assert n <= 2 * at_origin + N // 50


@pytest.mark.parametrize("dtype,N,D,K", [("f64", 60, 8192, 300), ("f64", 60, 8193, 300), ("f32", 60, 16385, 300), ("f32", 40, 1100, 9000)])
def test_longest_rows_with_a_reference_and_beyond(dtype, N, D, K):
    labels, mind = run(*(data := offset_blobs(D, N, D, K, 50.0, dtype)))
    check_assign(*data, labels, mind)


@pytest.mark.parametrize("dtype", ["f32", "f64"])
@pytest.mark.parametrize("at", [0, 517])
@pytest.mark.parametrize("D", [8, 32, 128, 200])
def test_one_far_centroid_lists_no_more_points(D, at, dtype):
    N, K = 20000, 1024
    X, C = offset_blobs(D, N, D, K, 0.0, dtype)
    near = refined(X, C)
    C[at] *= 100
    n = refined(X, C)
    print("listed", D, dtype, at, near, n, flush=True)
    assert n <= 2 * near + N // 50


@pytest.mark.parametrize("dtype", ["f32", "f64"])
@pytest.mark.parametrize("N,D,K", [(300, 4, 800), (40000, 9, 900), (2000, 17, 777), (40, 45, 800), (20000, 64, 1000),
                                   (700, 131, 800), (33, 513, 1500),
                                   (12000, 1160, 300), (90, 1201, 800)])
@pytest.mark.parametrize("kind", ["groups", "one feature", "groups with copies"])
def test_points_with_many_candidates(N, D, K, dtype, kind):
    """More centroids within the scan's bound than it notes: settled on the fp32 / fp64 matrix instructions
    where their bound tells them apart, else (equal centroids among them) by comparison with all."""
    print("many candidates", N, D, K, dtype, kind, flush=True)
    rng = np.random.default_rng(N + D)
    C = rng.normal(size=(K, D)) * 5
    X = C[rng.integers(0, K, N)] + rng.normal(size=(N, D))
    if kind == "one feature":
        X[:, 0] *= 1e4
        C[:, 0] *= 1e4
    else:
        X += np.where(rng.random(N) < 0.5, 3000.0, -3000.0)[:, None]
        C += np.where(np.arange(K) % 2 == 0, 3000.0, -3000.0)[:, None]
    if kind == "groups with copies":
        C[K - 40:] = C[:40]
        X[:20] = C[K - 20:]
    X, C = X.astype(NP[dtype]), C.astype(NP[dtype])
    labels, mind = run(X, C)
    ref = oracle.assign(X, C)
    check_assign(X, C, labels, mind, ref=ref)
    # distances of this path are direct: D differences, squares and sums, each rounded
    eps = 2.0 ** -24 if dtype == "f32" else 2.0 ** -53
    assert np.all(np.abs(mind.astype(np.float64) - ref[1]) <= 2 * (D + 4) * eps * ref[1] + 1e-5 * ref[1] * (labels != ref[0]))


@pytest.mark.parametrize("dtype", ["f32", "f64"])
@pytest.mark.parametrize("N,D,K", [(200003, 4, 769), (60001, 4, 1025), (8999, 8, 1100), (9001, 24, 400), (36001, 64, 230),
                                   (110001, 16, 170), (1201, 200, 150)])
def test_scan_on_both_sides_of_its_rule(N, D, K, dtype):
    """Calls just beyond the lines from which the scan takes over, whatever kernel runs on the near side."""
    print("rule", N, D, K, dtype, flush=True)
    for n, k in ((N, K), (N - 3, K - 20)):
        X, C = offset_blobs(N + D, n, D, k, 3.0, dtype)
        labels, mind = run(X, C)
        rows = np.arange(0, n, max(1, n // 4000))
        check_assign(X, C, labels, mind, rows=rows)


@pytest.mark.parametrize("dtype,N,D,K", [("f32", 20001, 160, 85), ("f32", 9001, 161, 66), ("f32", 36001, 384, 90), ("f32", 3001, 1024, 49),
                                         ("f32", 110003, 164, 66), ("f32", 60001, 1028, 66), ("f64", 9001, 161, 113),
                                         ("f64", 110003, 130, 82), ("f64", 36001, 385, 97), ("f64", 20001, 1025, 130)])
def test_lines_of_rows_beyond_128_features(dtype, N, D, K):
    """On the near side of a line distances may be of the expanded form; on the far side they are differences' squares."""
    print("line", dtype, N, D, K, flush=True)
    for k in (K - 4, K):
        X, C = offset_blobs(N + D, N, D, k, 3.0, dtype)
        labels, mind = run(X, C)
        rows = np.arange(0, N, max(1, N // 3000))
        check_assign(X, C, labels, mind, rows=rows)
    ref = ((X[rows].astype(np.float64) - C[labels[rows]].astype(np.float64)) ** 2).sum(1)
    eps = 2.0 ** -24 if dtype == "f32" else 2.0 ** -53
    assert np.all(np.abs(mind[rows].astype(np.float64) - ref) <= 2 * (D + 4) * eps * ref)
