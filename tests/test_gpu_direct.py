"""The one-launch assignment of small problems and few centroids (every distance in double, lanes share rows) against the
CPU oracle: every number of lanes and centroid groups its rule can choose, remainders, unaligned rows, ties, batches; and
the scan on batches of the sizes that as whole problems would go to it."""
import numpy as np
import pytest
import torch

from oracle import cpu as oracle
from paper_2408_01391_amd import binding as ftk, synth
from tests.gpu_util import DEV, check_assign, to_dev

pytestmark = pytest.mark.gpu

EPS = {"f32": 2.0 ** -24, "f64": 2.0 ** -53}
# rows of one to 32 lanes, one centroid to several rounds of them, one point to more than fill the chip, D % 4 of all kinds
SIZES = [(1, 70, 1), (3, 65, 2), (700, 33, 1), (5, 1500, 7), (1303, 639, 43), (2000, 1000, 20), (1500, 37, 90), (14665, 520, 2),
         (40001, 126, 2), (257, 1027, 11), (9001, 47, 33), (300, 300, 130), (100003, 34, 4), (6001, 50, 9), (400003, 3, 40),
         (2500, 2, 3000), (70001, 100, 4), (999, 35, 65), (64, 4097, 5)]


def check(X, C, dtype, labels, mind):
    ref = oracle.assign(X, C)
    check_assign(X, C, labels, mind, ref=ref)
    # in double and rounded once (fp32); the order of D terms on both sides (fp64)
    tol = EPS["f32"] if dtype == "f32" else 2 * (X.shape[1] + 4) * EPS["f64"]
    assert np.all(np.abs(mind.astype(np.float64) - ref[1]) <= 1.01 * tol * ref[1])


@pytest.mark.parametrize("dtype", ["f32", "f64"])
@pytest.mark.parametrize("N,D,K", SIZES)
def test_direct_assign_matches_oracle(N, D, K, dtype):
    print("direct", N, D, K, dtype, flush=True)
    X, C = synth.random_problem(N + D + K, N, D, K, dtype)
    stats = ftk.new_stats(DEV)
    labels, mind = ftk.kmeans_assign(to_dev(X), to_dev(C), stats=stats)
    check(X, C, dtype, labels.cpu().numpy(), mind.cpu().numpy())
    flat = torch.empty(X.size + 1, dtype=labels.new_empty(0, dtype=torch.float32 if dtype == "f32" else torch.float64).dtype, device=DEV)
    flat[1:] = to_dev(X).flatten()
    off, none = ftk.kmeans_assign(flat[1:].view(N, D), to_dev(C), want_mindist=False)
    assert none is None and torch.equal(off, labels)
    assert ftk.stats_dict(stats)["refined"] == 0


# the lanes and groups that the list above leaves out: few centroids, and doubles with one or two lanes
@pytest.mark.parametrize("N,D,K,dtype", [
    (3001, 9, 1, "f32"), (3001, 9, 3, "f32"), (3001, 17, 2, "f32"), (3001, 17, 4, "f32"), (3001, 64, 3, "f32"),
    (85003, 20, 30, "f32"), (2001, 150, 3, "f32"), (70, 1500, 1, "f32"), (70, 1500, 3, "f32"), (700001, 20, 4, "f32"),
    (3600001, 7, 2, "f64"), (1700001, 8, 4, "f64"), (1700001, 16, 2, "f64"), (1100001, 16, 4, "f64"), (30001, 18, 40, "f64"),
    (3001, 17, 2, "f64"), (70, 1500, 1, "f64"), (70, 1500, 3, "f64"), (14665, 520, 3, "f64")])
def test_every_cut_of_the_lanes(N, D, K, dtype):
    print("cut", N, D, K, dtype, flush=True)
    X, C = synth.random_problem(N + D + K, N, D, K, dtype)
    stats = ftk.new_stats(DEV)
    labels, mind = ftk.kmeans_assign(to_dev(X), to_dev(C), stats=stats)
    check(X, C, dtype, labels.cpu().numpy(), mind.cpu().numpy())
    flat = torch.empty(X.size + 1, dtype=mind.dtype, device=DEV)
    flat[1:] = to_dev(X).flatten()
    off, _ = ftk.kmeans_assign(flat[1:].view(N, D), to_dev(C), want_mindist=False)
    assert torch.equal(off, labels) and ftk.stats_dict(stats)["refined"] == 0


@pytest.mark.parametrize("N,D,K", [(6267, 22, 169), (5000, 30, 200), (3001, 64, 128), (8000, 17, 341)])
def test_small_problems_in_double_that_the_scan_would_take(N, D, K):
    X, C = synth.random_problem(N, N, D, K, "f64")
    stats = ftk.new_stats(DEV)
    labels, mind = ftk.kmeans_assign(to_dev(X), to_dev(C), stats=stats)
    check(X, C, "f64", labels.cpu().numpy(), mind.cpu().numpy())
    assert ftk.stats_dict(stats)["refined"] == 0  # nothing listed: one launch


@pytest.mark.parametrize("N,D,K,dtype", [(3000, 100, 40, "f32"), (2000, 300, 20, "f64"), (900, 37, 66, "f32")])
def test_direct_assign_ties_and_values_that_are_not_numbers(N, D, K, dtype):
    X, C = synth.random_problem(D, N, D, K, dtype)
    C[K // 2:] = C[: K - K // 2]
    good, _ = ftk.kmeans_assign(to_dev(X), to_dev(C))
    assert int(good.max()) < K // 2
    X[7, 3], X[8] = np.nan, np.inf
    bad, _ = ftk.kmeans_assign(to_dev(X), to_dev(C))
    keep = np.setdiff1d(np.arange(N), [7, 8])
    assert torch.equal(bad[keep], good[keep]) and 0 <= int(bad.min()) and int(bad.max()) < K


@pytest.mark.parametrize("N,D,K,dtype,batch", [(9000, 333, 3, "f64", 1000), (5000, 64, 100, "f64", 777), (30000, 99, 9, "f32", 4096),
                                               (1001, 700, 30, "f64", 1)])
def test_batches_take_the_cut_of_the_whole(N, D, K, dtype, batch):
    X, C = synth.random_problem(N + batch, N, D, K, dtype)
    labels, mind = ftk.kmeans_assign(to_dev(X), to_dev(C))
    lab_b, mind_b, _ = ftk.kmeans_step_batched(to_dev(X), to_dev(C).clone(), batch)
    assert torch.equal(labels, lab_b) and torch.equal(mind, mind_b)


def test_direct_assign_replays_from_a_graph():
    X, C = torch.empty(3001, 130, device="cuda"), torch.empty(25, 130, device="cuda")
    ws = ftk.new_workspace(X, 25, ftk.FT_OFF)
    labels, mind = torch.empty(3001, device="cuda", dtype=torch.int32), torch.empty(3001, device="cuda")
    X.normal_(), C.normal_()
    ftk.kmeans_assign(X, C, labels, mind, workspace=ws)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        ftk.kmeans_assign(X, C, labels, mind, workspace=ws)
    for _ in range(3):
        X.normal_(), C.normal_()
        want = ftk.kmeans_assign(X, C)
        labels.fill_(-1)
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(labels, want[0]) and torch.equal(mind, want[1])


@pytest.mark.parametrize("D,K,batch", [(4, 3000, 33), (8, 4000, 500), (9, 1500, 300), (16, 1024, 257), (17, 900, 1), (33, 900, 700), (40, 5000, 300),
                                       (65, 800, 900), (97, 777, 255), (128, 800, 64), (129, 768, 1030), (255, 1100, 513), (1021, 800, 300),
                                       (1153, 768, 200), (111, 33, 1001), (337, 9, 300), (867, 20, 513)])
def test_the_scan_on_batches_of_any_size(D, K, batch):
    """A batch takes the path of the whole problem, which is large enough for the scan here."""
    N = max(batch + 7, int(1.1e8 / (D * K)) + 1, 9001 if K < 100 else 0)
    if batch == 1:
        N = 4096
        K = 2000
    print("scan batches", N, D, K, batch, flush=True)
    rng = np.random.default_rng(D)
    C = (rng.normal(size=(K, D)) * 5).astype(np.float32)
    X = (C[rng.integers(0, K, N)] + rng.normal(size=(N, D))).astype(np.float32)
    C[K - K // 8:] = C[: K // 8]  # equal candidates: the third pass has something to settle
    labels, mind, _ = ftk.kmeans_step_batched(to_dev(X), to_dev(C).clone(), batch)
    labels, mind = labels.cpu().numpy(), mind.cpu().numpy()
    ref = oracle.assign(X, C)
    check_assign(X, C, labels, mind, ref=ref)
    assert np.all(np.abs(mind.astype(np.float64) - ref[1]) <= 2 * (D + 4) * EPS["f32"] * ref[1])
