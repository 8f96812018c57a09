"""The bucketed update (fp32, unprotected) against the CPU oracle and, bit for bit, against the
label-sorted path: both add the same integers.  Edges: a bucket that is empty, one that holds every
point, a last bucket and a last source that are not full, labels out of range, rows of several pieces."""
import numpy as np
import pytest
import torch

from oracle import cpu as oracle
from paper_2408_01391_amd import binding as ftk
from tests.gpu_util import DEV, check_centroids, to_dev

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def _restore_rules():
    yield
    ftk.tuning_override(-1, -1, -1)


def update(X, labels, C):
    Cd = to_dev(C).clone()
    _, counts = ftk.kmeans_update(to_dev(X), to_dev(labels), Cd)
    torch.cuda.synchronize()
    return Cd.cpu().numpy(), counts.cpu().numpy()


@pytest.mark.parametrize("N,D,K", [(65536, 16, 2100), (70001, 32, 4096), (73729, 20, 3001), (66000, 64, 1000),
                                   (65537, 128, 300), (81920, 4, 8192), (70000, 8, 8191), (66000, 256, 700)])
@pytest.mark.parametrize("spread", ["even", "one", "skewed", "holes"])
def test_bucketed_update_equals_sorted_path_and_oracle(N, D, K, spread):
    rng = np.random.default_rng(N + D + K)
    print("bucketed update", N, D, K, spread, flush=True)
    X = (rng.normal(size=(N, D)) * 3 + 1).astype(np.float32)
    if spread == "even":
        labels = rng.integers(0, K, N)
    elif spread == "one":
        labels = np.full(N, K - 1)
    elif spread == "skewed":
        labels = np.minimum((rng.random(N) ** 4 * K).astype(np.int64), K - 1)
    else:
        labels = rng.integers(0, K, N)
        labels[(labels >= K // 4) & (labels < K // 2)] = 0  # whole buckets without a point
    labels = labels.astype(np.int32)
    C = rng.normal(size=(K, D)).astype(np.float32)
    C_g, counts = update(X, labels, C)
    C_o, n_o = oracle.update(X, labels, C)
    assert np.array_equal(counts, n_o)
    check_centroids(C_g, C_o)
    ftk.tuning_override(-1, -1, 1)
    C_s, counts_s = update(X, labels, C)
    assert np.array_equal(C_g, C_s) and np.array_equal(counts, counts_s)


def test_bucketed_update_skips_labels_out_of_range():
    rng = np.random.default_rng(1)
    N, D, K = 70000, 32, 3000
    X = rng.normal(size=(N, D)).astype(np.float32)
    labels = rng.integers(0, K, N).astype(np.int32)
    bad = rng.choice(N, 500, replace=False)
    labels[bad[:250]] = K
    labels[bad[250:]] = -3
    C = rng.normal(size=(K, D)).astype(np.float32)
    C_g, counts = update(X, labels, C)
    keep = np.setdiff1d(np.arange(N), bad)
    C_o, n_o = oracle.update(X[keep], labels[keep], C)
    assert np.array_equal(counts, n_o)
    check_centroids(C_g, C_o)


@pytest.mark.parametrize("dtype", [np.float32, np.float64])
@pytest.mark.parametrize("N,D,K", [(2530, 1, 7782), (2530, 1, 7783), (300, 1, 8192), (70000, 1, 12797), (7, 1, 8541), (900, 2, 8192)])
def test_update_of_one_feature_with_many_clusters(N, D, K, dtype):
    """A table row of one feature and its pad, times 8192 clusters with their counts, is more LDS than there is."""
    rng = np.random.default_rng(N + K)
    print("one feature", N, D, K, dtype.__name__, flush=True)
    X = rng.normal(size=(N, D)).astype(dtype)
    labels = rng.integers(0, K, N).astype(np.int32)
    labels[0] = K - 1
    C = rng.normal(size=(K, D)).astype(dtype)
    C_o, n_o = oracle.update(X, labels, C)
    C_g, counts = update(X, labels, C)
    assert np.array_equal(counts, n_o)
    check_centroids(C_g, C_o)
    Cd = to_dev(C).clone()
    lab, _, cnt = ftk.kmeans_step_batched(to_dev(X), Cd, max(1, N // 3))
    C_s, n_s = oracle.update(X, lab.cpu().numpy(), C)
    assert np.array_equal(cnt.cpu().numpy(), n_s)
    check_centroids(Cd.cpu().numpy(), C_s)


# beside the shapes above, of which those with 4 and 8 features do not take this path: its shortest rows, and more
# sources than the workgroup that adds up has threads
@pytest.mark.parametrize("N,D,K", [(66001, 12, 8191), (70001, 16, 8192), (8400001, 12, 3001), (16800000, 16, 2100)])
def test_bucketed_update_of_short_rows_and_of_many_sources(N, D, K):
    print("bucketed update", N, D, K, flush=True)
    gen = torch.Generator(device=DEV).manual_seed(N)
    X = torch.randn(N, D, generator=gen, device=DEV) * 3 + 1
    labels = (torch.rand(N, generator=gen, device=DEV) ** 2 * K).to(torch.int32)
    C = torch.randn(K, D, generator=gen, device=DEV)
    ws = ftk.new_workspace(X, K)
    results = []
    for path in (-1, 1):
        ftk.tuning_override(-1, -1, path)
        C_new = C.clone()
        _, counts = ftk.kmeans_update(X, labels, C_new, workspace=ws)
        results.append((C_new, counts))
    torch.cuda.synchronize()
    assert torch.equal(results[0][0], results[1][0]) and torch.equal(results[0][1], results[1][1])
    n = torch.bincount(labels.long(), minlength=K)
    assert torch.equal(n, results[0][1].long())
    sums = torch.zeros(K, D, dtype=torch.float64, device=DEV)
    for r in range(0, N, 1 << 20):
        sums.index_add_(0, labels[r:r + (1 << 20)].long(), X[r:r + (1 << 20)].double())
    means = torch.where(n[:, None] > 0, sums / n.clamp(min=1)[:, None], C.double())
    check_centroids(results[0][0].cpu().numpy(), means.float().cpu().numpy())
