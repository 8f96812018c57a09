"""Updates of rows of any length and alignment on every path (tables with one to many slices and one to many row blocks,
buckets, label-sorted gather), protected and not, against the CPU oracle; fp32 sums are the same integers on all of them."""
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


def _update(x, lab, C, mode):
    Cd, stats = to_dev(C.copy()), ftk.new_stats(DEV)
    _, counts = ftk.kmeans_update(x, lab, Cd, ft_mode=mode, stats=stats)
    torch.cuda.synchronize()
    assert ftk.stats_dict(stats)["detected"] == 0
    return Cd.cpu().numpy(), counts.cpu().numpy()


# N, D, K: rows shorter than a piece, every remainder, one table of many slices and few row blocks, buckets, sorted rows
SIZES = [(900, 1, 5), (900, 3, 500), (3000, 5, 40), (3000, 6, 300), (3000, 7, 2000), (2500, 33, 50), (2500, 34, 400), (1500, 131, 700),
         (4000, 257, 90), (700, 1030, 40), (400, 1100, 200), (70001, 13, 900), (70001, 35, 600), (66001, 130, 270), (66001, 5, 3000),
         (70001, 17, 2500), (70003, 67, 5000), (180001, 13, 8000), (66002, 127, 4001)]


@pytest.mark.parametrize("dtype", ["f32", "f64"])
@pytest.mark.parametrize("N,D,K", SIZES)
def test_update_of_rows_of_any_length(N, D, K, dtype):
    print("update rows", N, D, K, dtype, flush=True)
    rng = np.random.default_rng(N + D + K)
    X = rng.normal(size=(N, D)).astype(np.float32 if dtype == "f32" else np.float64)
    C = rng.normal(size=(K, D)).astype(X.dtype)
    labels = rng.integers(0, K, N).astype(np.int32)
    labels[: N // 3] = K // 2  # one large cluster, and some empty ones
    labels[labels == K - 1] = 0
    ref, counts = oracle.update(X, labels, C)
    lab = to_dev(labels)
    flat = torch.empty(X.size + 1, dtype=torch.float32 if dtype == "f32" else torch.float64, device=DEV)
    flat[1:] = to_dev(X).flatten()
    first = None
    for path in (-1, 0, 1):
        ftk.tuning_override(-1, -1, path)
        for x in (to_dev(X), flat[1:].view(N, D)):
            for mode in (ftk.FT_OFF, ftk.FT_STRICT):
                out, n = _update(x, lab, C, mode)
                assert np.array_equal(n, counts)
                check_centroids(out, ref)
                if dtype == "f32":
                    first = out if first is None else first
                    assert np.array_equal(out, first)


@pytest.mark.parametrize("D", [30, 31])
def test_short_rows_of_doubles_beyond_the_cache(D):
    """Label-sorted: by elements where rows begin at odd places, by pieces where they do not."""
    N, K = 1000003, 2500
    gen = torch.Generator(device=DEV).manual_seed(D)
    flat = torch.randn(N * D + 1, generator=gen, device=DEV, dtype=torch.float64)
    labels = torch.randint(K, (N,), generator=gen, device=DEV, dtype=torch.int32)
    C = np.zeros((K, D))
    for x in (flat[:-1].view(N, D), flat[1:].view(N, D)):
        aligned = x.data_ptr() % 16 == 0 and D % 2 == 0
        assert ftk.update_geometry(ftk.F64, N, D, K, aligned).regs_per_tile == (2 if aligned else 1)
        sums = torch.zeros(K, D, device=DEV, dtype=torch.float64).index_add_(0, labels.long(), x)
        want = torch.bincount(labels, minlength=K)
        for mode in (ftk.FT_OFF, ftk.FT_STRICT):
            out, n = _update(x, labels, C, mode)
            assert np.array_equal(n, want.cpu().numpy())
            check_centroids(out, (sums / want.unsqueeze(1)).cpu().numpy())


@pytest.mark.parametrize("N,D,K,dtype,elements", [(700, 529, 4, "f32", True), (403, 1261, 5, "f32", True), (900, 631, 13, "f32", True),
                                                  (300, 1418, 11, "f32", True), (500, 727, 2, "f64", True), (301, 1027, 3, "f64", True),
                                                  (700, 529, 16, "f32", False), (700, 511, 4, "f32", False), (500, 509, 2, "f64", False)])
def test_long_ragged_rows_of_few_clusters(N, D, K, dtype, elements):
    """By elements where pieces would leave much of a pass idle, with every flip that the geometry names."""
    per_lane = ftk.update_geometry(ftk.F32 if dtype == "f32" else ftk.F64, N, D, K, False).regs_per_tile // 4
    assert per_lane == (1 if elements else 4 if dtype == "f32" else 2)
    rng = np.random.default_rng(D)
    X = rng.normal(size=(N, D)).astype(np.float32 if dtype == "f32" else np.float64)
    labels = rng.integers(0, K, N).astype(np.int32)
    ref, counts = oracle.update(X, labels, X[:K])
    flat = torch.empty(X.size + 1, dtype=torch.float32 if dtype == "f32" else torch.float64, device=DEV)
    flat[1:] = to_dev(X).flatten()
    clean = {}
    for x in (to_dev(X), flat[1:].view(N, D)):
        for mode in (ftk.FT_OFF, ftk.FT_STRICT):
            out, n = _update(x, to_dev(labels), X[:K], mode)
            check_centroids(out, ref)
            assert np.array_equal(n, counts) and np.array_equal(out, clean.setdefault(dtype, out))
    for lane, reg in ((0, 0), (63, 1), (17, 4 * per_lane - 1)):
        C, stats, faults = to_dev(X[:K].copy()), ftk.new_stats(DEV), ftk.make_faults([(0, 1, 0, reg, lane, 54)], DEV)
        ftk.kmeans_update(to_dev(X), to_dev(labels), C, ft_mode=ftk.FT_CORRECT, faults=faults, stats=stats)
        torch.cuda.synchronize()
        st = ftk.stats_dict(stats)
        assert st["injected"] == st["detected"] == st["recomputed"] >= 1 and np.array_equal(C.cpu().numpy(), clean[dtype])
    if dtype == "f32":
        C0 = to_dev(X[:K].copy())
        lab, _, n = ftk.kmeans_step_batched(to_dev(X), C0, 257)
        C1 = to_dev(X[:K].copy())
        lab1, _ = ftk.kmeans_assign(to_dev(X), C1)
        ftk.kmeans_update(to_dev(X), lab1, C1)
        assert torch.equal(lab, lab1) and torch.equal(C0, C1)
