"""Workspace sizes (host only) and what runs in a workspace of each size."""
import numpy as np
import pytest
import torch

from oracle import cpu as oracle
from paper_2408_01391_amd import binding as ftk

MB = 1 << 20


@pytest.fixture(autouse=True)
def _restore_rules():
    if not ftk._LIB_PATH.exists():
        pytest.skip("libftkmeans.so not built")
    yield
    ftk.tuning_override(-1, -1, -1)


@pytest.mark.parametrize("dtype,N,D,K,most", [(ftk.F32, 1 << 21, 256, 16384, 280 * MB), (ftk.F64, 1 << 20, 512, 8192, 280 * MB),
                                              (ftk.F32, 1 << 20, 130, 2048, 60 * MB), (ftk.F32, 2000, 32, 900, 9 * MB)])
def test_protected_calls_do_not_reserve_what_only_unprotected_ones_use(dtype, N, D, K, most):
    sizes = [ftk.workspace_bytes(dtype, N, D, K, m) for m in (ftk.FT_OFF, ftk.FT_DETECT, ftk.FT_CORRECT, ftk.FT_STRICT)]
    assert sizes[1] == sizes[2] == sizes[3] <= min(most, sizes[0])


@pytest.mark.parametrize("dtype,N,D,K", [(ftk.F32, 1 << 20, 16, 64), (ftk.F32, 1 << 20, 32, 300), (ftk.F32, 5000, 8, 4096),
                                         (ftk.F64, 1 << 20, 64, 1024), (ftk.F32, 4096, 16, 8)])
def test_size_does_not_depend_on_a_forced_kernel(dtype, N, D, K):
    for mode in (ftk.FT_OFF, ftk.FT_STRICT):
        ftk.tuning_override(-1, -1, -1)
        size = ftk.workspace_bytes(dtype, N, D, K, mode)
        for forced in ((0, 1, 0), (1, 8, 1)):
            ftk.tuning_override(*forced)
            assert ftk.workspace_bytes(dtype, N, D, K, mode) == size


@pytest.mark.parametrize("dtype", [ftk.F32, ftk.F64])
@pytest.mark.parametrize("D,K", [(1, 8), (17, 300), (64, 64), (65, 1000), (128, 256), (129, 4), (512, 64), (1024, 71)])
def test_a_workspace_for_the_most_points_serves_fewer(dtype, D, K):
    """A batch of fewer rows is accepted wherever a larger one is."""
    N = sorted({int(64 * 1.07 ** i) for i in range(150)} | {e + d for e in (65536, 131072, 262144, 524288) for d in (-1, 0, 1)})
    size = [ftk.workspace_bytes(dtype, n, D, K, ftk.FT_STRICT) for n in N]
    assert size == sorted(size)


@pytest.mark.parametrize("dtype,D", [(ftk.F32, 512), (ftk.F32, 1024), (ftk.F64, 256)])
def test_long_rows_reserve_a_walker_per_64_rows(dtype, D):
    """Two slots of 64-bit sums a walker, the rest as for a problem whose tables are larger than them."""
    N, K = 200000, 64
    more = ftk.workspace_bytes(dtype, N, D, K, ftk.FT_STRICT) - ftk.workspace_bytes(dtype, N // 2, D, K, ftk.FT_STRICT)
    assert more <= (N // 2 // 64 + 1) * 2 * D * 8 + N * 16


@pytest.mark.gpu
@pytest.mark.parametrize("dtype,N,D,K", [("f32", 70000, 32, 3000), ("f64", 5000, 40, 800), ("f32", 4096, 16, 8), ("f32", 3000, 200, 800)])
def test_unprotected_calls_in_a_workspace_of_a_protected_mode(dtype, N, D, K):
    """Accepted, with the results of the other paths; bytes beyond the size given stay untouched."""
    np_t = np.float32 if dtype == "f32" else np.float64
    rng = np.random.default_rng(N)
    C = (rng.normal(size=(K, D)) * 5).astype(np_t)
    X = (C[rng.integers(0, K, N)] + rng.normal(size=(N, D))).astype(np_t)
    Xd, Cd = torch.from_numpy(X).cuda(), torch.from_numpy(C).cuda()
    size = ftk.workspace_bytes(ftk.F32 if dtype == "f32" else ftk.F64, N, D, K, ftk.FT_STRICT)
    whole = torch.full((size + MB,), 0x5a, dtype=torch.uint8, device="cuda")
    start = -whole.data_ptr() % 256
    ws = whole[start:start + size]
    ref = oracle.assign(X, C)
    calls = [ftk.kmeans_assign] + ([ftk.kmeans_assign_fast] if dtype == "f32" and D <= 128 else [])
    for call in calls:
        labels, _ = call(Xd, Cd, workspace=ws)
        assert np.array_equal(labels.cpu().numpy(), ref[0])
    C_new = Cd.clone()
    _, counts = ftk.kmeans_update(Xd, labels, C_new, workspace=ws)
    assert np.array_equal(counts.cpu().numpy(), np.bincount(ref[0], minlength=K))
    out = ftk.kmeans_fit(Xd, K, 1, C_init=Cd, workspace=ws)
    assert torch.equal(out["C"], C_new) and torch.equal(out["labels"], labels)
    assert bool((whole[start + size:] == 0x5a).all()) and bool((whole[:start] == 0x5a).all())


@pytest.mark.gpu
@pytest.mark.parametrize("dtype,N,D,K", [("f32", 3000, 200, 800), ("f32", 9000, 129, 931), ("f64", 5000, 300, 900), ("f32", 20000, 33, 2000)])
def test_a_few_bytes_beyond_a_protected_mode_change_nothing(dtype, N, D, K):
    """What is left of an allocation after its alignment does not choose the path."""
    gen = torch.Generator(device="cuda").manual_seed(K)
    t = torch.float32 if dtype == "f32" else torch.float64
    C = torch.randn(K, D, generator=gen, device="cuda", dtype=t) * 5
    X = C[torch.randint(K, (N,), generator=gen, device="cuda")] + torch.randn(N, D, generator=gen, device="cuda", dtype=t)
    size = ftk.workspace_bytes(ftk.F32 if dtype == "f32" else ftk.F64, N, D, K, ftk.FT_STRICT)
    ws = torch.empty(size + 512, dtype=torch.uint8, device="cuda")
    ws = ws[-ws.data_ptr() % 256:]
    labels, mind = ftk.kmeans_assign(X, C, workspace=ws[:size])
    for more in (1, 255):
        lab2, mind2 = ftk.kmeans_assign(X, C, workspace=ws[:size + more])
        assert torch.equal(labels, lab2) and torch.equal(mind, mind2)


@pytest.mark.parametrize("dtype,N,D,K", [(ftk.F32, 1 << 21, 256, 16384), (ftk.F64, 1 << 20, 512, 8192), (ftk.F32, 1 << 24, 132, 33000)])
def test_records_of_the_scan_do_not_grow_with_points_times_centroids(dtype, N, D, K):
    """64 MB of records, 8 bytes a listed point, a copy of the centroids, the tables of the bucketed update."""
    more = ftk.workspace_bytes(dtype, N, D, K, ftk.FT_OFF) - ftk.workspace_bytes(dtype, N, D, K, ftk.FT_STRICT)
    assert more <= 256 * MB


def test_new_workspace_serves_unprotected_calls_at_full_speed():
    X = torch.empty(4000, 40, dtype=torch.float64)
    size = ftk.workspace_bytes(ftk.F64, 4000, 40, 900, ftk.FT_OFF)
    assert size > ftk.workspace_bytes(ftk.F64, 4000, 40, 900, ftk.FT_STRICT)
    for mode in (ftk.FT_OFF, ftk.FT_CORRECT, ftk.FT_STRICT):
        assert ftk.new_workspace(X, 900, mode).numel() >= size


@pytest.mark.gpu
@pytest.mark.parametrize("dtype,N,D,K", [("f32", 4300001, 4, 768), ("f32", 70001, 132, 20000), ("f64", 30011, 1160, 40000)])
def test_scan_in_several_launches(dtype, N, D, K):
    """More points than one launch has records for: rows on both sides of the launches' ends, and points to
    settle (equal centroids) in each of them."""
    print("several launches", dtype, N, D, K, flush=True)
    gen = torch.Generator(device="cuda").manual_seed(N)
    t = torch.float32 if dtype == "f32" else torch.float64
    C = torch.randn(K, D, generator=gen, device="cuda", dtype=t) * 5
    C[K - 100:] = C[:100]
    pick = torch.randint(K, (N,), generator=gen, device="cuda")
    pick[::97] = K - 1 - (pick[::97] % 100)
    X = torch.randn(N, D, generator=gen, device="cuda", dtype=t) * 0.1 + C[pick]
    stats = ftk.new_stats("cuda:0")
    labels, mind = ftk.kmeans_assign(X, C, stats=stats)
    torch.cuda.synchronize()
    assert ftk.stats_dict(stats)["refined"] >= N // 97
    rows = torch.unique(torch.cat([torch.arange(0, N, max(1, N // 150)), torch.arange(0, N - 4, 2048)[:: max(1, N // 2048 // 60)] + 1,
                                   torch.arange(N - 20, N), torch.arange(0, N, 97)[:: max(1, N // 97 // 60)]]))
    Xr, Cn = X[rows.cuda()].cpu().numpy(), C.cpu().numpy()
    ref = oracle.assign(Xr, Cn)
    assert np.array_equal(labels.cpu().numpy()[rows], ref[0])
    err = np.abs(mind.cpu().numpy()[rows].astype(np.float64) - ref[1])
    assert np.all(err <= 2 * (D + 4) * (2.0 ** -24 if dtype == "f32" else 2.0 ** -53) * ref[1])


@pytest.mark.gpu
@pytest.mark.parametrize("dtype,N,D,K", [("f32", 30001, 32, 3000), ("f64", 20001, 40, 900), ("f32", 1500, 16, 1024),
                                         ("f32", 4300001, 4, 768), ("f64", 3001, 1160, 2000)])
def test_captured_assignment_replays_on_new_contents(dtype, N, D, K):
    """A recorded unprotected assignment (one launch of the scan and several, points that it lists: equal
    centroids) against the eager call on what the operands hold at each replay."""
    print("replay", dtype, N, D, K, flush=True)
    gen = torch.Generator(device="cuda").manual_seed(D)
    t = torch.float32 if dtype == "f32" else torch.float64
    X, C = torch.empty(N, D, device="cuda", dtype=t), torch.empty(K, D, device="cuda", dtype=t)

    def fill():
        C.normal_(generator=gen).mul_(5)
        C[K - 100:] = C[:100]
        pick = torch.randint(K, (N,), generator=gen, device="cuda")
        X.normal_(generator=gen).mul_(0.1).add_(C[pick])

    fill()
    ws = ftk.new_workspace(X, K, ftk.FT_OFF)
    labels = torch.empty(N, device="cuda", dtype=torch.int32)
    mind = torch.empty(N, device="cuda", dtype=t)
    ftk.kmeans_assign(X, C, labels, mind, workspace=ws)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        ftk.kmeans_assign(X, C, labels, mind, workspace=ws)
    for _ in range(4):
        fill()
        want = ftk.kmeans_assign(X, C)
        labels.fill_(-1)
        mind.fill_(-1)
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(labels, want[0]) and torch.equal(mind, want[1])
        assert int(labels.max()) < K - 100
