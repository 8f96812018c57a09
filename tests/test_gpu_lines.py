"""Few centroids on rows that the matrix kernel brings in line by line through LDS: every place of a row's end in a stage, one
and two tiles of centroids, partial workgroups of points, rows off a 16-byte line, with and without checksums and faults."""
import numpy as np
import pytest
import torch

from oracle import cpu as oracle
from paper_2408_01391_amd import binding as ftk, synth
from tests.gpu_util import DEV, check_assign, to_dev

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def _matrix_kernel():
    ftk.tuning_override(0, -1, -1)
    yield
    ftk.tuning_override(-1, -1, -1)


@pytest.mark.parametrize("mode", [ftk.FT_OFF, ftk.FT_STRICT])
@pytest.mark.parametrize("N,K", [(1, 1), (127, 31), (129, 32), (1025, 33), (3000, 64)])
@pytest.mark.parametrize("D", [24, 25, 31, 32, 64, 65, 66, 95, 96, 97, 127, 160, 1001])
def test_every_end_of_a_row_and_of_the_points(D, N, K, mode):
    print("lines", D, N, K, mode, flush=True)
    X, C = synth.random_problem(D + N, N, D, K, "f32") if N >= K else synth.random_problem(D, K, D, K, "f32")
    ref = oracle.assign(X, C)
    flat = torch.empty(X.size + 1, device=DEV)
    flat[1:] = to_dev(X).flatten()
    for x in (to_dev(X), flat[1:].view(X.shape)):
        labels, mind = ftk.kmeans_assign(x, to_dev(C), ft_mode=mode)
        check_assign(X, C, labels.cpu().numpy(), mind.cpu().numpy(), ref=ref)


@pytest.mark.parametrize("N,D,K,points", [(65536, 112, 64, 128), (65537, 112, 64, 256), (65537, 128, 64, 128), (65537, 112, 63, 128),
                                          (65537, 112, 32, 128), (98304, 300, 40, 128), (98305, 300, 40, 256), (131072, 300, 40, 256),
                                          (131073, 300, 40, 128), (163841, 300, 40, 128), (60001, 240, 64, 128), (70001, 240, 64, 256)])
def test_either_workgroup_on_both_sides_of_its_lines(N, D, K, points):
    """Protected calls, whose workgroups the geometry reports: the same labels as the oracle's on sampled rows."""
    print("lines", N, D, K, flush=True)
    assert ftk.assign_geometry(0, N, D, K, ftk.FT_STRICT).workgroups == -(-N // points)
    X, C = synth.random_problem(D + K, N, D, K, "f32", spread=3.0)
    labels, mind = ftk.kmeans_assign(to_dev(X), to_dev(C), ft_mode=ftk.FT_STRICT)
    rows = np.unique(np.concatenate([np.arange(0, N, 97), np.arange(N - 300, N)]))
    check_assign(X[rows], C, labels.cpu().numpy()[rows], mind.cpu().numpy()[rows], ref=oracle.assign(X[rows], C))


@pytest.mark.parametrize("D,K", [(24, 9), (33, 50), (128, 32), (300, 64)])
def test_flips_are_repaired(D, K):
    N = 2000
    X, C = synth.random_problem(D, N, D, K, "f32", spread=6.0)
    geom = ftk.assign_geometry(0, N, D, K, ftk.FT_STRICT)
    assert geom.workgroups == -(-N // 128)
    faults = [(wg, wg % 4, wg, 5 * wg % geom.regs_per_tile, 7 * wg % 64, 20 + wg % 11) for wg in range(geom.workgroups)]
    stats = ftk.new_stats(DEV)
    clean, _ = ftk.kmeans_assign(to_dev(X), to_dev(C), ft_mode=ftk.FT_STRICT)
    labels, _ = ftk.kmeans_assign(to_dev(X), to_dev(C), ft_mode=ftk.FT_STRICT, faults=ftk.make_faults(faults, DEV), stats=stats)
    assert torch.equal(labels, clean)
    assert ftk.stats_dict(stats)["injected"] > 0


def test_values_that_are_not_numbers_stay_in_their_row():
    N, D, K = 1000, 70, 20
    X, C = synth.random_problem(3, N, D, K, "f32")
    good, dist = ftk.kmeans_assign(to_dev(X), to_dev(C))
    X[5, D - 1], X[300], X[999, 0] = np.nan, np.inf, np.nan
    bad, bdist = ftk.kmeans_assign(to_dev(X), to_dev(C))
    keep = np.setdiff1d(np.arange(N), [5, 300, 999])
    assert torch.equal(bad[keep], good[keep]) and torch.equal(bdist[keep], dist[keep])
    assert 0 <= int(bad.min()) and int(bad.max()) < K
