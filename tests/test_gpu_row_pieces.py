"""Rows that are not whole 16-byte pieces, or do not begin on one, against the CPU oracle: every remainder of the last piece,
rows shorter than a piece, the last row of a buffer, with and without checksums; values that are not numbers stay in their row."""
import numpy as np
import pytest
import torch

from oracle import cpu as oracle
from paper_2408_01391_amd import binding as ftk, synth
from tests.gpu_util import DEV, check_assign, to_dev

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def _restore_rules():
    yield
    ftk.tuning_override(-1, -1, -1)


def _shifted(a):
    """the same values in a tensor that starts one element behind a 16-byte line and ends with its storage"""
    flat = torch.empty(a.size + 1, dtype=torch.from_numpy(a[:1]).dtype, device=DEV)
    flat[1:] = to_dev(a).flatten()
    return flat[1:].view(a.shape)


@pytest.mark.parametrize("mode", [ftk.FT_OFF, ftk.FT_STRICT])
@pytest.mark.parametrize("dtype,D", [("f32", d) for d in (1, 2, 3, 4, 5, 6, 7, 16, 17, 18, 19, 33, 67, 126, 131)]
                         + [("f64", d) for d in (1, 2, 3, 5, 16, 17, 33, 131)])
@pytest.mark.parametrize("K", [3, 40, 300])
def test_matrix_kernel_on_rows_of_any_length_and_alignment(dtype, D, K, mode):
    N = 700
    print("rows", dtype, D, K, mode, flush=True)
    X, C = synth.random_problem(D + K, N, D, K, dtype)
    ref = oracle.assign(X, C)
    ftk.tuning_override(0, -1, -1)
    for x, c in ((to_dev(X), to_dev(C)), (_shifted(X), _shifted(C))):
        labels, mind = ftk.kmeans_assign(x, c, ft_mode=mode)
        check_assign(X, C, labels.cpu().numpy(), mind.cpu().numpy(), ref=ref)


@pytest.mark.parametrize("mode", [ftk.FT_OFF, ftk.FT_STRICT])
def test_values_that_are_not_numbers_stay_in_their_row(mode):
    X, C = synth.random_problem(3, 500, 67, 20, "f32")
    ftk.tuning_override(0, -1, -1)
    good, _ = ftk.kmeans_assign(to_dev(X), to_dev(C), ft_mode=mode)
    X[7], X[300, 0] = np.nan, np.inf
    bad, _ = ftk.kmeans_assign(to_dev(X), to_dev(C), ft_mode=mode)
    keep = np.setdiff1d(np.arange(500), [7, 300])
    assert torch.equal(bad[keep], good[keep]) and 0 <= int(bad.min()) and int(bad.max()) < 20


@pytest.mark.parametrize("dtype,D", [("f32", 65), ("f32", 515), ("f64", 33), ("f64", 259)])
def test_refined_points_of_long_rows_with_a_remainder(dtype, D):
    """Equal centroids send their points to the refine kernel, whose lanes share a row here."""
    N, K = 900, 12
    X, C = synth.random_problem(D, N, D, K, dtype)
    C = np.concatenate([C, C, C])
    ftk.tuning_override(0, -1, -1)
    labels, mind = ftk.kmeans_assign(_shifted(X), _shifted(C))
    labels = labels.cpu().numpy()
    assert labels.max() < K
    check_assign(X, C, labels, mind.cpu().numpy())
