"""Fits whose outputs lie over their inputs: centroids that replace the initial ones, in place or some elements further on,
and centroids that take the place of the first points.  The objective of every iteration, whose partial sums the block
that ends last adds up."""
import numpy as np
import pytest
import torch

from paper_2408_01391_amd import binding as ftk
from tests.gpu_util import DEV

pytestmark = pytest.mark.gpu

# in one launch an iteration; through the matrix kernels; through the scan; in double
SHAPES = [(4096, 16, 8, torch.float32, ftk.FT_OFF), (3000, 40, 30, torch.float32, ftk.FT_STRICT),
          (70000, 32, 900, torch.float32, ftk.FT_OFF), (5000, 33, 60, torch.float64, ftk.FT_OFF)]


def _fit(X, K, iters, C_init, C_out, mode, like):
    N, D = like.shape
    labels = torch.empty(N, dtype=torch.int32, device=DEV)
    counts = torch.empty(K, dtype=torch.int32, device=DEV)
    ws = ftk.new_workspace(like, K, mode)
    wp, wn = ftk._ws_args(ws)
    ftk._check(ftk.load().ftk_kmeans_fit(ftk._dtype_code(like), X.data_ptr(), N, D, K, iters, 7, ftk._ptr(C_init),
                                         C_out.data_ptr(), labels.data_ptr(), counts.data_ptr(), None, mode, None, wp, wn,
                                         ftk._stream()))
    torch.cuda.synchronize()
    return C_out.clone(), labels, counts


@pytest.mark.parametrize("iters", [0, 1, 3])
@pytest.mark.parametrize("N,D,K,dtype,mode", SHAPES)
def test_outputs_over_inputs(N, D, K, dtype, mode, iters):
    gen = torch.Generator(device=DEV).manual_seed(N)
    X = torch.randn(N, D, generator=gen, device=DEV, dtype=dtype) * 3
    C0 = X[torch.randperm(N, generator=gen, device=DEV)[:K]].contiguous()
    want = _fit(X, K, iters, C0, torch.empty_like(C0), mode, X)
    n = K * D
    for first, out in ((0, 0), (0, 4), (4, 0), (0, D), (3 * D, 0), (0, 1), (1, 1)):
        print("fit", N, D, K, iters, first, out, flush=True)
        both = torch.empty(n + 4 * D, device=DEV, dtype=dtype)
        C_init = both[first:first + n].view(K, D)
        C_init.copy_(C0)
        got = _fit(X, K, iters, C_init, both[out:out + n].view(K, D), mode, X)
        assert torch.equal(got[0], want[0])
        if iters:
            assert torch.equal(got[1], want[1]) and torch.equal(got[2], want[2])
    for C_init in (C0, None):
        want = _fit(X, K, iters, C_init, torch.empty_like(C0), mode, X)
        over = X.clone()
        got = _fit(over, K, iters, C_init, over[:K], mode, X)
        assert torch.equal(got[0], want[0]) and torch.equal(over[K:], X[K:])
        if iters:
            assert torch.equal(got[1], want[1]) and torch.equal(got[2], want[2])


@pytest.mark.parametrize("dtype", [torch.float32, torch.float64])
@pytest.mark.parametrize("N", [1, 255, 2048, 2049, 100003, 262144, 700001])
def test_objective_of_every_iteration(N, dtype):
    """One block, two, all 128; the ticket starts over for each of 12 iterations, and each fit gives the same bits."""
    gen = torch.Generator(device=DEV).manual_seed(N)
    X = torch.randn(N, 5, generator=gen, device=DEV, dtype=dtype)
    C0 = torch.randn(3, 5, generator=gen, device=DEV, dtype=dtype)
    runs = [ftk.kmeans_fit(X, 3, 12, C_init=C0, ft_mode=ftk.FT_STRICT)["inertia"] for _ in range(3)]
    assert np.array_equal(runs[0], runs[1]) and np.array_equal(runs[0], runs[2])
    want, C = [], C0
    for _ in range(12):
        labels, mind = ftk.kmeans_assign(X, C, ft_mode=ftk.FT_STRICT)
        want.append(float(mind.double().sum()))
        C, _ = ftk.kmeans_update(X, labels, C.clone(), ft_mode=ftk.FT_STRICT)
    # N terms of one sign in double, added up in two orders
    assert np.all(np.abs(runs[0] - want) <= 2 * N * 2.0 ** -53 * np.abs(want))
