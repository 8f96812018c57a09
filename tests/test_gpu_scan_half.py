"""The scan on fp16 pieces, which large unprotected assignments take where their rows allow it: widths and ragged rows of its compiled
variants, data that make it hand over to the bf16 pieces, points with more candidates than it notes, values beyond the
range of fp16, a workspace without room for it.  Sampled rows against the CPU oracle; every row against the same call
in parts that are too small for it.  Results are those of the bf16 form by design, so which form ran is told by the
points listed for the third pass: more than the bf16 form lists where it was fp16, no more where it was not."""
import numpy as np
import pytest
import torch

from oracle import cpu as oracle
from paper_2408_01391_amd import binding as ftk
from tests.gpu_util import DEV, check_assign, to_dev
from tests.test_gpu_scan import EPS, NP, run

pytestmark = pytest.mark.gpu


def blobs(seed, N, D, K, dtype):
    rng = np.random.default_rng(seed)
    centres = (rng.normal(size=(K, D)) * 5).astype(NP[dtype])
    X = rng.normal(size=(N, D)).astype(NP[dtype])
    X += centres[rng.integers(0, K, N)]
    return X, X[rng.permutation(N)[:K]].copy()


def counted(X, C, **kw):
    stats = ftk.new_stats(DEV)
    labels, mind = run(X, C, stats=stats, **kw)
    return labels, mind, ftk.stats_dict(stats)["refined"]


def in_parts(X, C):
    """The same by the bf16 form alone: parts of fewer rows than any call on fp16 pieces has."""
    out = [counted(p, C) for p in np.array_split(X, -(-len(X) // 32000))]
    return np.concatenate([o[0] for o in out]), np.concatenate([o[1] for o in out]), sum(o[2] for o in out)


def check(X, C, dtype, half, seed=0):
    """half: whether the call has to stay on fp16 pieces."""
    labels, mind, listed = counted(X, C)
    rows = np.sort(np.random.default_rng(seed).permutation(len(X))[:1500])
    lab_o, d1, d2 = ref = oracle.assign(X, C, rows)
    check_assign(X, C, labels, mind, rows=rows, ref=ref)
    # direct differences: D terms of at most 3 roundings each, the oracle's own included
    tol = 2 * (X.shape[1] + 4) * EPS[dtype]
    assert np.all(np.abs(mind[rows].astype(np.float64) - d1) <= tol * d1)
    lab_p, mind_p, listed_p = in_parts(X, C)
    print("listed", listed, "by two pieces", listed_p, flush=True)
    assert (listed > listed_p) == half
    assert np.array_equal(labels, lab_p)
    assert np.all(np.abs(mind.astype(np.float64) - mind_p) <= tol * mind_p)
    return labels


SIZES = [("f32", 300007, 17, 2950), ("f32", 250001, 33, 1900), ("f32", 130003, 64, 1805), ("f32", 100001, 97, 1550),
         ("f32", 60001, 128, 1960), ("f32", 100003, 129, 931), ("f32", 40001, 255, 1200), ("f32", 33001, 512, 720),
         ("f32", 32769, 513, 720), ("f32", 33333, 1024, 360), ("f64", 300007, 20, 6700), ("f64", 150001, 128, 2085),
         ("f64", 130003, 90, 3500), ("f64", 70001, 192, 900), ("f64", 33001, 1021, 357),
         ("f32", 530001, 130, 2100)]  # the last one in two launches, the second on the image of the first


@pytest.mark.parametrize("dtype,N,D,K", SIZES)
def test_labels_and_distances_at_the_edges(dtype, N, D, K):
    print("half", dtype, N, D, K, flush=True)
    check(*blobs(N + D, N, D, K, dtype), dtype, half=True)


@pytest.mark.parametrize("dtype,N,D,K", [("f32", 75001, 131, 1300), ("f32", 66017, 150, 1300), ("f32", 60007, 160, 1300), ("f32", 35009, 511, 700),
                                         ("f32", 33031, 1019, 400), ("f64", 70023, 203, 900), ("f64", 48001, 529, 480)])
def test_rows_that_end_anywhere_in_a_line(dtype, N, D, K):
    """Long rows are rounded 32 features of eight rows at a time: every place of a row's end among them, partial blocks of rows."""
    print("half", dtype, N, D, K, flush=True)
    check(*blobs(N + D, N, D, K, dtype), dtype, half=True)


# 25 and 35 tiles of centroids: rows of 3 and 6 blocks, whose bf16 image is padded by a tile more than the fp16 chunks take
@pytest.mark.parametrize("dtype,N,D,K", [("f32", 400001, 48, 800), ("f32", 290003, 47, 1120), ("f32", 210011, 96, 777),
                                         ("f32", 150001, 91, 1120), ("f64", 530001, 96, 800), ("f64", 750001, 48, 1119)])
def test_chunks_of_the_two_forms_that_pad_the_centroids_differently(dtype, N, D, K):
    print("half", dtype, N, D, K, flush=True)
    check(*blobs(N + D, N, D, K, dtype), dtype, half=True)


@pytest.mark.parametrize("dtype,N,D,K", [("f32", 130003, 64, 1805), ("f32", 33001, 512, 720), ("f64", 70001, 192, 900)])
@pytest.mark.parametrize("data", ["groups", "offset", "last points"])
def test_data_that_it_cannot_tell(data, dtype, N, D, K):
    X, C = blobs(D, N, D, K, dtype)
    rng = np.random.default_rng(1)
    if data == "groups":  # refused: every point has the centroids of its group within the bound
        X += np.where(rng.random(N) < 0.5, 300, -300)[:, None].astype(X.dtype)
        C = X[rng.permutation(N)[:K]].copy()
    elif data == "offset":
        X += X.dtype.type(400)
        C = C + C.dtype.type(400)
    else:  # more candidates than are noted, equal ones among them
        C[40:70] = C[5] + (rng.normal(size=(30, D)) * 1e-5).astype(C.dtype)
        C[50] = C[5]
        X[-400:] = C[5]
    labels = check(X, C, dtype, half=data == "last points")
    if data == "last points":
        assert np.all(labels[-400:] == 5)


@pytest.mark.parametrize("N,D,K", [(130003, 64, 1805), (33001, 512, 720)])
def test_values_beyond_fp16_and_values_that_are_not_numbers(N, D, K):
    X, C = blobs(D + 1, N, D, K, "f32")
    clean, mind = run(X, C)
    Xb = X.copy()
    Xb[7, 3], Xb[600, 0], Xb[N - 3, D - 1], Xb[9000, 5] = np.nan, np.inf, 3e38, 1e7
    labels, md = run(Xb, C)
    keep = np.ones(N, bool)
    keep[[7, 600, N - 3, 9000]] = False
    assert np.array_equal(labels[keep], clean[keep]) and np.array_equal(md[keep], mind[keep])
    assert labels.min() >= 0 and labels.max() < K
    rows = np.array([9000])
    check_assign(Xb, C, labels, rows=rows, ref=oracle.assign(Xb, C, rows))
    far = C.copy()
    far[17] = -1e8  # refused whatever the points' products with it
    bad = C.copy()
    bad[17] = np.nan
    a, b = run(X, far), run(X, bad)
    assert np.array_equal(a[0], b[0])
    assert np.all(np.abs(a[1].astype(np.float64) - b[1]) <= 2 * (D + 4) * EPS["f32"] * b[1])  # listed points: in double
    rows = np.arange(0, N, 97)
    check_assign(X, far, *a, rows=rows, ref=oracle.assign(X, far, rows))


# powers of two, so that the data are the same but for the exponent: squares of differences leave the range of their type
@pytest.mark.parametrize("dtype,N,D,K,exps", [("f32", 130003, 64, 1805, (-40, -55, -62, -67, -75, -84, 40, 75)),
                                              ("f32", 33001, 512, 720, (-62, -75, -84, 75)),
                                              ("f64", 150001, 128, 2085, (-515, -550, 505, 550)),
                                              ("f64", 70001, 192, 900, (-515, -550, 550))])
def test_labels_do_not_depend_on_the_scale_of_the_data(dtype, N, D, K, exps):
    rng = np.random.default_rng(D)
    X = rng.random((N, D)).astype(NP[dtype])  # nothing stands out: what one fp16 product names is often wrong
    C = X[rng.permutation(N)[:K]].copy()
    want = check(X, C, dtype, half=True)
    for e in exps:
        labels, mind = run(np.ldexp(X, e), np.ldexp(C, e))
        assert np.array_equal(labels, want), (e, int((labels != want).sum()))
        assert not np.isnan(mind).any()


@pytest.mark.parametrize("dtype,N,D,K", [("f64", 300007, 20, 6700), ("f32", 100003, 129, 931), ("f32", 33333, 1024, 360)])
def test_a_workspace_without_room_for_it(dtype, N, D, K):
    X, C = blobs(3, N, D, K, dtype)  # nothing else needs more of the workspace
    Xd, Cd = to_dev(X), to_dev(C)
    full = ftk.new_workspace(Xd, len(C), ftk.FT_OFF)
    labels, mind, listed = counted(X, C, workspace=full)
    lab2, mind2, listed2 = counted(X, C, workspace=torch.empty(full.numel() - 4096, dtype=full.dtype, device=DEV))
    assert np.array_equal(labels, lab2) and np.array_equal(mind, mind2)  # the form does not show
    _, _, listed_p = in_parts(X, C)
    assert listed > listed2 and abs(listed2 - listed_p) <= 0.01 * listed_p


def grouped(X, rows, off=40):
    """Two groups on either side of the origin, in these rows: the bf16 bound tells them, the fp16 bound does not."""
    X[rows] += np.where(np.random.default_rng(1).random(len(X[rows])) < 0.5, off, -off)[:, None].astype(X.dtype)
    return X


@pytest.mark.parametrize("dtype,N,D,K,rows", [
    ("f32", 400000, 32, 2000, slice(120000, None)),  # in order: all that comes first is easy
    ("f32", 130003, 256, 1024, slice(80000, None)),
    ("f64", 150001, 128, 2085, slice(0, 90000)),
    ("f32", 530001, 130, 2100, slice(0, 266240)),    # the first of two launches alone
])
def test_rows_in_any_order_choose_the_form_for_all_launches(dtype, N, D, K, rows):
    X, C = blobs(D, N, D, K, dtype)
    grouped(X, rows)
    check(X, X[np.random.default_rng(2).permutation(N)[:K]].copy(), dtype, half=False)


@pytest.mark.parametrize("N,D,K", [(130003, 64, 1805), (33001, 512, 720)])
def test_a_captured_call_replays_on_new_contents(N, D, K):
    X, C = blobs(4, N, D, K, "f32")
    X2, C2 = blobs(5, N, D, K, "f32")
    X2 += np.float32(400)  # the form is chosen anew by every replay
    C2 += np.float32(400)
    Xd, Cd = to_dev(X), to_dev(C)
    ws = ftk.new_workspace(Xd, K, ftk.FT_OFF)
    labels = torch.empty(N, dtype=torch.int32, device=DEV)
    mind = torch.empty(N, dtype=torch.float32, device=DEV)
    ftk.kmeans_assign(Xd, Cd, labels=labels, mindist=mind, workspace=ws)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        ftk.kmeans_assign(Xd, Cd, labels=labels, mindist=mind, workspace=ws)
    for x, c in ((X2, C2), (X, C), (X2, C2)):
        want = run(x, c)
        Xd.copy_(to_dev(x))
        Cd.copy_(to_dev(c))
        labels.fill_(-1)
        g.replay()
        torch.cuda.synchronize()
        assert np.array_equal(labels.cpu().numpy(), want[0])
        assert np.allclose(mind.cpu().numpy(), want[1], rtol=2 * (D + 4) * EPS["f32"], atol=0)
