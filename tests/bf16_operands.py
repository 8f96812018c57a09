"""Operands on which a reduction to two bf16 pieces loses as much as it can, with signs that push two
nearly equal scores apart in the wrong direction."""
from __future__ import annotations

import numpy as np

U = 2.0 ** -24
FIRST, SECOND = 5, 9  # the two centroids in question; FIRST is the nearer one


def bf16(x):
    """Round to nearest even at 8 significant bits, as a float64 (finite values of float32's range)."""
    b = np.asarray(x, np.float32).view(np.uint32)
    return ((b + 0x7FFF + ((b >> 16) & 1)) & 0xFFFF0000).astype(np.uint32).view(np.float32).astype(np.float64)


def pieces(v):
    """Two pieces of v and the residual that neither holds."""
    v = np.asarray(v, np.float64)
    p0 = bf16(v)
    p1 = bf16(v - p0)
    return p0, p1, v - p0 - p1


# magnitudes near 1 whose first remainder is +-2^-8 and whose second one is +-2^-17 (both a hair less)
_TINY = 2.0 ** -22
_MAG = {(+1, +1): 1 + 2.0 ** -8 - 2.0 ** -16 - 2.0 ** -17 - _TINY,
        (+1, -1): 1 + 2.0 ** -8 - 2.0 ** -16 - 2.0 ** -17 + _TINY,
        (-1, +1): 1 + 2.0 ** -8 + 2.0 ** -16 + 2.0 ** -17 - _TINY,
        (-1, -1): 1 + 2.0 ** -8 + 2.0 ** -16 + 2.0 ** -17 + _TINY}


def _signed(sign, first, second):
    """sign * magnitude with first remainder of sign `first` and residual of sign `second`."""
    return sign * _MAG[(first * sign, second * sign)]


def adversarial(D, K, a, four_products=False, moved=False, gap=4.0, copies=()):
    """X [8, D], C [K, D] float32: every point is nearest to centroid FIRST by `gap` u of ||x|| ||c||,
    while sums over two-piece products (without the product of the second pieces, unless
    four_products) prefer SECOND by all that such a sum can be off.  All other centroids are one
    vector; `moved`: the extremes are reached after that vector is subtracted from everything; `copies`:
    higher indices that repeat FIRST."""
    f = max(2, 2 * int(np.ceil((a * D / 2 + 1) / 2)))  # features on which both agree: they beat the rest
    half = (D - f) // 2
    s5, s9, sx = np.ones(D), np.ones(D), np.ones(D)
    s5[f + half:] = -1
    s9[f:f + half] = -1
    if (D - f) % 2:
        s9[D - 1] = -1  # the odd feature: the same for both
    sx[f + half:] = -1
    x = np.array([_signed(1, +1, int(sx[d])) for d in range(D)])
    # x1.c1 is lost unless four products are kept; x.r_c and r_x.c always
    c5 = np.array([_signed(int(s5[d]), +1, +1) for d in range(D)]) * a
    c9 = np.array([_signed(int(s9[d]), -1 if not four_products else +1, -1) for d in range(D)]) * a

    def score(c):
        return float(np.dot(x, c) - 0.5 * np.dot(c, c))

    want = gap * U * np.linalg.norm(x) * np.linalg.norm(c5)
    for _ in range(3):  # (float32 spacing of a feature is far below `want`)
        c5[0] = np.float32(c5[0] + (score(c9) + want - score(c5)) / (x[0] - c5[0]))
    other = np.full(D, -a / 2)
    C = np.tile(other if not moved else np.zeros(D), (K, 1))
    C[FIRST], C[SECOND] = c5, c9
    C[list(copies)] = c5
    X = np.tile(x, (8, 1))
    if moved:
        X, C = X + other, C + other
    Xf, Cf = X.astype(np.float32), C.astype(np.float32)
    d = ((Xf.astype(np.float64)[:1] - Cf.astype(np.float64)) ** 2).sum(1)
    assert int(np.argmin(d)) == FIRST and d[FIRST] < d[SECOND] < np.delete(d, [FIRST, SECOND, *copies]).min()
    return Xf, Cf


def truncated_scores(X, C, four_products=False):
    """Scores of the first point from the pieces, summed without rounding."""
    x0, x1, _ = pieces(X[0])
    c0, c1, _ = pieces(C)
    s = c0 @ x0 + c1 @ x0 + c0 @ x1 - 0.5 * (C.astype(np.float64) ** 2).sum(1)
    return s + c1 @ x1 if four_products else s
