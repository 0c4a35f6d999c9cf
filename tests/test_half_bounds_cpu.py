"""The bound E_k = e w_k + h of the fp16 pre-selection as an arithmetic fact, in the kernel's own precision: the score of every
codeword that the rounded operands give, less the most that the accumulation may lose, is within E_k of the exact one -- and where
the roundings all point the same way it comes so near that a bound half as large would not hold."""
import numpy as np
import pytest

UNIT = np.float32(17.0 * 2.0 ** -23)
TINY = 2.0 ** -14


def _round(v, scale, neg):
    """Scaled, centred fp32 coordinates, their fp16 values, ||.||^2 and the square of what the rounding left out."""
    c = (v.astype(np.float64) * scale + neg).astype(np.float32)
    q = c.astype(np.float16)
    d = c.astype(np.float64) - q.astype(np.float64)
    return c, q.astype(np.float64), (c.astype(np.float64) ** 2).sum(1), (d * d).sum(1)


def _bound(X, C):
    """(largest error of a score over its bound, largest over the part of the bound that is not the accumulation's)"""
    K, D = C.shape
    NC = (D + 63) // 64
    h = 0.5 * (C.astype(np.float64) ** 2).sum(1).max()
    scale = 2.0 ** (7 - np.frexp(np.float32(np.sqrt(2 * h)))[1])
    rows = C[(np.arange(8) * K) // 8]
    neg = (rows.sum(0, dtype=np.float32) * np.float32(-scale / 8)).astype(np.float32)
    c32, cq, sq, dsq = _round(C, scale, neg)
    x32, xq, x2, dx2 = _round(X, scale, neg)
    # constants of the dictionary
    cmax = np.sqrt(sq.max()) * 1.001
    wk = np.maximum(np.sqrt(sq) * 1.001, cmax / 256)
    rho = ((np.sqrt(dsq) * 1.001 + wk * 1.2e-7) / wk).max()
    acc = (4 * NC + 3) * UNIT
    hc = acc * (0.501 * sq.max() + 6.2e-5 * cmax + 3.8e-9)
    w = (wk * 1.002 + 6e-8).astype(np.float16).astype(np.float64)
    # of the vectors
    xn = np.sqrt(x2) * 1.001
    dx = np.sqrt(dx2) * 1.001 + xn * 1.2e-7
    e = np.maximum((dx * (1 + rho) + xn * (rho + acc * (1 + rho))) * 1.002, 6.2e-5).astype(np.float16).astype(np.float64)
    E = e[:, None] * w[None] + hc + (acc * 6.2e-5 * xn)[:, None]
    # exact scores of the scaled, centred data; those of the rounded operands; the most the accumulation may lose of the latter
    Xe = X.astype(np.float64) * scale + neg
    Ce = C.astype(np.float64) * scale + neg
    exact = Xe @ Ce.T - 0.5 * (Ce * Ce).sum(1)
    got = xq @ cq.T + (-0.5 * sq).astype(np.float32).astype(np.float64)
    p = np.maximum(np.abs(xq), TINY).max(1)[:, None] * np.maximum(np.abs(cq), TINY).max(1)[None]
    largest = np.maximum(np.maximum(p, 0.5 * sq[None]), np.sqrt(x2)[:, None] * np.sqrt(sq)[None] + 0.5 * sq[None])
    lost = (4 * NC + 1) * float(UNIT) * np.maximum(largest, e[:, None] * w[None])
    err = np.abs(exact - got)
    return float(((err + lost) / E).max()), float((err / (e[:, None] * w[None])).max())


@pytest.mark.parametrize("D", [4, 16, 64, 128, 960])
@pytest.mark.parametrize("kind", ["plain", "residues", "offset", "far offset", "small spread", "exact", "one long codeword", "long vectors",
                                  "one coordinate"])
def test_bound_holds(kind, D):
    g = np.random.default_rng(D)
    K, N = 64, 300
    C = g.standard_normal((K, D))
    X = C[g.integers(0, K, N)] + 0.5 * g.standard_normal((N, D))
    if kind == "residues":
        X = np.rint(40 * X) / 7
        C = np.rint(40 * C) / 7
    elif kind == "offset":
        X, C = X + 900, C + 900
    elif kind == "far offset":           # centred coordinates below fp16's normal numbers
        X, C = X + 1e5, C + 1e5
    elif kind == "small spread":
        C = 50 + 2.0 ** -16 * np.rint(4 * C)
        X = 50 + 0.25 * X
    elif kind == "exact":                # numbers that fp16 holds
        X, C = np.rint(16 * X), np.rint(16 * C)
    elif kind == "one long codeword":
        C[1] *= 1000
    elif kind == "long vectors":
        X *= 300
    elif kind == "one coordinate":       # codewords a few units of the last place apart: subnormal against one large coordinate
        C = 50 + 2.0 ** -18 * np.rint(2 * C)
        X = 50 + 0 * X
        X[:, 0] += 8
    over, _ = _bound(X.astype(np.float32), C.astype(np.float32))
    print("%s, D = %d: largest error %.2f of the bound" % (kind, D, over))
    assert over <= 1.0


@pytest.mark.parametrize("which", ["vector", "codeword"])
def test_half_the_bound_would_not_hold(which):
    """Roundings that all point the same way, along the other operand: the norms bound them with equality."""
    K, D = 16, 64
    sign = np.array([1.0, 1.0, -1.0, -1.0] * 4)              # the rows whose mean centres the scores cancel
    C = sign[:, None] * np.ones((K, D))
    X = np.ones((4, D))
    if which == "vector":
        X *= 1 + 2.0 ** -11 * 0.49                           # rounds to one
    else:
        C *= 1 + 2.0 ** -11 * 0.49
    over, rounding = _bound(X.astype(np.float32), C.astype(np.float32))
    print("%s: %.2f of the bound, its rounding part %.2f" % (which, over, rounding))
    assert over <= 1.0 and rounding > 0.8
