"""The eigen-solver's loops, blocked over columns and compiled for the host's vector unit, against the plain loops they stand
for (here with numpy, one operation per element and step): the same bits, around the edges of the blocks (8 and 32 columns,
4 rows, 4096 queued rotations) and for a matrix that is not symmetric to the last bit."""
import numpy as np
import pytest

from paper_1509_05194_amd import hclae


def _dot(a, b):
    s = np.float64(0.0)
    for x, y in zip(a, b):
        s = s + x * y
    return s


def _plain(A):
    A = A.copy()
    n = len(A)
    d, e, beta = np.zeros(n), np.zeros(max(n - 1, 1)), np.zeros(n)
    for k in range(n - 2):
        x = A[k, k + 1:]
        tail = _dot(x[1:], x[1:])
        d[k] = A[k, k]
        if tail == 0.0:
            e[k] = x[0]
            continue
        norm = np.sqrt(x[0] * x[0] + tail)
        alpha = -norm if x[0] > 0.0 else norm
        e[k] = alpha
        x[0] -= alpha
        b = 2.0 / (x[0] * x[0] + tail)
        beta[k] = b
        B = A[k + 1:, k + 1:]
        s = np.zeros(len(x))
        for j in range(len(x)):
            s = s + B[:, j] * x[j]
        p = b * s
        vp = _dot(x, p)
        p = p - (0.5 * b * vp) * x
        B -= np.multiply.outer(x, p) + np.multiply.outer(p, x)
    if n >= 2:
        d[n - 2], e[n - 2] = A[n - 2, n - 2], A[n - 2, n - 1]
    d[n - 1] = A[n - 1, n - 1]
    V = np.eye(n)
    for k in range(n - 3, -1, -1):
        if beta[k] == 0.0:
            continue
        v, Q = A[k, k + 1:], V[k + 1:, k + 1:]
        u = np.zeros(len(v))
        for i in range(len(v)):
            u = u + v[i] * Q[i]
        Q -= np.multiply.outer(beta[k] * v, u)
    V = V.T.copy()
    while True:
        for i in range(n - 1):
            if abs(e[i]) <= 2.220446049250313e-16 * (abs(d[i]) + abs(d[i + 1])):
                e[i] = 0.0
        hi = n - 1
        while hi > 0 and e[hi - 1] == 0.0:
            hi -= 1
        if hi == 0:
            break
        lo = hi - 1
        while lo > 0 and e[lo - 1] != 0.0:
            lo -= 1
        dd, off = 0.5 * (d[hi - 1] - d[hi]), e[hi - 1]
        den = dd + (1.0 if dd >= 0.0 else -1.0) * np.hypot(dd, off)
        mu = d[hi] - (off * off / den if den != 0.0 else 0.0)
        x, z = d[lo] - mu, e[lo]
        for k in range(lo, hi):
            r = np.hypot(x, z)
            c, s = (x / r, -z / r) if r != 0.0 else (np.float64(1.0), np.float64(0.0))
            if k > lo:
                e[k - 1] = r
            a, b, g = d[k], e[k], d[k + 1]
            d[k] = c * c * a - 2.0 * c * s * b + s * s * g
            d[k + 1] = s * s * a + 2.0 * c * s * b + c * c * g
            e[k] = c * s * (a - g) + (c * c - s * s) * b
            if k + 1 < hi:
                x, z = e[k], -s * e[k + 1]
                e[k + 1] = c * e[k + 1]
            V[k], V[k + 1] = c * V[k] - s * V[k + 1], s * V[k] + c * V[k + 1]
    order = np.argsort(-d, kind="stable")
    V = V[order]
    at = np.argmax(np.abs(V), axis=1)
    return d[order], V * np.where(V[np.arange(n), at] < 0.0, -1.0, 1.0)[:, None]


@pytest.mark.parametrize("n", [1, 2, 3, 5, 8, 9, 31, 32, 33, 41, 100])
def test_same_bits_as_the_plain_loops(n):
    B = np.random.default_rng(n).standard_normal((n, n))
    uneven = B + B.T
    uneven[0, -1] *= 1.0 + 2.0 ** -50
    for A in (B + B.T, B @ np.diag(np.arange(n) % 3.0) @ B.T, uneven):
        A = A if A is uneven else 0.5 * (A + A.T)
        w, Vt = hclae.symmetric_eigen(A)
        w0, V0 = _plain(A)
        np.testing.assert_array_equal(w, w0)
        np.testing.assert_array_equal(Vt, V0)
