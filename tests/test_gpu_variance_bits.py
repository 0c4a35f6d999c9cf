"""The bits of the dictionary variances (Sec. 3.3): per coordinate a chain of additions for the mean and a chain of fused
multiply-adds for the squares, in ascending codeword order, then the sums of a block.  The fused step is rounded once, here by
way of exact fractions."""
from fractions import Fraction

import numpy as np
import pytest

from parity_util import to_dev

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def _fma(a, b, c):
    return float(Fraction(a) * Fraction(b) + Fraction(c))


def _variance(Cm):
    K, D = Cm.shape
    lanes = [0.0] * 256
    for d in range(D):
        s = 0.0
        for k in range(K):
            s += float(Cm[k, d])
        mu = s / K
        q = 0.0
        for k in range(K):
            t = float(Cm[k, d]) - mu
            q = _fma(t, t, q)
        lanes[d % 256] += q
    total = 0.0
    for w in range(4):
        v = lanes[64 * w:64 * w + 64]
        for o in (32, 16, 8, 4, 2, 1):
            v = [v[i] + v[i ^ o] for i in range(64)]
        total += v[0]
    return total / K


# more codewords than an unrolled run of 32 holds, with and without a remainder; rows of one lane group and of more than a block
@pytest.mark.parametrize("K,D", [(1, 4), (31, 16), (64, 8), (100, 68), (256, 12), (33, 260)])
def test_variance_bits(K, D):
    from paper_1509_05194_amd import hclae
    M = 2
    C = np.random.default_rng(K + D).standard_normal((M, K, D)).astype(np.float32)
    ctx = hclae.Context(8, D, M, K)
    var, _ = ctx.reorder_by_variance(to_dev(C), torch.zeros((8, M), dtype=torch.uint8, device="cuda:0"))
    ctx.close()
    np.testing.assert_array_equal(var, [_variance(C[m]) for m in range(M)])
