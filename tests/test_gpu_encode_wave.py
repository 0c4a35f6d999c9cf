"""The encoder of large calls (a tile of 32 vectors per wave, rows up to 128 coordinates): a vector's codes and residual do not depend on
the vectors beside it, so they are the bits that small calls give, which another kernel takes (checked against the oracle elsewhere).
Row lengths and dictionaries at the edges of the kernel's instances, one and several tiles to a wave, ragged ends, and data whose
vectors have many candidates or exact ties."""
import numpy as np
import pytest

from parity_util import to_dev

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def _data(kind, N, D, M, K, rng):
    C = rng.standard_normal((M, K, D), np.float32) * np.float32(0.7)
    X = C[0, rng.integers(0, K, N)] + np.float32(0.8) * rng.standard_normal((N, D), np.float32)
    if kind == "offset":
        X += np.float32(300)
        C[0] += np.float32(300)
    elif kind == "groups":
        X[::3] += np.float32(30)
        C[0, ::2] += np.float32(30)
    elif kind == "tiny":
        C *= np.float32(1e-4)
    elif kind == "wild":
        X[::7] *= np.float32(3e4)
        C[0, K // 2] *= np.float32(2e3)
    elif kind == "twins":
        C[:, K // 2:2 * (K // 2)] = C[:, :K // 2]
    elif kind == "zero":
        C[M - 1] = 0
    elif kind == "huge":
        X *= np.float32(1e20)
        C *= np.float32(1e20)
    return X, C


def _same_as_small_calls(X, C, piece):
    from paper_1509_05194_amd import hclae
    N, D = X.shape
    M, K, _ = C.shape
    Xg, Cg = to_dev(X), to_dev(C)
    ctx = hclae.Context(N, D, M, K)
    codes, r = torch.full((N, M), 7, dtype=torch.uint8, device="cuda:0"), torch.empty_like(Xg)
    ctx.encode(Xg, Cg, codes, r)
    torch.cuda.synchronize()
    ctx.close()
    ctx = hclae.Context(piece, D, M, K)
    for n in range(0, N, piece):
        m = min(piece, N - n)
        c, q = torch.zeros((m, M), dtype=torch.uint8, device="cuda:0"), torch.empty((m, D), device="cuda:0")
        ctx.encode(Xg[n:n + m].contiguous(), Cg, c, q)
        torch.cuda.synchronize()
        assert torch.equal(codes[n:n + m], c), "codes of %d.." % n
        # nan: what exceeds fp32 subtracts from itself
        assert torch.equal(torch.nan_to_num(r[n:n + m], nan=1.5), torch.nan_to_num(q, nan=1.5)), "residues of %d.." % n
    ctx.close()


@pytest.mark.parametrize("N,D,M,K", [(20000 + 9, 128, 3, 256), (140000 + 1, 128, 2, 256), (20000, 100, 4, 200), (17000, 124, 2, 129),
                                     (9000 + 31, 64, 3, 256), (140000 + 33, 60, 3, 255), (9001, 4, 2, 130),
                                     (50000 + 5, 128, 2, 128), (34000, 64, 2, 65), (50000, 68, 3, 64), (34000 + 1, 32, 3, 33),
                                     (50001, 128, 2, 32), (34001, 16, 4, 16), (50000, 72, 2, 1)])
def test_large_calls_equal_small_ones(N, D, M, K):
    _same_as_small_calls(*_data("plain", N, D, M, K, np.random.default_rng(D + K)), 8000)


@pytest.mark.parametrize("kind", ["offset", "groups", "tiny", "wild", "twins", "zero", "huge"])
@pytest.mark.parametrize("N,D,M,K", [(20000 + 3, 128, 2, 256), (9000 + 1, 52, 3, 140), (34000, 100, 2, 96)])
def test_many_candidates_and_ties(kind, N, D, M, K):
    _same_as_small_calls(*_data(kind, N, D, M, K, np.random.default_rng(K)), 4000)


@pytest.mark.parametrize("kind", ["groups", "tiny", "zero", "some", "late"])
@pytest.mark.parametrize("N,D,M,K", [(140000 + 5, 128, 1, 256), (140000 + 5, 64, 3, 200), (210000, 76, 2, 33), (80000 + 31, 20, 5, 130)])
def test_tiles_left_to_the_second_launch(kind, N, D, M, K):
    """Several rounds of tiles: all left from the first round on, or from some dictionary on, or few of them (at different dictionaries)."""
    rng = np.random.default_rng(N + D)
    X, C = _data(kind if kind in ("groups", "tiny", "zero") else "plain", N, D, M, K, rng)
    if kind == "some":                                   # vectors between all the codewords of one dictionary
        C[1:] *= np.float32(0.3)
        for m in range(M):
            X[100 + 700 * m::5000] = C[:m].sum(0)[0] if m else 0
            C[m, K // 2:] *= np.float32(1e-3)
    elif kind == "late":
        C[M // 2 + (M > 1):] *= np.float32(1e-4)
    _same_as_small_calls(X, C, 8000)
