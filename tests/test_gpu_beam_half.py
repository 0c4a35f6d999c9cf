"""The fp16 pre-selection of the multi-path scoring at the sizes and values where it can go wrong: the kept candidates against
all K * Lc direct-form errors in fp64, position by position (equal errors in (l, k) order)."""
import numpy as np
import pytest

from parity_util import to_dev

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


# widths at the edges of a 32-column tile and of the doublings that cover a group; K and D at the edges of blocks, steps and of
# the dictionary that fits LDS; N one vector, a ragged tile, several
@pytest.mark.parametrize("kind", ["plain", "offset", "wild", "ties"])
@pytest.mark.parametrize("N,D,K,Lc,L", [(1, 4, 1, 1, 5), (3, 16, 2, 2, 2), (33, 20, 17, 3, 10), (50, 64, 33, 10, 10), (65, 100, 100, 16, 16),
                                        (40, 128, 256, 32, 32), (101, 128, 256, 1, 10), (97, 128, 256, 10, 12), (30, 256, 256, 5, 7),
                                        (40, 260, 256, 10, 10), (37, 512, 64, 11, 31), (20, 516, 129, 17, 20)])
def test_step_keeps_the_best(kind, N, D, K, Lc, L):
    from paper_1509_05194_amd import hclae
    rng = np.random.default_rng(D + K + Lc)
    C = rng.standard_normal((K, D)).astype(np.float32)
    rows = (C[rng.integers(0, K, (N, Lc))] + rng.standard_normal((N, Lc, D))).astype(np.float32)
    if kind == "offset":
        C += np.float32(300.0)
        rows += np.float32(300.0)
    elif kind == "wild":
        rows[::3, 0] *= np.float32(2e4)
        C[K // 2] *= np.float32(1e3)
    elif kind == "ties":
        C[K // 2:2 * (K // 2)] = C[:K // 2]
        rows[::2, Lc // 2:] = rows[::2, :1]
    Ln = min(L, K * Lc)
    ctx = hclae.Context(N, D, 1, K)
    rn = torch.empty((N, Ln, D), dtype=torch.float32, device="cuda:0")
    en = torch.empty((N, Ln), dtype=torch.float64, device="cuda:0")
    par = torch.empty((N, Ln), dtype=torch.uint8, device="cuda:0")
    cod = torch.empty((N, Ln), dtype=torch.uint8, device="cuda:0")
    err = (rows.astype(np.float64) ** 2).sum(2)
    ctx.beam_step(to_dev(rows), to_dev(err), to_dev(C), L, rn, en, par, cod)
    ctx.close()
    e = np.stack([((rows.astype(np.float64) - C[k].astype(np.float64)) ** 2).sum(2) for k in range(K)], 2).reshape(N, Lc * K)
    order = np.argsort(e, axis=1, kind="stable")[:, :Ln]
    best = np.take_along_axis(e, order, 1)
    got = par.cpu().numpy().astype(np.int64) * K + cod.cpu().numpy()
    assert got.max() < Lc * K
    # fp64 sums in another order: 1e-13 relative; neighbours closer than that may change places
    np.testing.assert_allclose(en.cpu().numpy(), best, rtol=1e-12, atol=0)
    np.testing.assert_allclose(np.take_along_axis(e, got, 1), best, rtol=1e-12, atol=0)
    assert all(len(set(row)) == Ln for row in got)
    same = got == order
    near = np.zeros_like(same)
    d = np.abs(np.diff(np.take_along_axis(e, np.argsort(e, axis=1, kind="stable")[:, :Ln + 1], 1), axis=1))
    tight = d <= 1e-12 * best[:, :d.shape[1]]
    near[:, :d.shape[1]] |= tight
    near[:, 1:] |= tight[:, :Ln - 1]
    assert np.all(same | near)
    want = rows[np.arange(N)[:, None], got // K] - C[got % K]
    np.testing.assert_array_equal(rn.cpu().numpy(), want)
