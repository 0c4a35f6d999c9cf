"""Centroid updates after many vectors have moved sum all of them instead of those that moved, decided on the device: stages whose
dictionaries start far from their data end in the bits of single steps, which always sum everything."""
import numpy as np
import pytest

from parity_util import to_dev

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

FULL = 4                                     # all vectors are summed from a share of 1 / FULL of them on
DIRECT = 2 ** 17                             # up to so many additions of one sign the moved ones go to memory one by one


def _poor_start(N, D, K):
    """Rows of three skewed latent coordinates, and codewords all near one of them: half of the vectors move at first, then fewer and fewer."""
    g = np.random.default_rng(N)
    z = g.random((N, 3), np.float32) ** 3
    X = 4 * z @ g.standard_normal((3, D)).astype(np.float32) + np.float32(0.02) * g.standard_normal((N, D), np.float32)
    C0 = X[:1] + np.float32(0.001) * g.standard_normal((K, D), np.float32)
    C0[0] = X.mean(0)
    return X, C0[None]


# around a block's least share of 1024 rows and of two such blocks, with rows so long that a quarter of the vectors is more than the short way
# out takes; many blocks, several windows of coordinates and a ragged one
@pytest.mark.parametrize("N,D,K", [(1023, 1024, 40), (1024, 1024, 40), (1025, 1020, 40), (2047, 1024, 70), (2048, 516, 40), (2049, 1024, 40),
                                   (70000, 20, 256), (9000, 960, 100), (300000, 32, 64)])
def test_stage_from_a_poor_dictionary(N, D, K):
    from paper_1509_05194_amd import hclae
    assert N // FULL * D > DIRECT
    X, C0 = _poor_start(N, D, K)
    iters = 10
    ctx = hclae.Context(N, D, 1, K)
    r0 = X - C0[0, 0]
    Cs, cs, rs = to_dev(C0), torch.zeros((N, 1), dtype=torch.uint8, device="cuda:0"), to_dev(r0)
    ctx.heat(0, Cs, cs, rs)
    moved = []
    for _ in range(iters):
        before = cs.clone()
        ctx.assign(0, rs, Cs, cs)
        ctx.update(0, rs, Cs, cs)
        moved.append(int((before != cs).sum()))
    ctx.assign(0, rs, Cs, cs)
    ctx.cool(0, Cs, cs, rs)
    # (the first update sums everything in any case)
    assert any(FULL * n > N for n in moved[1:]) and any(FULL * n <= N for n in moved[1:]), moved
    C, codes, r = to_dev(C0), torch.zeros((N, 1), dtype=torch.uint8, device="cuda:0"), to_dev(r0)
    ctx.anneal_stage(0, C, codes, r, iters)
    torch.cuda.synchronize()
    assert torch.equal(C, Cs) and torch.equal(codes, cs) and torch.equal(r, rs)
    ctx.close()


@pytest.mark.parametrize("N,D,K", [(1023, 16, 16), (1024, 64, 40), (1025, 60, 40), (70000, 20, 256), (9000, 60, 100)])
def test_improved_stage_equals_its_steps(N, D, K):
    """The stage on growing prefixes of the rotated coordinates, which sums every vector in each update, from such a start."""
    from paper_1509_05194_amd import hclae
    X, C0 = _poor_start(N, D, K)
    ctx = hclae.Context(N, D, 1, K)
    r0 = X - C0[0, 0]
    C, codes, r = to_dev(C0), torch.zeros((N, 1), dtype=torch.uint8, device="cuda:0"), to_dev(r0)
    R = ctx.pca_axes(to_dev(X))
    R = R[0] if isinstance(R, tuple) else R
    dims = [2, 5, 11, D]
    ctx.anneal_stage_pca(0, C, codes, r, R, dims, 2, torch.empty_like(r))
    Cs, cs, rs = to_dev(C0), torch.zeros((N, 1), dtype=torch.uint8, device="cuda:0"), to_dev(r0)
    ctx.heat(0, Cs, cs, rs)
    rot, back = torch.empty_like(Cs[0]), torch.empty_like(Cs[0])
    ctx.rotate(Cs[0].contiguous(), R, rot)
    Cr, xs = rot[None].contiguous(), torch.empty_like(rs)
    ctx.rotate(rs, R, xs)
    for d in dims:
        for _ in range(2):
            ctx.assign_prefix(0, xs, Cr, cs, d)
            ctx.update(0, xs, Cr, cs)
    ctx.rotate(Cr[0].contiguous(), R, back, transpose=True)
    Cs = back[None].contiguous()
    ctx.assign(0, rs, Cs, cs)
    ctx.cool(0, Cs, cs, rs)
    torch.cuda.synchronize()
    assert torch.equal(C, Cs) and torch.equal(codes, cs) and torch.equal(r, rs)
    ctx.close()
