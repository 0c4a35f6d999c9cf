"""Centroid updates after most vectors have moved sum all of them instead of those that moved, decided on the device: stages whose
dictionaries start far from their data end in the bits of single steps, which always sum everything.  Few and many moved vectors, and
sizes around a block's least share of 1024 rows."""
import numpy as np
import pytest

from parity_util import to_dev

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("improved", [False, True])
@pytest.mark.parametrize("N,D,K", [(1023, 16, 16), (1024, 64, 40), (1025, 130 * 4, 40), (70000, 20, 256), (9000, 960, 100)])
def test_stage_from_a_poor_dictionary(N, D, K, improved):
    from paper_1509_05194_amd import hclae
    if improved and D > 64:
        D = 60
    g = np.random.default_rng(N)
    X = (g.standard_normal((max(4, K // 3), D))[g.integers(0, max(4, K // 3), N)] + 0.5 * g.standard_normal((N, D))).astype(np.float32)
    C0 = (X[g.choice(N, K)] * 0.05 + 0.5 * g.standard_normal((K, D)))[None].astype(np.float32)
    iters = 8
    ctx = hclae.Context(N, D, 1, K)
    r0 = X - C0[0, 0]
    C, codes, r = to_dev(C0), torch.zeros((N, 1), dtype=torch.uint8, device="cuda:0"), to_dev(r0)
    if improved:
        R = ctx.pca_axes(to_dev(X))
        R = R[0] if isinstance(R, tuple) else R
        dims = [2, 5, 11, D]
        xr = torch.empty_like(r)
        ctx.anneal_stage_pca(0, C, codes, r, R, dims, 2, xr)
    else:
        ctx.anneal_stage(0, C, codes, r, iters)
    Cs, cs, rs = to_dev(C0), torch.zeros((N, 1), dtype=torch.uint8, device="cuda:0"), to_dev(r0)
    ctx.heat(0, Cs, cs, rs)
    if improved:
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
    else:
        for _ in range(iters):
            ctx.assign(0, rs, Cs, cs)
            ctx.update(0, rs, Cs, cs)
    ctx.assign(0, rs, Cs, cs)
    ctx.cool(0, Cs, cs, rs)
    torch.cuda.synchronize()
    assert torch.equal(C, Cs) and torch.equal(codes, cs) and torch.equal(r, rs)
    ctx.close()
