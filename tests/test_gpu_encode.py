"""The fused greedy encoder (Eq. 3 with one path) against the same steps taken one by one -- assign, subtract, dictionary by
dictionary -- bit for bit, at the edges of its tiles, waves and chunks and with ties."""
import numpy as np
import pytest

from parity_util import to_dev

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


# K: 1, 2, 4 and 8 waves to a block; D: 1, 2 and 4 chunks (one that rounds up) and rows too long for the fused kernel;
# N: one vector, the edges of a 32-vector tile, and a call that the encoder with a tile per wave takes
@pytest.mark.parametrize("kind", ["plain", "ties", "spread"])
@pytest.mark.parametrize("N,D,M,K", [(1, 4, 1, 1), (31, 16, 4, 16), (33, 64, 3, 32), (65, 100, 2, 20), (95, 60, 3, 33),
                                     (1000, 128, 4, 64), (777, 200, 2, 50), (513, 68, 3, 65), (600, 128, 8, 128),
                                     (64, 256, 2, 100), (1, 128, 8, 256), (2050, 128, 8, 256), (300, 36, 5, 200),
                                     (129, 132, 3, 256), (260, 256, 2, 129), (100, 260, 2, 256), (70, 512, 2, 17),
                                     (49152 + 33, 16, 2, 140)])
def test_encode_equals_its_steps(kind, N, D, M, K):
    from paper_1509_05194_amd import hclae
    rng = np.random.default_rng(N + D + K)
    C = rng.standard_normal((M, K, D)).astype(np.float32) / np.float32(3) ** np.arange(M, dtype=np.float32)[:, None, None]
    X = sum(C[m][rng.integers(0, K, N)] for m in range(M)) + np.float32(0.05) * rng.standard_normal((N, D)).astype(np.float32)
    if kind == "ties":
        C[:, K // 2:2 * (K // 2)] = C[:, :K // 2]            # every codeword twice
        X[::5] = 0.0
        X[1::9] *= np.float32(1e5)                           # rows beyond the range the dictionaries set
        C[M - 1] = 0.0                                       # every score ties
    if kind == "spread":                                     # norms over several orders: many candidates
        f = np.exp(2 * rng.standard_normal((M, K, 1)))
        C = (C * f).astype(np.float32)
        X = X * np.exp(2 * rng.standard_normal((N, 1)))
    X = X.astype(np.float32)
    Xg, Cg = to_dev(X), to_dev(C)
    ctx = hclae.Context(N, D, M, K)
    codes = torch.full((N, M), 9, dtype=torch.uint8, device="cuda:0")
    r = torch.empty_like(Xg)
    for _ in range(2):
        ctx.encode(Xg, Cg, codes, r)
    want, rw = torch.full_like(codes, 9), Xg.clone()
    for m in range(M):
        ctx.assign(m, rw, Cg, want)
        ctx.cool(m, Cg, want, rw)
    assert torch.equal(codes, want)
    assert torch.equal(r, rw)
    ctx.work_counters(reset=True)
    ctx.encode(Xg, Cg, codes, r)
    a, v, f = ctx.work_counters()
    assert (a, v) == (M, M * N) and 0 <= ctx.last_refined() <= f <= v
    ctx.close()


def test_encode_with_more_tiles_than_blocks():
    """From 2^20 tiles of 32 vectors a block takes several of them."""
    from paper_1509_05194_amd import hclae
    N, D, M, K = (1 << 25) + 32 * 3 + 5, 4, 2, 16
    g = torch.Generator(device="cuda").manual_seed(3)
    X = torch.randn((N, D), generator=g, device="cuda")
    C = torch.randn((M, K, D), generator=g, device="cuda")
    ctx = hclae.Context(N, D, M, K)
    codes = torch.full((N, M), 9, dtype=torch.uint8, device="cuda:0")
    r = torch.full_like(X, 9.0)
    ctx.encode(X, C, codes, r)
    want, rw = torch.full_like(codes, 9), X.clone()
    for m in range(M):
        ctx.assign(m, rw, C, want)
        ctx.cool(m, C, want, rw)
    assert torch.equal(codes, want)
    assert torch.equal(r, rw)
    ctx.close()


# 256 CUs.  Three ways to encode, told apart by the launches that decide: one (a tile for all waves of a block), two (a tile per wave; the
# second takes up what the first leaves) or one per dictionary.  Rows of up to 64 and 128 coordinates change from the first to the
# second above 4 and 6 tiles of 32 vectors per CU (K <= 64), 4 (K <= 128), 1 and 2; longer ones from the first to the third above 12 and,
# from D = 208 on, 48 (K <= 64), 16 and never (K <= 128), 6.  N: at the line and one more
@pytest.mark.parametrize("N,D,K,launches", [
    (32768, 64, 32, 1), (32769, 64, 32, 2), (32769, 16, 33, 2), (49152, 68, 32, 1), (49153, 128, 64, 2),
    (32768, 16, 65, 1), (32769, 16, 65, 2), (32768, 128, 128, 1), (32769, 128, 128, 2), (32769, 68, 65, 2),
    (8192, 64, 129, 1), (8193, 64, 129, 2), (8193, 4, 256, 2), (16384, 68, 129, 1), (16385, 128, 256, 2), (400000, 20, 64, 2),
    (98304, 132, 33, 1), (98305, 204, 64, 3), (393216, 208, 33, 1), (393217, 208, 64, 3),
    (131072, 132, 65, 1), (131073, 204, 65, 3), (131073, 208, 65, 1), (49152, 132, 140, 1), (49153, 256, 140, 3),
    (100, 260, 20, 3), (100, 132, 32, 3)])
def test_encoder_by_size(N, D, K, launches):
    """The encoders on either side of the lines between them."""
    from paper_1509_05194_amd import hclae
    M = 3
    g = torch.Generator(device="cuda").manual_seed(N + K)
    C = torch.randn((M, K, D), generator=g, device="cuda") * torch.tensor([1.0, 0.5, 0.3], device="cuda")[:, None, None]
    X = torch.randn((N, D), generator=g, device="cuda")
    ctx = hclae.Context(N, D, M, K)
    codes, r = torch.full((N, M), 9, dtype=torch.uint8, device="cuda:0"), torch.empty_like(X)
    ctx.timing_enable(["assign"])
    ctx.encode(X, C, codes, r)
    assert ctx.timing_read()["assign"][1] == launches
    ctx.timing_enable([])
    want, rw = torch.full_like(codes, 9), X.clone()
    for m in range(M):
        ctx.assign(m, rw, C, want)
        ctx.cool(m, C, want, rw)
    assert torch.equal(codes, want)
    assert torch.equal(r, rw)
    ctx.close()
