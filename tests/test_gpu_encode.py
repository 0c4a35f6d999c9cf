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


# 256 CUs: 8192 vectors are a tile of 32 for each, 65536 a round of k_encode_wave.  Each line of the choice, at it and one vector on: F a tile for
# all waves of a block (one launch decides), W a tile per wave (two), S dictionary by dictionary (one each, and a row pass each)
@pytest.mark.parametrize("N,D,M,K,way", [
    (8192, 128, 1, 256, "F"), (8193, 64, 1, 129, "S"), (8193, 20, 1, 256, "S"), (32768, 16, 1, 128, "F"), (32769, 100, 1, 65, "S"),
    (65536, 32, 1, 33, "F"), (65537, 128, 1, 32, "S"), (32769, 16, 1, 16, "S"), (300000, 36, 1, 32, "F"), (300000, 20, 1, 64, "F"),
    (65536, 128, 2, 256, "W"), (65537, 96, 2, 129, "S"), (65537, 68, 2, 129, "W"), (131072, 64, 2, 256, "W"), (131073, 64, 2, 129, "S"),
    (131073, 32, 2, 64, "S"), (131073, 36, 2, 64, "W"), (131073, 16, 2, 32, "S"), (131073, 28, 2, 32, "F"),
    (24576, 128, 2, 256, "F"), (24577, 68, 2, 256, "W"), (20480, 128, 3, 256, "F"), (20481, 128, 4, 129, "W"), (16384, 64, 3, 256, "F"),
    (16385, 4, 3, 256, "W"), (12288, 64, 4, 256, "F"), (12289, 64, 4, 256, "W"),
    (49152, 96, 3, 65, "F"), (49153, 128, 3, 128, "W"), (36864, 128, 4, 128, "F"), (36865, 92, 3, 65, "W"), (73728, 128, 4, 128, "F"),
    (73729, 100, 4, 128, "W"), (32768, 64, 3, 128, "F"), (32769, 16, 4, 65, "W"),
    (36864, 32, 3, 64, "F"), (36865, 16, 4, 33, "W"), (40960, 48, 4, 64, "F"), (40961, 36, 3, 64, "W"), (53248, 64, 4, 64, "F"),
    (53249, 128, 4, 64, "W"), (300000, 64, 3, 64, "F"), (57344, 128, 3, 64, "F"), (57345, 128, 3, 33, "W"), (45056, 92, 4, 64, "F"),
    (45057, 68, 3, 64, "W"), (49152, 128, 4, 32, "F"), (49153, 68, 3, 32, "W"), (32768, 24, 4, 32, "F"), (32769, 4, 3, 16, "W"),
    (300000, 28, 4, 16, "F"),
    (98304, 132, 3, 33, "F"), (98305, 204, 3, 64, "S"), (393216, 208, 3, 33, "F"), (393217, 208, 3, 64, "S"),
    (131072, 132, 3, 65, "F"), (131073, 204, 3, 65, "S"), (131073, 208, 3, 65, "F"), (49152, 132, 3, 140, "F"), (49153, 256, 3, 140, "S"),
    (100, 260, 3, 20, "S"), (100, 132, 3, 32, "S")])
def test_encoder_by_size(N, D, M, K, way):
    """The encoders on either side of the lines between them."""
    from paper_1509_05194_amd import hclae
    g = torch.Generator(device="cuda").manual_seed(N + K)
    C = torch.randn((M, K, D), generator=g, device="cuda") * torch.tensor([1.0, 0.5, 0.3, 0.2][:M], device="cuda")[:, None, None]
    X = torch.randn((N, D), generator=g, device="cuda")
    ctx = hclae.Context(N, D, M, K)
    codes, r = torch.full((N, M), 9, dtype=torch.uint8, device="cuda:0"), torch.empty_like(X)
    ctx.timing_enable(["assign", "cool"])
    ctx.encode(X, C, codes, r)
    times = ctx.timing_read()
    assert (times["assign"][1], times["cool"][1]) == {"F": (1, 0), "W": (2, 0), "S": (M, M)}[way]
    ctx.timing_enable([])
    want, rw = torch.full_like(codes, 9), X.clone()
    for m in range(M):
        ctx.assign(m, rw, C, want)
        ctx.cool(m, C, want, rw)
    assert torch.equal(codes, want)
    assert torch.equal(r, rw)
    ctx.close()
