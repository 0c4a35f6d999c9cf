"""The fp16 pre-selection of the nearest-codeword kernels at the sizes and values where it can go wrong: every code against
the fp64 direct-form oracle.  The kernel's decisions are fp64 (or fp32 with a proven margin) direct-form decisions on the fp32
data, lowest index on exact ties, so the codes are equal one by one -- except where the oracle's own two best distances agree
to 1e-14 relative, closer than the order of fp64 additions."""
import numpy as np
import pytest

from parity_util import to_dev

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def _data(kind, N, D, K, rng):
    C = rng.standard_normal((K, D)).astype(np.float32)
    X = (C[rng.integers(0, K, N)] + 0.5 * rng.standard_normal((N, D))).astype(np.float32)
    if kind == "offset":                 # a common offset three orders above the spread
        C += np.float32(900.0)
        X += np.float32(900.0)
    elif kind == "small":
        C *= np.float32(1e-15)
        X *= np.float32(1e-15)
    elif kind == "large":
        C *= np.float32(3e14)
        X *= np.float32(3e14)
    elif kind == "twins":                # every codeword twice, and pairs an ulp apart
        C[K // 2:2 * (K // 2)] = C[:K // 2]
        if K >= 4:
            C[K - 1] = np.nextafter(C[0], np.float32(10))
    elif kind == "wild":                 # rows far outside the range the dictionary sets, and one huge codeword
        X[::7] *= np.float32(3e4)
        X[3::11] = 0.0
        C[K // 2] *= np.float32(2e3)
    elif kind == "zero":
        C[:] = 0.0
    # more candidates than fp16 scores can tell apart: they are scored again in fp32
    elif kind == "groups":               # two groups 30 standard deviations apart
        C[::2] += np.float32(30.0)
        X = (C[rng.integers(0, K, N)] + 0.5 * rng.standard_normal((N, D))).astype(np.float32)
    elif kind == "tiny":                 # codewords far below the vectors
        C *= np.float32(1e-4)
        X *= np.float32(rng.choice([0.1, 1.0, 30.0]))
    elif kind == "spread":               # norms over several orders
        C *= np.exp(2 * rng.standard_normal((K, 1))).astype(np.float32)
        X = (C[rng.integers(0, K, N)] * (1 + 0.3 * rng.standard_normal((N, D)))).astype(np.float32)
    elif kind == "huge":                 # squares beyond fp32
        C *= np.float32(1e20)
        X *= np.float32(1e20)
    return X, C


# K and D at the edges of the 32-codeword blocks and the 16- and 64-dim steps, up to the largest dictionary LDS holds and one
# beyond it; N at the edges of a 32-vector tile
SHAPES = [(1, 4, 1), (31, 8, 2), (33, 16, 31), (32, 20, 33), (257, 60, 64), (1000, 64, 65), (511, 68, 100), (1025, 96, 128),
          (4099, 128, 256), (700, 132, 200), (2049, 256, 256), (600, 260, 256), (300, 508, 128), (333, 2048, 32)]


@pytest.mark.parametrize("kind", ["plain", "offset", "small", "large", "twins", "wild", "zero", "groups", "tiny", "spread",
                                  "huge"])
@pytest.mark.parametrize("N,D,K", SHAPES)
def test_codes_equal_fp64_decisions(kind, N, D, K, oracle):
    from paper_1509_05194_amd import hclae
    rng = np.random.default_rng(1000 * D + K)
    X, C = _data(kind, N, D, K, rng)
    M = 2
    Call = np.zeros((M, K, D), np.float32)
    Call[1] = C
    ctx = hclae.Context(N, D, M, K)
    codes = torch.full((N, M), 7, dtype=torch.uint8, device="cuda:0")
    ctx.assign(1, to_dev(X), to_dev(Call), codes)
    got = codes.cpu().numpy()
    ctx.close()
    want = np.zeros((N, M), np.uint8)
    d1, d2, _ = oracle.assign(X.astype(np.float64), Call.astype(np.float64), want, 1, top2=True)
    assert np.all(got[:, 0] == 7)
    differ = got[:, 1] != want[:, 1]
    tied = d2 - d1 <= 1e-14 * d2
    assert not np.any(differ & ~tied), "%d codes differ" % int((differ & ~tied).sum())
    same = d2 == d1                      # exact ties, lowest index
    assert not np.any(differ & same)


@pytest.mark.parametrize("dact", [1, 2, 3, 15, 16, 17, 48, 49, 63, 64, 65, 127, 128])
def test_prefix_codes(dact, oracle):
    from paper_1509_05194_amd import hclae
    N, D, K = 1500 + 5, 128, 200
    rng = np.random.default_rng(dact)
    X, C = _data("offset", N, D, K, rng)
    X[:, dact:] += np.float32(1e6)       # must not count
    ctx = hclae.Context(N, D, 1, K)
    codes = torch.zeros((N, 1), dtype=torch.uint8, device="cuda:0")
    ctx.assign_prefix(0, to_dev(X), to_dev(C[None]), codes, dact)
    got = codes.cpu().numpy()[:, 0]
    ctx.close()
    want = np.zeros((N, 1), np.uint8)
    d1, d2, _ = oracle.assign(np.ascontiguousarray(X[:, :dact]).astype(np.float64),
                              np.ascontiguousarray(C[None, :, :dact]).astype(np.float64), want, 0, top2=True)
    assert not np.any((got != want[:, 0]) & (d2 - d1 > 1e-14 * d2))


@pytest.mark.parametrize("kind", ["plain", "offset", "twins", "wild", "groups", "tiny", "spread"])
# N K D on both sides of the line from which a stage keeps bounds (2^23)
@pytest.mark.parametrize("N,D,K", [(5000 + 7, 128, 256), (3000 + 1, 100, 90), (2500, 16, 33), (20000 + 1, 16, 33),
                                   (2000 + 3, 516, 70), (200 + 3, 516, 70)])
def test_bounds_never_keep_a_wrong_code(kind, N, D, K):
    """A stage that skips what its bounds settle ends with the bits of a stage that assigns every vector every time."""
    from paper_1509_05194_amd import hclae
    rng = np.random.default_rng(D + K)
    X, C = _data(kind, N, D, K, rng)
    out = []
    for pruned in (False, True):
        ctx = hclae.Context(N, D, 1, K)
        ctx.set_pruning(pruned)
        Cg, codes, r = to_dev(C[None]), torch.zeros((N, 1), dtype=torch.uint8, device="cuda:0"), to_dev(X - C[0])
        st = ctx.anneal_stage(0, Cg, codes, r, 6)
        out.append((Cg, codes, r, st["err_after"]))
        ctx.close()
    for a, b in zip(out[0][:3], out[1][:3]):
        assert torch.equal(a, b)
    assert out[0][3] == out[1][3]


def test_many_candidates_do_not_cost_one_by_one():
    """Where fp16 scores leave every codeword a candidate of every vector (codewords 10^-4 of the vectors), the assignment takes
    some seven times as long as one without undecided vectors: another pass in fp32.  Deciding among all 256 in the direct form
    took 80 times as long; 25 lies between the two with room for a slow clock."""
    from paper_1509_05194_amd import hclae
    N, D, K = 200000, 128, 256
    g = torch.Generator(device="cuda").manual_seed(2)
    X = torch.randn((N, D), generator=g, device="cuda")
    C = X[:K][None].clone()
    ctx = hclae.Context(N, D, 1, K)
    codes = torch.zeros((N, 1), dtype=torch.uint8, device="cuda:0")
    us = []
    for f in (1.0, 1e-4):
        Cf = C * f
        best = float("inf")
        for _ in range(5):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            ctx.assign(0, X, Cf, codes)
            b.record()
            torch.cuda.synchronize()
            best = min(best, a.elapsed_time(b) * 1e3)
        us.append(best)
    print("ordinary codewords %.0f us, codewords far below the vectors %.0f us" % tuple(us))
    assert us[1] < 25 * us[0]
    ctx.close()
