"""Stages that keep distance bounds assign from a copy of x' in fp16 operands, left by the pass that writes x', and from a dictionary
image that the centroid update keeps up: a training ends in the same bits as one without bounds, which reads x' itself and rounds it
anew in every assignment.  Row lengths at the edges of the 16-dim steps, of the units of 64 and 128 dims, of the kernels for long rows
(768) and of dictionaries that LDS holds; one tile of 32 vectors to a wave and several; both ways into a stage (its own heat pass, the boundary pass of the one before)."""
import numpy as np
import pytest

from parity_util import to_dev

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def _train(X, C0, idx, sweeps, pruned, iters=4):
    from paper_1509_05194_amd import hclae
    M, K, D = C0.shape
    ctx = hclae.Context(X.shape[0], D, M, K)
    ctx.set_pruning(pruned)
    C, codes, r = to_dev(C0), torch.zeros((X.shape[0], M), dtype=torch.uint8, device="cuda:0"), to_dev(X - C0[:, 0].sum(0))
    err = ctx.anneal(C, codes, r, iters, sweeps, init_idx=idx)
    torch.cuda.synchronize()
    ctx.close()
    return C.cpu().numpy(), codes.cpu().numpy(), r.cpu().numpy(), err


def _same(X, C0, idx=None, sweeps=3):
    a, b = _train(X, C0, idx, sweeps, True), _train(X, C0, idx, sweeps, False)
    for x, y, name in zip(a, b, ("C", "codes", "residue", "err")):
        assert np.array_equal(x, y), name


@pytest.mark.parametrize("N,D,K", [(200000 + 1, 4, 256), (150000 + 3, 16, 64), (150000, 20, 33), (140000 + 31, 60, 64), (140000 + 3, 64, 256), (140000 + 7, 72, 65),
                                   (3001, 128, 100), (140000 + 1, 128, 256), (140000 + 1, 132, 256), (2000, 132, 256),
                                   (70000 + 33, 256, 256), (140000 + 5, 260, 256), (70000, 764, 32), (70000 + 3, 768, 200),
                                   (500 + 9, 1028, 33), (70000, 2304, 30)])
@pytest.mark.parametrize("seeded", [True, False])
def test_training_by_row_length(N, D, K, seeded):
    N = max(N, 2 ** 23 // (K * D) + 1)                     # else the stage keeps no bounds
    g = np.random.default_rng(D + K)
    means = g.standard_normal((max(8, K // 2), D), np.float32)
    X = means[g.integers(0, len(means), N)] + np.float32(0.3) * g.standard_normal((N, D), np.float32) + np.float32(2)
    M = 3
    C0 = np.zeros((M, K, D), np.float32)
    idx = np.stack([g.choice(N, K, replace=False) for _ in range(M)]).astype(np.int64) if seeded else None
    if not seeded:
        C0[:] = 0.5 * X[g.choice(N, (M, K))]
    _same(X, C0, idx)


@pytest.mark.parametrize("kind", ["zero", "tiny", "outlier", "outliers", "offset", "large", "small"])
def test_dictionaries_that_leave_their_scale(kind):
    """The centre and scale of the rows come from the dictionary as the stage finds it."""
    N, D, M, K = 6000, 64, 2, 64
    g = np.random.default_rng(7)
    X = (g.standard_normal((40, D))[g.integers(0, 40, N)] + 0.3 * g.standard_normal((N, D))).astype(np.float32)
    C0 = X[g.choice(N, (M, K))] * np.float32(0.5)
    if kind == "zero":                                     # nothing to take a scale from but the rows
        C0[:] = 0
    elif kind == "tiny":
        C0 *= np.float32(1e-5)
    elif kind == "outlier":                                # a centroid far beyond the codewords and the sampled rows
        X[1] *= np.float32(1e3)
    elif kind == "outliers":
        X[1::97] *= np.float32(300)
    elif kind == "offset":
        X += np.float32(700)
        C0 += np.float32(700)
    elif kind == "large":
        X *= np.float32(1e14)
        C0 *= np.float32(1e14)
    elif kind == "small":
        X *= np.float32(1e-14)
        C0 *= np.float32(1e-14)
    _same(X, C0, sweeps=2)


def test_first_call_under_capture():
    """While the stream is captured the arrays of the fp16 rows cannot be had: the call reads x' itself, with the same bits, and so do
    the replays after eager calls that have them."""
    from paper_1509_05194_amd import hclae
    N, D, M, K, T = 20000 + 7, 64, 2, 64, 4
    g = np.random.default_rng(3)
    X = (g.standard_normal((40, D))[g.integers(0, 40, N)] + 0.3 * g.standard_normal((N, D))).astype(np.float32)
    C0 = X[g.choice(N, (M, K))] * np.float32(0.5)
    s = torch.cuda.Stream()
    with torch.cuda.stream(s):
        start = [to_dev(C0), torch.zeros((N, M), dtype=torch.uint8, device="cuda:0"), to_dev(X - C0[:, 0].sum(0))]
        eager = [t.clone() for t in start]
        ctx = hclae.Context(N, D, M, K)
        ctx.sweep(*eager, T, want_err=False)
        torch.cuda.synchronize()
        other = hclae.Context(N, D, M, K)                 # no call of its own before the captured one
        run = [t.clone() for t in start]
        torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=s):
            other.sweep(*run, T, want_err=False)
        for i in range(3):
            for a, b in zip(run, start):
                a.copy_(b)
            graph.replay()
            torch.cuda.synchronize()
            for a, b in zip(run, eager):
                assert torch.equal(a, b), "replay %d" % i
            again = [t.clone() for t in start]
            (ctx if i == 0 else other).sweep(*again, T, want_err=False)      # eager work between: other gets its arrays
            torch.cuda.synchronize()
            for a, b in zip(again, eager):
                assert torch.equal(a, b)
        ctx.close()
        other.close()


def test_without_memory_for_the_rows():
    """A context made for more vectors than the device has room for in fp16: its trainings read x' itself, with the same bits, call after
    call, and the second call leaves the free memory as it was."""
    N, D, M, K = 4000, 2304, 2, 32
    assert N * K * D > 2 ** 23                             # else the stage keeps no bounds
    from paper_1509_05194_amd import hclae
    n_max = torch.cuda.get_device_properties(0).total_memory // (2 * D) + 1
    g = np.random.default_rng(5)
    X = (g.standard_normal((20, D))[g.integers(0, 20, N)] + 0.3 * g.standard_normal((N, D))).astype(np.float32)
    idx = np.stack([g.choice(N, K, replace=False) for _ in range(M)]).astype(np.int64)
    out = []
    for size in (N, n_max):
        ctx = hclae.Context(size, D, M, K)
        free = []
        for _ in range(2):
            C, codes, r = torch.zeros((M, K, D), device="cuda"), torch.zeros((N, M), dtype=torch.uint8, device="cuda"), to_dev(X)
            ctx.anneal(C, codes, r, 4, 2, init_idx=idx)
            out.append([t.cpu().numpy() for t in (C, codes, r)])
            free.append(torch.cuda.mem_get_info()[0])
        assert abs(free[0] - free[1]) < 2 ** 26
        ctx.close()
    for other in out[1:]:
        for a, b in zip(out[0], other):
            assert np.array_equal(a, b)
