"""Every code of a training against direct-form distances in 64 bits, on shapes of all contraction kernels: dictionaries that fit
the LDS of a compute unit and dictionaries that pass through it in slices (D = 516 and longer), 1, 2, 4 and 8 blocks of codewords,
ragged last slices.  hclae_set_contraction is kept for callers: both of its modes are accepted and change nothing."""
import numpy as np
import pytest

from paper_1509_05194_amd import synth
from parity_util import judge_codes, to_dev

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def _assert_nearest(x, c, codes):
    """Codes are argmin_k ||x - c_k||^2 of the fp32 rows, in 64 bits; the lowest index where that ties exactly.  Distances that
    agree to 1e-14 relative, closer than the order of the additions, may go either way."""
    c = c.double()
    step = max(1, (1 << 26) // (c.shape[0] * c.shape[1]))
    wrong = 0
    for n in range(0, len(x), step):
        d = ((x[n:n + step].double()[:, None, :] - c) ** 2).sum(2)
        got = d.gather(1, codes[n:n + step].long()[:, None])[:, 0]
        best, at = d.min(1)
        tie = (d == best[:, None]).sum(1) > 1
        first = (d == best[:, None]).to(torch.uint8).argmax(1)
        wrong += int(((got > best * (1 + 1e-14)) | (tie & (got == best) & (first != codes[n:n + step]))).sum())
    assert wrong == 0, "%d of %d codes are not the nearest codeword" % (wrong, len(x))


@pytest.mark.parametrize("gen,N,D,M,K", [("tiny", 10000 + 3, 16, 4, 16), ("sift", 30000 + 7, 128, 3, 256),
                                         ("sift", 5000 + 1, 20, 2, 100), ("gist", 3000 + 5, 64, 2, 256),
                                         # D-chunked shapes: 8, 4, 2 and 1 codeword blocks, a ragged last slice
                                         ("gist", 6000 + 5, 960, 2, 256), ("gist", 3000 + 1, 516, 2, 100),
                                         ("gist", 2000 + 3, 1412, 2, 40), ("gist", 1500 + 7, 2052, 2, 16)])
def test_every_code_of_a_training_is_the_nearest(gen, N, D, M, K):
    """Two sweeps, step by step with every assignment checked, and the same two as stages (which skip what their bounds settle),
    in either mode of hclae_set_contraction: the same bits."""
    from paper_1509_05194_amd import hclae
    X = to_dev({"tiny": lambda: synth.tiny_gmm(N=N, D=D), "sift": lambda: synth.sift_like(N, D=D),
                "gist": lambda: synth.gist_like(N, D=D)}[gen]())
    T, idx = 3, synth.init_indices(N, M, K)
    ctx = hclae.Context(N, D, M, K)
    C = torch.zeros((M, K, D), dtype=torch.float32, device="cuda:0")
    codes = torch.zeros((N, M), dtype=torch.uint8, device="cuda:0")
    r = X.clone()
    for sweep in range(2):
        for m in range(M):
            ctx.heat(m, C, codes, r)
            if sweep == 0:
                C[m] = r[torch.from_numpy(idx[m]).cuda()]
            for t in range(T + 1):
                ctx.assign(m, r, C, codes)
                _assert_nearest(r, C[m], codes[:, m])
                if t < T:
                    ctx.update(m, r, C, codes)
            ctx.cool(m, C, codes, r)
    q, qr, row = torch.empty_like(codes), torch.empty_like(X), X.clone()
    ctx.encode(X, C, q, qr)
    for m in range(M):
        _assert_nearest(row, C[m], q[:, m])
        row -= C[m][q[:, m].long()]
    assert torch.equal(row, qr)
    for mode in (0, 1):
        ctx.set_contraction(mode)
        Cs, cs, rs = torch.zeros_like(C), torch.zeros_like(codes), X.clone()
        for sweep in range(2):
            for m in range(M):
                ctx.anneal_stage(m, Cs, cs, rs, T, init_idx=idx[m] if sweep == 0 else None)
        assert torch.equal(Cs, C) and torch.equal(cs, codes) and torch.equal(rs, r)
    ctx.close()


def test_fullsize_codes(oracle):
    """N = 1,000,000, D = 128, K = 256: sampled codes against the oracle one by one, every fourth code in 64 bits; integer data
    against rows of it, then real-valued residues against real-valued codewords."""
    from paper_1509_05194_amd import hclae
    N, D, K, M = 1_000_000, 128, 256, 2
    X = synth.sift_like(N, D=D)
    Xg = to_dev(X)
    idx = synth.init_indices(N, M, K)
    C = torch.zeros((M, K, D), dtype=torch.float32, device="cuda:0")
    C[0] = Xg[torch.from_numpy(idx[0]).cuda()]
    ctx = hclae.Context(N, D, M, K)
    codes = torch.zeros((N, M), dtype=torch.uint8, device="cuda:0")
    rng = np.random.default_rng(2)
    sample = np.sort(rng.choice(N, 4096, replace=False))
    sample[-1] = N - 1
    codes_s = np.zeros((len(sample), M), np.uint8)

    def check(m, x, rows64):
        ctx.assign(m, x, C, codes)
        print("full-size assign %d: %d of %d undecided by the scores" % (m, ctx.last_refined(), N))
        _assert_nearest(x[::4], C[m], codes[::4, m])
        C64 = C.cpu().numpy().astype(np.float64)
        d1, d2, _ = oracle.assign(rows64, C64, codes_s, m, top2=True)
        ndiff, nex, bad = judge_codes(oracle, rows64, C64, m, codes.cpu().numpy()[sample, m], codes_s[:, m], d1, d2)
        assert not bad

    check(0, Xg, X[sample].astype(np.float64))
    # residues: one centroid update, then x minus its codeword against rows of that
    ctx.update(0, Xg, C, codes)
    r = Xg.clone()
    ctx.cool(0, C, codes, r)
    C[1] = r[torch.from_numpy(idx[1]).cuda()]
    check(1, r, r.cpu().numpy()[sample].astype(np.float64))
    ctx.close()
