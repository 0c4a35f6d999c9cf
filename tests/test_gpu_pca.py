"""Improved k-means for high-dimensional residue (Sec. 3.2 of arXiv 1509.05194) on the GPU against
the oracle: second moments, rotation, prefix assignment, and the whole cool-down in lockstep."""
import numpy as np
import pytest

from paper_1509_05194_amd import synth
from parity_util import fresh_state, judge_codes, narrow_state, rel_fro, to_dev

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

SHAPES = {
    "tiny": dict(gen="tiny", N=5000 + 3, D=16, M=2, K=16),
    "sift": dict(gen="sift", N=12000 + 5, D=128, M=2, K=256),
    "d132": dict(gen="sift", N=2000 + 1, D=132, M=1, K=40),
    "gist": dict(gen="gist", N=2500 + 7, D=960, M=1, K=256),
}


def _data(c):
    if c["gen"] == "tiny":
        return synth.tiny_gmm(N=c["N"], D=c["D"])
    if c["gen"] == "sift":
        return synth.sift_like(c["N"], D=c["D"])
    return synth.gist_like(c["N"], D=c["D"])


def _ctx(c):
    from paper_1509_05194_amd import hclae
    return hclae.Context(c["N"], c["D"], c["M"], c["K"])


@pytest.mark.parametrize("case", list(SHAPES))
def test_covariance(case):
    c = SHAPES[case]
    X = _data(c)
    ctx = _ctx(c)
    mean, cov = ctx.covariance(to_dev(X))
    X64 = X.astype(np.float64)
    ref_mean = X64.mean(0)
    ref = np.cov(X64, rowvar=False, bias=True)
    assert np.abs(mean.cpu().numpy() - ref_mean).max() <= 1e-12 * max(np.abs(ref_mean).max(), 1.0)
    err = np.abs(cov.cpu().numpy() - ref).max() / np.abs(ref).max()
    print("%s covariance: max error %.2e of the largest entry" % (case, err))
    assert err <= 1e-5
    ctx.close()


@pytest.mark.parametrize("case", list(SHAPES))
def test_rotate(case, oracle):
    c = SHAPES[case]
    X = _data(c)
    D = c["D"]
    R = np.linalg.qr(np.random.default_rng(D).standard_normal((D, D)))[0]
    R32 = np.ascontiguousarray(R, np.float32)
    ctx = _ctx(c)
    xg, Rg = to_dev(X), to_dev(R32)
    out = torch.empty_like(xg)
    for tr in (False, True):
        out.fill_(float("nan"))
        ctx.rotate(xg, Rg, out, transpose=tr)
        ref = oracle.rotate(X.astype(np.float64), R32.astype(np.float64), transpose=tr)
        err = np.abs(out.cpu().numpy() - ref).max() / np.abs(ref).max()
        print("%s rotate(transpose=%s): max error %.2e of the largest entry" % (case, tr, err))
        assert err <= 1e-5          # fp32 contraction over D terms
    ctx.close()


@pytest.mark.parametrize("case", list(SHAPES))
def test_assign_prefix(case, oracle):
    """Distance over the first dact coordinates = full distance with the other coordinates zeroed on
    both sides, which is how the oracle's (pinned) assign is used here."""
    c = SHAPES[case]
    X = _data(c)
    N, D, M, K = c["N"], c["D"], c["M"], c["K"]
    g = np.random.default_rng(1)
    C32 = np.ascontiguousarray(X[g.choice(N, M * K, replace=False)].reshape(M, K, D))
    ctx = _ctx(c)
    xg, Cg = to_dev(X), to_dev(C32)
    # 131, 222, 243: prefixes that are no multiple of 4 and too long for an LDS-resident dictionary at K = 256
    # (the D-chunked kernels: the last 4-float piece of a row prefix straddles its end)
    for dact in sorted(set([1, 2, 3, 5, min(D, 63), min(D, 66), min(D, 131), min(D, 222), min(D, 243), D])):
        codes_g = torch.full((N, M), 255, dtype=torch.uint8, device="cuda:0")
        ctx.assign_prefix(M - 1, xg, Cg, codes_g, dact)
        xm = X.astype(np.float64)
        Cm = C32.astype(np.float64)
        xm[:, dact:] = 0.0
        Cm[:, :, dact:] = 0.0
        codes_o = np.zeros((N, M), np.uint8)
        d1, d2, _ = oracle.assign(xm, Cm, codes_o, M - 1, top2=True)
        nd, nex, bad = judge_codes(oracle, xm, Cm, M - 1, codes_g.cpu().numpy()[:, M - 1], codes_o[:, M - 1], d1, d2)
        assert not bad, "dact=%d: %s" % (dact, bad[:5])
    ctx.close()


def _lockstep_pca_stage(ctx, oracle, m, T, dims, Rg, R64, Cg, codes_g, rg, xr_g, C64, codes64, r64, idx):
    """Drives the stage through the single-step entry points on the GPU and through the pinned
    primitives on the oracle, adopting exempt near-ties after every assignment."""
    adopted = 0
    N, D = r64.shape
    ctx.heat(m, Cg, codes_g, rg)
    oracle.heat(r64, codes64, C64, m)
    if idx is not None:
        Cg[m] = rg[torch.from_numpy(idx).to(rg.device)]
        C64[m] = r64[idx]
    ctx.rotate(rg, Rg, xr_g, transpose=False)
    crot = torch.empty_like(Cg[m])
    ctx.rotate(Cg[m].contiguous(), Rg, crot, transpose=False)
    Cg[m] = crot
    xr64 = oracle.rotate(r64, R64)
    Cp = C64.copy()
    Cp[m] = oracle.rotate(C64[m], R64)
    assert rel_fro(xr_g.cpu().numpy(), xr64) <= 1e-5 and rel_fro(Cg[m].cpu().numpy(), Cp[m]) <= 1e-5
    # step-locked from here: the k-means on prefixes starts from the GPU's rotated data and dictionary
    # (the rotation is an fp32 contraction, good to 1e-5; checked just above and in test_rotate)
    xr64 = xr_g.cpu().numpy().astype(np.float64)
    Cp[m] = Cg[m].cpu().numpy().astype(np.float64)
    for d in dims:
        for t in range(T):
            ctx.assign_prefix(m, xr_g, Cg, codes_g, int(d))
            xm, Cm = xr64.copy(), Cp.copy()
            xm[:, d:] = 0.0
            Cm[m][:, d:] = 0.0
            d1, d2, _ = oracle.assign(xm, Cm, codes64, m, top2=True)
            got = codes_g.cpu().numpy()[:, m]
            nd, nex, bad = judge_codes(oracle, xm, Cm, m, got, codes64[:, m], d1, d2)
            assert not bad, "prefix %d iteration %d: %s" % (d, t, bad[:5])
            adopted += nex
            codes64[:, m] = got
            ctx.update(m, xr_g, Cg, codes_g)
            oracle.update(xr64, codes64, Cp, m)
            assert rel_fro(Cg[m].cpu().numpy(), Cp[m]) <= 2e-5
    back = torch.empty_like(Cg[m])
    ctx.rotate(Cg[m].contiguous(), Rg, back, transpose=True)
    Cg[m] = back
    C64[m] = oracle.rotate(Cp[m], R64, transpose=True)
    assert rel_fro(Cg[m].cpu().numpy(), C64[m]) <= 2e-5
    C64[m] = Cg[m].cpu().numpy().astype(np.float64)                   # step-locked re-encode
    ctx.assign(m, rg, Cg, codes_g)
    d1, d2, _ = oracle.assign(r64, C64, codes64, m, top2=True)
    got = codes_g.cpu().numpy()[:, m]
    nd, nex, bad = judge_codes(oracle, r64, C64, m, got, codes64[:, m], d1, d2)
    assert not bad, "re-encode: %s" % bad[:5]
    adopted += nex
    codes64[:, m] = got
    ctx.cool(m, Cg, codes_g, rg)
    oracle.cool(r64, codes64, C64, m)
    return adopted


@pytest.mark.parametrize("case", ["tiny", "sift", "gist"])
def test_pca_stage_lockstep_and_entry_point(case, oracle):
    from paper_1509_05194_amd import hclae
    c = SHAPES[case]
    N, D, M, K = c["N"], c["D"], c["M"], c["K"]
    T = 2 if case != "gist" else 1
    X = _data(c)
    idx = synth.init_indices(N, M, K)
    dims = oracle.dimension_schedule(D, 10)
    if case == "gist":
        dims = dims[[1, 4, 7, 9]]                                     # keep the oracle's share of the test short
    ctx = _ctx(c)
    C64, codes64, r64 = fresh_state(X, M, K)
    Cg = torch.zeros((M, K, D), dtype=torch.float32, device="cuda:0")
    codes_g = torch.zeros((N, M), dtype=torch.uint8, device="cuda:0")
    rg = to_dev(X)
    xr_g = torch.empty_like(rg)
    # a second GPU state driven through the one-call entry point
    C2, codes2, r2, xr2 = Cg.clone(), codes_g.clone(), rg.clone(), torch.empty_like(rg)
    adopted = 0
    for m in range(M):
        # principal axes of the GPU's own x' (heat of a fresh stage is the identity: x' = residue)
        mean, cov = ctx.covariance(rg)
        w, V = np.linalg.eigh(cov.cpu().numpy())
        R64 = np.ascontiguousarray(V[:, np.argsort(-w, kind="stable")].T)
        R32 = R64.astype(np.float32)
        R64 = R32.astype(np.float64)                                  # both sides use the same fp32 matrix
        Rg = to_dev(R32)
        adopted += _lockstep_pca_stage(ctx, oracle, m, T, dims, Rg, R64, Cg, codes_g, rg, xr_g,
                                       C64, codes64, r64, idx[m])
        Eg, Eo = ctx.quant_error(rg), oracle.quant_error(r64)
        assert abs(Eg - Eo) <= 1e-4 * Eo
        assert rel_fro(rg.cpu().numpy(), r64) <= 1e-4
        st = ctx.anneal_stage_pca(m, C2, codes2, r2, Rg, dims, T, xr2, init_idx=idx[m])
        assert torch.equal(C2, Cg) and torch.equal(codes2, codes_g) and torch.equal(r2, rg)
        assert st["iters_run"] == T * len(dims) and abs(st["err_after"] - Eg) <= 1e-12 * Eg
    print("%s improved k-means: adopted %d near-ties; E after the stages %.6g" % (case, adopted, Eg))
    assert rel_fro(Cg.cpu().numpy(), C64) <= 1e-4
    ctx.close()


@pytest.mark.parametrize("case", ["tiny", "sift"])
def test_pca_stage_free_running_against_oracle_stage(case, oracle):
    """Free-running: hclae_anneal_stage_pca (principal axes found inside the library) against the oracle's own
    anneal_stage_pca with the oracle's axes, from the same start, nothing exchanged in between.  The cases have
    no near-tie that the two sides decide differently: codes must be EQUAL, the rest within 1e-4.  (SIFT-shaped
    data: the first stage only.  Seeds of a later stage can be rows whose residue is exactly zero -- sole members of
    their clusters -- which tie exactly in the oracle and not on the GPU's fp32 state; the lockstep test covers those.)"""
    c = SHAPES[case]
    N, D, M, K = c["N"], c["D"], c["M"], c["K"]
    stages = M if case == "tiny" else 1
    T = 2
    X = _data(c)
    idx = synth.init_indices(N, M, K)
    dims = oracle.dimension_schedule(D, 10)
    ctx = _ctx(c)
    C64, codes64, r64 = fresh_state(X, M, K)
    Cg = torch.zeros((M, K, D), dtype=torch.float32, device="cuda:0")
    codes_g = torch.zeros((N, M), dtype=torch.uint8, device="cuda:0")
    rg = to_dev(X)
    xr = torch.empty_like(rg)
    for m in range(stages):
        R64 = oracle.pca_axes(r64)                                    # heat of a fresh stage is the identity
        Eo = oracle.anneal_stage_pca(m, C64, codes64, r64, R64, dims, T, idx[m])
        st = ctx.anneal_stage_pca(m, Cg, codes_g, rg, None, dims, T, xr, init_idx=idx[m])
        ndiff = int((codes_g.cpu().numpy() != codes64).sum())
        print("%s free-running improved k-means, stage %d: %d codes differ, E gpu %.6g oracle %.6g, C err %.2e"
              % (case, m, ndiff, st["err_after"], Eo, rel_fro(Cg[m].cpu().numpy(), C64[m])))
        assert ndiff == 0
        assert abs(st["err_after"] - Eo) <= 1e-4 * Eo
        assert rel_fro(Cg[m].cpu().numpy(), C64[m]) <= 1e-4
        assert rel_fro(rg.cpu().numpy(), r64) <= 1e-4
    ctx.close()


def test_pca_axes_against_oracle_axes(oracle):
    """hclae_pca_axes (second moments on the device, eigen-solver inside the library) against oracle.pca_axes
    (NumPy covariance + LAPACK) on data with a clear spectrum: same axes in the same order with the same signs;
    on the SIFT-shaped data, whose small eigenvalues are close to one another: the same invariant subspaces
    (R diagonalises the oracle's covariance, eigenvalues descending and equal to LAPACK's)."""
    from paper_1509_05194_amd import hclae
    g = np.random.default_rng(11)
    N, D = 30000 + 7, 32
    Q = np.linalg.qr(g.standard_normal((D, D)))[0]
    X = ((g.standard_normal((N, D)) * 0.8 ** np.arange(D)) @ Q.T + 2.0).astype(np.float32)
    ctx = hclae.Context(N, D, 1, 16)
    R, w = ctx.pca_axes(to_dev(X))
    R = R.cpu().numpy().astype(np.float64)
    R_o = oracle.pca_axes(X.astype(np.float64))
    cov = np.cov(X.astype(np.float64), rowvar=False, bias=True)
    w_o = np.linalg.eigvalsh(cov)[::-1]
    print("clear spectrum: max axis error %.2e, max eigenvalue error %.2e of the largest"
          % (np.abs(R - R_o).max(), np.abs(w - w_o).max() / w_o[0]))
    assert np.abs(w - w_o).max() <= 1e-5 * w_o[0]          # the covariance comes from an fp32 matrix-core contraction
    # an axis moves by about (error of the covariance) / (gap to the next eigenvalue)
    gap = np.minimum(np.abs(np.diff(w_o, prepend=np.inf)), np.abs(np.diff(w_o, append=-np.inf)))
    assert np.all(np.abs(R - R_o).max(axis=1) <= 2e-5 * w_o[0] / gap + 1e-6)
    for i in range(D):
        assert R[i, np.argmax(np.abs(R_o[i]))] > 0         # the oracle's sign convention
    ctx.close()

    c = SHAPES["sift"]
    X = _data(c)
    ctx = _ctx(c)
    R, w = ctx.pca_axes(to_dev(X))
    R = R.cpu().numpy().astype(np.float64)
    cov = np.cov(X.astype(np.float64), rowvar=False, bias=True)
    w_o = np.linalg.eigvalsh(cov)[::-1]
    assert np.all(np.diff(w) <= 0) and np.abs(w - w_o).max() <= 1e-5 * w_o[0]
    assert np.abs(R @ R.T - np.eye(c["D"])).max() <= 1e-6
    T = R @ cov @ R.T
    assert np.abs(T - np.diag(np.diag(T))).max() <= 2e-5 * w_o[0]
    np.testing.assert_allclose(np.diag(T), w_o, atol=2e-5 * w_o[0])
    ctx.close()


@pytest.mark.parametrize("case", ["tiny", "d132", "gist"])
def test_pca_stage_with_its_own_axes_equals_the_stage_given_them(case):
    """hclae_anneal_stage_pca with R = NULL finds the principal axes of its own x' (hclae_pca_axes inside the call):
    the result must be the very bits of the stage that is handed the axes hclae_pca_axes returns for that x'."""
    c = SHAPES[case]
    N, D, M, K = c["N"], c["D"], c["M"], c["K"]
    X = _data(c)
    idx = synth.init_indices(N, M, K)
    dims = np.array([2, D // 3, D], np.int32)
    ctx = _ctx(c)
    out = []
    for own in (True, False):
        C = torch.zeros((M, K, D), dtype=torch.float32, device="cuda:0")
        codes = torch.zeros((N, M), dtype=torch.uint8, device="cuda:0")
        r = to_dev(X)
        xr = torch.empty_like(r)
        for m in range(M):
            if own:
                ctx.anneal_stage_pca(m, C, codes, r, None, dims, 1, xr, init_idx=idx[m])
            else:
                R, w = ctx.pca_axes(r)                                # a fresh stage: x' is the residue
                assert np.all(np.diff(w) <= 0) and w[-1] >= -1e-9 * w[0]
                ctx.anneal_stage_pca(m, C, codes, r, R, dims, 1, xr, init_idx=idx[m])
        out.append((C, codes, r))
    assert torch.equal(out[0][0], out[1][0]) and torch.equal(out[0][1], out[1][1]) and torch.equal(out[0][2], out[1][2])
    ctx.close()


@pytest.mark.parametrize("case", ["tiny", "d132"])
def test_sweep_cooled_by_the_improved_kmeans(case, oracle):
    """hclae_set_cooldown(improved): hclae_sweep and hclae_anneal_stage then cool every dictionary with the improved
    k-means.  The sweep must give the bits of hclae_anneal_stage_pca called stage by stage with R = NULL, the library's
    schedule and ceil(iters / prefixes) iterations per prefix; E per stage is the error of the residue; x = sum of the
    selected codewords + residue; and (tiny case, free-running, no near-tie decided differently) codes, dictionaries
    and E are the oracle's own anneal_stage_pca with the oracle's axes."""
    from paper_1509_05194_amd import hclae
    c = SHAPES[case]
    N, D, M, K = c["N"], c["D"], c["M"], c["K"]
    X = _data(c)
    idx = synth.init_indices(N, M, K)
    iters = 15
    dims = hclae.dimension_schedule(D, 10)
    per = -(-iters // len(dims))
    ctx = _ctx(c)
    ctx.set_cooldown(True, 10)
    C = torch.zeros((M, K, D), dtype=torch.float32, device="cuda:0")
    codes = torch.zeros((N, M), dtype=torch.uint8, device="cuda:0")
    r = to_dev(X)
    E1 = ctx.sweep(C, codes, r, iters, init_idx=idx)
    E2 = ctx.sweep(C, codes, r, iters)
    assert abs(ctx.quant_error(r) - E2[-1]) <= 1e-12 * E2[-1]
    recon = r.clone()
    for m in range(M):
        recon += C[m][codes[:, m].long()]
    assert float((recon - to_dev(X)).abs().max()) <= 1e-5 * max(float(np.abs(X).max()), 1.0)
    # stage by stage through the explicit entry point (plain cool-down selected: that call does not depend on it)
    ctx.set_cooldown(False)
    C2 = torch.zeros_like(C)
    codes2 = torch.zeros_like(codes)
    r2 = to_dev(X)
    xr = torch.empty_like(r2)
    Es = []
    for s in range(2):
        for m in range(M):
            st = ctx.anneal_stage_pca(m, C2, codes2, r2, None, dims, per, xr, init_idx=idx[m] if s == 0 else None)
            assert st["iters_run"] == per * len(dims)
            Es.append(st["err_after"])
    assert torch.equal(C, C2) and torch.equal(codes, codes2) and torch.equal(r, r2)
    np.testing.assert_array_equal(np.concatenate([E1, E2]), Es)
    # hclae_anneal_stage obeys the setting too
    ctx.set_cooldown(True, 10)
    st = ctx.anneal_stage(0, C, codes, r, iters)
    st2 = ctx.anneal_stage_pca(0, C2, codes2, r2, None, dims, per, xr)
    assert torch.equal(C, C2) and torch.equal(codes, codes2) and st["err_after"] == st2["err_after"]
    assert st["iters_run"] == per * len(dims)
    if case == "tiny":
        C64, codes64, r64 = fresh_state(X, M, K)
        Cg = torch.zeros_like(C)
        cg = torch.zeros_like(codes)
        rg = to_dev(X)
        Eg = ctx.sweep(Cg, cg, rg, iters, init_idx=idx)
        for m in range(M):
            Eo = oracle.anneal_stage_pca(m, C64, codes64, r64, oracle.pca_axes(r64), oracle.dimension_schedule(D, 10), per, idx[m])
            assert abs(Eg[m] - Eo) <= 1e-4 * Eo
        assert int((cg.cpu().numpy() != codes64).sum()) == 0
        assert rel_fro(Cg.cpu().numpy(), C64) <= 1e-4 and rel_fro(rg.cpu().numpy(), r64) <= 1e-4
    ctx.close()
