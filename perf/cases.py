"""The work a user of this library has it do, as measurable cases: one dict per case, with sizes from the repository's own
configurations (SIFT-shaped D = 128, GIST-shaped D = 960, the tiny mixture, 64- and 128-bit codes, byte chunks) and the ranges
around them.  A case names the call (`kind`), the data it runs on (`data`) and the sizes.

  encode    Context.encode: greedy codes of new vectors under learned dictionaries (queries, a base set)
  beam      Context.encode_beam: the multi-path encoder of Sec. 3.3
  train     Context.anneal from all-zero dictionaries with seed rows: the whole training in one call
  resume    Context.anneal from a saved learner (dictionaries, codes, residue), as a program that keeps a checkpoint does
  online    Context.online_chunk: one chunk of byte descriptors through the online learner
  improved  Context.anneal_stage cooled by the improved k-means of Sec. 3.2
  report    Context.quant_error, code_stats and reorder_by_variance: what is asked of a finished learner
"""
import math

import numpy as np
import torch

from paper_1509_05194_amd import hclae


def listed():
    return [
        # a handful of queries of a search front end: launches and latency are all there is
        {"name": "encode_queries", "kind": "encode", "data": "sift", "N": 64, "D": 128, "M": 8, "K": 256, "split": False},
        # the held-out queries of the benchmark
        {"name": "encode_heldout", "kind": "encode", "data": "sift", "N": 10000, "D": 128, "M": 8, "K": 256, "split": False},
        # a base set of a million 64-bit codes
        {"name": "encode_base", "kind": "encode", "data": "sift", "N": 1000000, "D": 128, "M": 8, "K": 256, "split": False},
        # long rows, an odd count: the dictionary does not fit the LDS of a compute unit
        {"name": "encode_gist", "kind": "encode", "data": "gist", "N": 100003, "D": 960, "M": 8, "K": 256, "split": False},
        # the better codes of the multi-path encoder, ten paths as in the paper
        {"name": "beam_sift", "kind": "beam", "data": "sift", "N": 200000, "D": 128, "M": 8, "K": 256, "L": 10, "split": False},
        # the tiny mixture: three sweeps of small launches
        {"name": "train_tiny", "kind": "train", "data": "gmm", "N": 10000, "D": 16, "M": 4, "K": 16, "iters": 10, "sweeps": 3,
         "split": False},
        # the headline configuration: the sweep from zero dictionaries and the annealing sweep after it
        {"name": "train_sift", "kind": "train", "data": "sift", "N": 1000000, "D": 128, "M": 8, "K": 256, "iters": 10, "sweeps": 2,
         "split": False},
        # long rows, trained
        {"name": "train_gist", "kind": "train", "data": "gist", "N": 200003, "D": 960, "M": 4, "K": 256, "iters": 10, "sweeps": 2,
         "split": False},
        # 128-bit codes, a learner taken up again for four more sweeps, with the split contraction switched on
        {"name": "resume_codes128", "kind": "resume", "data": "sift", "N": 250000, "D": 128, "M": 16, "K": 256, "iters": 10,
         "sweeps": 4, "split": True},
        # one chunk of a stream of byte descriptors
        {"name": "online_chunk", "kind": "online", "data": "sift", "N": 1000000, "D": 128, "M": 8, "K": 256, "split": False},
        # one stage cooled by the improved k-means: second moments, principal axes, rotation, growing prefixes
        {"name": "improved_stage", "kind": "improved", "data": "sift", "N": 300000, "D": 128, "M": 8, "K": 256, "iters": 10,
         "split": False},
        # error, code statistics and dictionary order of a finished learner
        {"name": "report", "kind": "report", "data": "sift", "N": 1000000, "D": 128, "M": 8, "K": 256, "split": False},
    ]


def _between(rng, lo, hi):
    """A whole number from lo to hi, spread over its logarithm."""
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi + 1)))))))


# most vector coordinates of a drawn case of each kind: no drawn case costs more than the largest listed one
_MOST = {"encode": 128e6, "beam": 25e6, "train": 64e6, "resume": 40e6, "online": 128e6, "improved": 40e6, "report": 128e6}


def draw(rng):
    kind = rng.choice(["encode", "encode", "encode", "train", "train", "train", "beam", "resume", "online", "improved", "report"])
    data = rng.choice(["sift", "sift", "gist", "gmm"])
    if kind == "online":
        data = "sift"
    if data == "sift":
        D = rng.choice([128, 128, 4 * _between(rng, 8, 48)])
    elif data == "gist":
        D = rng.choice([960, 4 * _between(rng, 49, 256)]) if kind != "improved" else 4 * _between(rng, 16, 64)
    else:
        D = 4 * _between(rng, 4, 32)
    K = rng.choice([256, 256, 256, _between(rng, 16, 255)])
    M = rng.choice([8, 8, 16, _between(rng, 2, 16)])
    if kind in ("train", "resume", "beam"):
        M = min(M, 8)
    n_most = int(_MOST[kind] * 8 / max(M, 8) / D)
    n_least = 1 if kind == "encode" else 100 if kind in ("beam", "report") else 3000
    case = {"kind": kind, "data": data, "N": _between(rng, n_least, max(n_least, n_most)), "D": D, "M": M, "K": K,
            "split": kind != "report" and rng.random() < 0.15}
    if kind == "beam":
        case["L"] = rng.choice([10, 10, _between(rng, 2, 16)])
    if kind in ("train", "resume", "improved"):
        case["iters"] = rng.choice([10, _between(rng, 3, 12)])
    if kind in ("train", "resume"):
        case["sweeps"] = rng.choice([1, 2, 3])
    return case


# ---- inputs ---------------------------------------------------------------------------------------------------------------

def _rows(data, N, D, seed):
    """N vectors shaped like the workloads of the repository's synthetic inputs, made on the device from the seed alone."""
    g = torch.Generator(device="cuda").manual_seed(int(seed))
    dev = torch.device("cuda:0")
    if data == "gmm":                    # isotropic mixture: means U[-1, 1], sigma 0.1
        mean = torch.rand((32, D), generator=g, device=dev) * 2 - 1
        comp = torch.randint(0, 32, (N,), generator=g, device=dev)
        return (mean[comp] + 0.1 * torch.randn((N, D), generator=g, device=dev)).contiguous()
    if data == "sift":                   # integers in [0, 255], about 30 % zeros, 256 components
        mean = 38.0 * torch.empty((256, D), device=dev).exponential_(1.0, generator=g) - 12.7
        sigma = 6.0 + 8.0 * torch.rand((256,), generator=g, device=dev)
        comp = torch.randint(0, 256, (N,), generator=g, device=dev)
        x = torch.randn((N, D), generator=g, device=dev)
        x.mul_(sigma[comp][:, None]).add_(mean[comp])
        return x.clamp_(0.0, 255.0).round_().contiguous()
    base = torch.randn((64, D), generator=g, device=dev) / 8.0      # gist: values in [0, 1], rank 64 and noise, 512 components
    lat = torch.randn((512, 64), generator=g, device=dev)
    comp = torch.randint(0, 512, (N,), generator=g, device=dev)
    z = lat[comp] + 0.5 * torch.randn((N, 64), generator=g, device=dev)
    x = 0.03 + 0.03 * (z @ base)
    return x.add_(0.02 * torch.randn((N, D), generator=g, device=dev)).clamp_(0.0, 1.0).contiguous()


def _dictionaries(X, M, K, seed):
    """M dictionaries fitted to a sample of X, each to what the ones before it leave: two rounds of k-means from rows that are
    not nearly zero (a row that was alone in its cluster is, and dictionaries of such rows would be full of equal codewords)."""
    g = torch.Generator().manual_seed(int(seed) + 17)
    r = X[torch.randint(0, X.shape[0], (max(4096, 48 * K),), generator=g).to(X.device)]
    C = torch.zeros((M, K, X.shape[1]))

    def nearest(c):
        c = c.to(X.device)
        return torch.addmm(-0.5 * (c * c).sum(1), r, c.T).argmax(1)

    for m in range(M):
        host, norm = r.cpu(), r.norm(dim=1).cpu()
        live = torch.nonzero(norm > 0.5 * norm.median()).flatten()
        c = host[live[torch.randperm(len(live), generator=g)[:K]]].clone()
        for _ in range(2):
            a = nearest(c).cpu()
            n = torch.bincount(a, minlength=K)
            s = torch.zeros_like(c).index_add_(0, a, host)       # on the host: the same sums every time
            c = torch.where(n[:, None] > 0, s / n.clamp(min=1)[:, None], c)
        C[m] = c
        r = r - c.to(X.device)[nearest(c)]
    return C.to(X.device).contiguous()


def _greedy(X, C):
    """Codes and residue of a learner on X, by torch: where a saved learner stands."""
    r = X.clone()
    codes = torch.empty((X.shape[0], C.shape[0]), dtype=torch.uint8, device=X.device)
    for m in range(C.shape[0]):
        a = torch.addmm(-0.5 * (C[m] * C[m]).sum(1), r, C[m].T).argmax(1)
        codes[:, m] = a.to(torch.uint8)
        r -= C[m][a]
    return codes, r


def _seed_rows(N, M, K, seed):
    rng = np.random.default_rng(int(seed) + 5194)
    return np.stack([rng.choice(N, size=K, replace=False) for _ in range(M)]).astype(np.int64)


def prepare(case, seed):
    N, D, M, K = case["N"], case["D"], case["M"], case["K"]
    kind = case["kind"]
    X = _rows(case["data"], N, D, seed)
    s = {"case": case, "X": X}
    if kind == "online":
        s["X"] = X.to(torch.uint8)
    if kind in ("encode", "beam", "online"):
        fit = X if N >= 20000 else _rows(case["data"], 20000, D, seed)   # queries come from the data the learner saw
        s["C"] = _dictionaries(fit, M, K, seed)
        s["codes"] = torch.zeros((N, M), dtype=torch.uint8, device=X.device)
        s["r"] = torch.empty_like(X)
    elif kind in ("train", "improved"):
        s["idx"] = _seed_rows(N, M, K, seed)
        s["C"] = torch.zeros((M, K, D), device=X.device)
        s["codes"] = torch.zeros((N, M), dtype=torch.uint8, device=X.device)
        s["r"] = torch.empty_like(X)
    else:                                                               # resume, report: a learner as it was saved
        C = _dictionaries(X, M, K, seed)
        s["saved"] = (C,) + _greedy(X, C)
        s["C"], s["codes"], s["r"] = (t.clone() for t in s["saved"])
    s["ctx"] = hclae.Context(N, D, M, K)
    if case["split"]:
        s["ctx"].set_contraction(1)
    if kind == "online":
        s["ctx"].online_begin(s["C"], np.full((M, K), 16, np.int64))
    if kind == "improved":
        s["ctx"].set_cooldown(True)
    return s


# ---- the calls ------------------------------------------------------------------------------------------------------------

def run(s):
    case, ctx, C, codes, r = s["case"], s["ctx"], s["C"], s["codes"], s["r"]
    kind = case["kind"]
    if kind == "encode":
        ctx.encode(s["X"], C, codes, r)
        return {"codes": codes, "residue": r}
    if kind == "beam":
        ctx.encode_beam(s["X"], C, case["L"], codes, r)
        return {"codes": codes, "residue": r}
    if kind == "train":                  # from scratch: all-zero dictionaries, the residue is the data
        C.zero_()
        codes.zero_()
        r.copy_(s["X"])
        err = ctx.anneal(C, codes, r, case["iters"], case["sweeps"], init_idx=s["idx"])
        return {"C": C, "codes": codes, "residue": r, "err": err}
    if kind == "resume":                 # the saved learner is loaded and taken further
        for to, saved in zip((C, codes, r), s["saved"]):
            to.copy_(saved)
        err = ctx.anneal(C, codes, r, case["iters"], case["sweeps"])
        return {"C": C, "codes": codes, "residue": r, "err": err}
    if kind == "online":
        err = ctx.online_chunk(s["X"], C, codes, r, want_err=True)
        return {"C": C, "codes": codes, "residue": r, "err": err}
    if kind == "improved":               # the first stage, from scratch
        C.zero_()
        codes.zero_()
        r.copy_(s["X"])
        stats = ctx.anneal_stage(0, C, codes, r, case["iters"], init_idx=s["idx"][0])
        return {"C": C[0], "codes": codes[:, 0], "residue": r, "err": stats["err_after"]}
    err = ctx.quant_error(r)             # report
    hist, joint = ctx.code_stats(codes, pair=(0, case["M"] - 1))
    var, order = ctx.reorder_by_variance(C, codes)
    return {"err": err, "hist": hist, "joint": joint, "var": var, "order": order, "C": C, "codes": codes}


def work(case):
    """Each input read and each output written once; one contraction of every vector with every codeword wherever codes are
    decided anew (per sweep and dictionary in training: what later iterations of a stage compute again is the method's choice,
    not part of the floor)."""
    N, D, M, K = case["N"], case["D"], case["M"], case["K"]
    kind = case["kind"]
    x, c, codes = 4.0 * N * D, 4.0 * M * K * D, 1.0 * N * M
    one = 2.0 * N * K * D
    if kind == "encode":
        return {"bytes": 2 * x + c + codes, "flops": one * M}
    if kind == "beam":
        return {"bytes": 2 * x + c + codes, "flops": one * (1 + (M - 1) * min(case["L"], K))}
    if kind == "train":
        return {"bytes": 2 * x + c + codes, "flops": one * M * case["sweeps"]}
    if kind == "resume":
        return {"bytes": 2 * x + 2 * c + 2 * codes, "flops": one * M * case["sweeps"]}
    if kind == "online":
        return {"bytes": 1.25 * x + 2 * c + codes, "flops": 2 * one * M}
    if kind == "improved":
        # second moments, rotation, one full assignment
        return {"bytes": 2 * x + c / M + 2.0 * N, "flops": 1.0 * N * D * D + 2.0 * N * D * D + one}
    return {"bytes": x + 2 * c + 2 * codes, "flops": 2.0 * N * D}


def tolerance(case):
    kind = case["kind"]
    if kind == "report":                 # whole numbers; the error and the variances are 64-bit sums (measured: 1e-16)
        return {"rel": 1e-12, "max": 1e-11}
    if kind in ("encode", "beam"):
        # Decisions are those of direct-form distances in 64 bits of 32-bit rows that are rounded once per dictionary: the same
        # bits from both contractions (measured).  Against 64 bits throughout the residues are 1.3e-7 off and no element more
        # than 2.2e-6, but for the vectors where the rounding of a row turns a near-tie (1 of 800000 codes)
        return {"rel": 5e-7, "max": 1e-5, "differ": 5e-6}
    # Training iterates k-means, where one near-tie moves everything after it.  But the decisions are those of direct-form
    # distances in 64 bits and the centroid sums are exact integers, so another contraction or another order of the work gives
    # the same bits (measured: not one code, dictionary or residue element differs between the two contractions, in any of these
    # kinds); rounding is what is left: against 64 bits C 4.8e-8, residues 2.8e-7, no element more than 2.6e-6, errors 1e-9.
    return {"rel": 1.2e-6, "max": 1e-5, "differ": 0.0}


# ---- the same in 64 bits --------------------------------------------------------------------------------------------------

_CHUNK = 1 << 26


def _nearest(r, c):
    """argmin_k ||r_n - c_k||^2 in 64 bits."""
    h = 0.5 * (c * c).sum(1)
    step = max(1, _CHUNK // c.shape[0])
    return torch.cat([(x @ c.T - h).argmax(1) for x in r.split(step)])


def _means(r, a, c):
    K = c.shape[0]
    n = torch.bincount(a, minlength=K)
    s = torch.zeros_like(c).index_add_(0, a, r)
    return torch.where(n[:, None] > 0, s / n.clamp(min=1)[:, None], c)


def _mse(r):
    return float((r * r).sum() / r.shape[0])


def _beam(X, C, L):
    N, D = X.shape
    M, K, _ = C.shape
    rows, codes = X[:, None, :], torch.zeros((N, 1, 0), dtype=torch.uint8, device=X.device)
    for m in range(M):
        Lc = rows.shape[1]
        keep = 1 if m == M - 1 else min(L, K * Lc)
        d = (rows * rows).sum(2)[:, :, None] - 2 * (rows.reshape(-1, D) @ C[m].T).reshape(N, Lc, K) + (C[m] * C[m]).sum(1)
        best = d.reshape(N, Lc * K).topk(keep, dim=1, largest=False, sorted=True).indices
        l, k = best // K, best % K
        rows = rows.gather(1, l[:, :, None].expand(-1, -1, D)) - C[m][k]
        codes = torch.cat([codes.gather(1, l[:, :, None].expand(-1, -1, m)), k[:, :, None].to(torch.uint8)], 2)
    return codes[:, 0], rows[:, 0]


def exact(case, seed):
    kind, N, D, M, K = case["kind"], case["N"], case["D"], case["M"], case["K"]
    if kind == "improved" or (kind in ("train", "resume") and case["data"] != "gmm"):
        # one near-tie of the 32-bit state (the improved k-means starts on two or three coordinates, where there are many) and
        # the two runs end in different local optima: 0.1 to 0.9 of the codes of a whole training
        return None
    s = prepare(case, seed)
    C = s["C"].double()
    if kind == "report":
        codes = s["codes"].long()
        hist = torch.stack([torch.bincount(codes[:, m], minlength=K) for m in range(M)])
        joint = torch.bincount(codes[:, 0] * K + codes[:, M - 1], minlength=K * K).reshape(K, K)
        var = ((C - C.mean(1, keepdim=True)) ** 2).sum(2).mean(1)
        order = torch.sort(var, descending=True, stable=True).indices
        return {"err": _mse(s["r"].double()), "hist": hist.cpu().numpy(), "joint": joint.cpu().numpy(), "var": var.cpu().numpy(),
                "order": order.int().cpu().numpy(), "C": C[order], "codes": s["codes"][:, order]}
    X = s["X"].double()
    codes = torch.zeros((N, M), dtype=torch.uint8, device=X.device)
    if kind == "encode":
        r = X
        for m in range(M):
            a = _nearest(r, C[m])
            codes[:, m] = a.to(torch.uint8)
            r = r - C[m][a]
        return {"codes": codes, "residue": r}
    if kind == "beam":
        step = max(1, _CHUNK // (case["L"] * max(K, D)))
        parts = [_beam(x, C, case["L"]) for x in X.split(step)]
        return {"codes": torch.cat([p[0] for p in parts]), "residue": torch.cat([p[1] for p in parts])}
    if kind == "online":
        r = X
        for m in range(M):
            a = _nearest(r, C[m])
            n = torch.bincount(a, minlength=K) + 16
            C[m] = (16.0 * C[m]).index_add_(0, a, r) / n[:, None]
            a = _nearest(r, C[m])
            codes[:, m] = a.to(torch.uint8)
            r = r - C[m][a]
        # integer data and means of few members tie often; what a tie decides moves the means: only the error has a value
        return {"C": None, "codes": None, "residue": None, "err": _mse(r)}
    r = X                                # train, resume on the well-separated mixture
    errs = np.zeros((case["sweeps"], M))
    if kind == "resume":
        codes, r = s["codes"].clone(), s["r"].double()
    for t in range(case["sweeps"]):
        for m in range(M):
            r = r + C[m][codes[:, m].long()]
            if kind == "train" and t == 0:
                C[m] = r[torch.from_numpy(s["idx"][m]).to(r.device)]
            for _ in range(case["iters"]):
                C[m] = _means(r, _nearest(r, C[m]), C[m])
            a = _nearest(r, C[m])
            codes[:, m] = a.to(torch.uint8)
            r = r - C[m][a]
            errs[t, m] = _mse(r)
    return {"C": C, "codes": codes, "residue": r, "err": errs}
