"""hclae_set_pruning(0) makes every centroid sum of a stage run over all vectors, in stages cooled by the improved k-means too; the
results are the same bits either way."""
import numpy as np
import pytest

from paper_1509_05194_amd import hclae, synth

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("N,D,K", [(700, 16, 16), (40000 + 9, 32, 64)])
def test_improved_stage_without_the_shortcuts(N, D, K):
    X = torch.from_numpy(synth.tiny_gmm(N=N, D=D)).cuda()
    idx = synth.init_indices(N, 1, K)[0]
    out = []
    for on in (True, False):
        ctx = hclae.Context(N, D, 1, K)
        ctx.set_cooldown(True, 4)
        ctx.set_pruning(on)
        C, codes, r = torch.zeros((1, K, D), device="cuda"), torch.zeros((N, 1), dtype=torch.uint8, device="cuda"), X.clone()
        ctx.timing_enable(["accumulate", "accumulate_moved"])
        stats = ctx.anneal_stage(0, C, codes, r, 8, init_idx=idx)
        times = ctx.timing_read()
        if not on:
            assert times["accumulate_moved"][1] == 0 and times["accumulate"][1] == stats["iters_run"] > 1
        out.append([t.cpu().numpy() for t in (C, codes, r)] + [stats["err_after"]])
        ctx.close()
    for a, b in zip(*out):
        assert np.array_equal(a, b)
