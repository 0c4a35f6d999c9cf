"""The ageing of the distance bounds takes 1, 2 or 4 vectors per thread, by the number of vectors: at the sizes where that changes
and just past them, a training with the bounds ends in the same bits as one that assigns every vector every time."""
import numpy as np
import pytest
import torch

from paper_1509_05194_amd import hclae, synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("blocks,more", [(1, 0), (1, 1), (2, -1), (2, 0), (2, 1), (4, 1)])
def test_bounds_by_number_of_vectors(blocks, more):
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    N, D, M, K = 1024 * cus * blocks + more, 8, 2, 32
    assert N * K * D > 2 ** 23                           # else the stage keeps no bounds
    X = torch.from_numpy(synth.tiny_gmm(N=N, D=D)).cuda()
    idx = synth.init_indices(N, M, K)
    out = []
    for on in (True, False):
        ctx = hclae.Context(N, D, M, K)
        ctx.set_pruning(on)
        C, codes, r = torch.zeros((M, K, D), device="cuda"), torch.zeros((N, M), dtype=torch.uint8, device="cuda"), X.clone()
        ctx.anneal(C, codes, r, 6, 2, init_idx=idx)
        torch.cuda.synchronize()
        out.append([t.cpu().numpy() for t in (C, codes, r)])
        ctx.close()
    for a, b in zip(*out):
        assert np.array_equal(a, b)
