"""The code counters (Sec. 2.2) where their kernel splits the work differently: row lengths that divide 16 and that do not, more
columns than a block's LDS holds, codes that are not 16-byte aligned."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("N,M,K,offset", [(1, 1, 1, 0), (1000, 8, 256, 0), (100003, 16, 256, 0), (5000, 8, 100, 3), (3001, 3, 7, 0),
                                          (70000, 5, 256, 1), (2000, 100, 256, 0), (999, 256, 256, 0), (65, 2, 2, 0)])
def test_code_counts(N, M, K, offset):
    from paper_1509_05194_amd import hclae
    rng = np.random.default_rng(N + M)
    flat = torch.zeros(N * M + offset, dtype=torch.uint8, device="cuda:0")
    codes = flat[offset:].view(N, M)
    host = rng.integers(0, K, (N, M)).astype(np.uint8)
    host[: N // 2, 0] = 0                                    # half of a column in one counter
    codes.copy_(torch.from_numpy(host))
    ctx = hclae.Context(N, 4, M, K)
    hist, joint = ctx.code_stats(codes, pair=(0, M - 1))
    ctx.close()
    for m in range(M):
        np.testing.assert_array_equal(hist[m], np.bincount(host[:, m], minlength=K))
    want = np.bincount(host[:, 0].astype(np.int64) * K + host[:, M - 1], minlength=K * K).reshape(K, K)
    np.testing.assert_array_equal(joint, want)
