"""The codeword norms behind the second scoring of the large encoder come from 64-bit sums: -||c||^2/2 to the last bit but one rounding,
as the bound of those scores assumes, also where squares of very different size are added."""
import ctypes

import numpy as np
import pytest

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("M,K,D", [(1, 1, 4), (3, 33, 20), (2, 130, 64), (2, 256, 128), (1, 100, 256)])
def test_norms_are_rounded_once(M, K, D):
    from paper_1509_05194_amd import build
    g = np.random.default_rng(D)
    C = (g.standard_normal((M, K, D)) * 2.0 ** g.integers(-12, 1, (M, K, D))).astype(np.float32)
    kpad = next(32 * b for b in (1, 2, 4, 8) if 32 * b >= K)
    lib = ctypes.CDLL(build.PROBE)
    lib.hclae_probe_encode_norms.argtypes = [ctypes.c_void_p] + [ctypes.c_int] * 3 + [ctypes.c_void_p]
    c, out = torch.from_numpy(C).cuda(), torch.full((M, kpad), 7.0, device="cuda")
    assert lib.hclae_probe_encode_norms(c.data_ptr(), M, K, D, out.data_ptr()) == 0
    got = out.cpu().numpy()
    want = -0.5 * (C.astype(np.float64) ** 2).sum(2)
    # half a unit of the last place of fp32, and what 64-bit sums in another order differ by
    assert (np.abs(got[:, :K] - want) <= np.abs(want) * (2.0 ** -24 + 1e-13)).all()
    assert np.isneginf(got[:, K:]).all()
