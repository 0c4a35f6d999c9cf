"""What the rounding bounds of the distance contraction take for granted about the matrix instructions, measured: the error of one
of them is a small part of what the bounds allow it of the largest magnitude it adds.  A product of fp16 numbers counts as if its
factors were not below the smallest normal number, which is how the hardware aligns subnormal ones."""
import ctypes
import os

import numpy as np
import pytest

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

TINY = 2.0 ** -14        # smallest normal fp16 number


def _run(k, A, B, C):
    from paper_1509_05194_amd import build
    lib = ctypes.CDLL(build.PROBE)
    lib.hclae_probe_allowance.restype = ctypes.c_float
    lib.hclae_probe_mfma.argtypes = [ctypes.c_int] + [ctypes.c_void_p] * 4 + [ctypes.c_int]
    a, b, c = [torch.from_numpy(np.ascontiguousarray(x)).cuda() for x in (A, B, C)]
    out = torch.empty_like(c)
    assert lib.hclae_probe_mfma(k, a.data_ptr(), b.data_ptr(), c.data_ptr(), out.data_ptr(), A.shape[0]) == 0
    return out.cpu().numpy(), lib.hclae_probe_allowance(k)


def _operands(kind, k, g, n=300):
    T = np.float32 if k == 2 else np.float16
    A, B = (g.standard_normal((n, 32, k)).astype(T) for _ in range(2))
    C = g.standard_normal((n, 32, 32)).astype(np.float32)
    if kind == "large accumulator":          # products fall off its end
        C = (C * 2.0 ** g.integers(0, 26, C.shape)).astype(np.float32)
    elif kind == "cancellation":             # products in opposite pairs, and the accumulator against the sum
        A[:, :, 1::2] = A[:, :, 0::2]
        B[:, :, 1::2] = -B[:, :, 0::2]
    elif kind == "opposed":
        C = -np.einsum("nik,njk->nij", A.astype(np.float64), B.astype(np.float64)).astype(np.float32)
    elif kind == "mixed exponents":
        A = (A * 2.0 ** g.integers(-8, 8, A.shape)).astype(T)
        B = (B * 2.0 ** g.integers(-8, 8, B.shape)).astype(T)
    elif kind == "truncation":               # products just below the last bit of the accumulator, all of one sign
        C[:] = 1.0
        A[:], B[:] = T(2.0 ** -12 * (2 - 2.0 ** -10)), T(2.0 ** -13 * (2 - 2.0 ** -10))
    elif kind == "subnormal vector":
        B, C = (B * 2.0 ** -18).astype(T), (C * 2.0 ** -18).astype(np.float32)
    elif kind == "subnormal codeword":
        A, C = (A * 2.0 ** -18).astype(T), (C * 2.0 ** -18).astype(np.float32)
    elif kind == "subnormal both":
        A, B, C = (A * 2.0 ** -18).astype(T), (B * 2.0 ** -18).astype(T), (C * 2.0 ** -34).astype(np.float32)
    return A, B, C


@pytest.mark.parametrize("kind", ["random", "large accumulator", "cancellation", "opposed", "mixed exponents", "truncation",
                                  "subnormal vector", "subnormal codeword", "subnormal both"])
@pytest.mark.parametrize("k", [16, 8, 2])
def test_error_of_one_instruction(k, kind):
    A, B, C = _operands(kind, k, np.random.default_rng(k))
    out, allowed = _run(k, A, B, C)
    # 64 bits of significand: its own rounding is nothing against 2^-24
    a, b = A.astype(np.longdouble)[:, :, None, :], B.astype(np.longdouble)[:, None, :, :]
    exact = (a * b).sum(3) + C
    least = 0.0 if k == 2 else TINY
    mag = np.maximum((np.maximum(np.abs(a), least) * np.maximum(np.abs(b), least)).max(3), np.abs(C))
    rel = float((np.abs(out - exact) / mag).max())
    print("%d terms, %s: error %.2f units of 2^-24 of the largest magnitude, allowed %.0f" % (k, kind, rel * 2 ** 24, allowed * 2 ** 24))
    assert rel <= allowed * (1.0 if k == 2 else 0.5)
    assert k == 2 or np.any(out != C)        # subnormal operands count
