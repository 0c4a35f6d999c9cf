// Support for the tests: single instructions of the distance contraction, so that what the rounding bounds of assign_half.hpp
// take for granted about them can be measured, and tables that no entry point returns.  Built next to the library, not part of it.
#include "encode.hpp"

namespace {

using namespace hclae;

// A problem per wave: out = acc + A B^T for A and B of 32 rows of K numbers (fp16; fp32 for K = 2), acc and out [32 rows of A]
// [32 rows of B].
template <int K, typename T>
__global__ __launch_bounds__(kWave) void k_probe_mfma(const T *A, const T *B, const float *acc_in, float *out)
{
    const int lane = lane_id(), h = lane >> 5, r = lane & 31;
    const size_t p = blockIdx.x;
    constexpr int J = K / 2;                                        // terms per lane
    typedef T vec __attribute__((ext_vector_type(J)));
    const vec a = *reinterpret_cast<const vec *>(A + (p * 32 + r) * K + J * h);
    const vec b = *reinterpret_cast<const vec *>(B + (p * 32 + r) * K + J * h);
    floatx16 c;
#pragma unroll
    for (int v = 0; v < 16; ++v) c[v] = acc_in[(p * 32 + 8 * (v >> 2) + 4 * h + (v & 3)) * 32 + r];
    if constexpr (K == 16) c = __builtin_amdgcn_mfma_f32_32x32x16_f16(a, b, c, 0, 0, 0);
    else if constexpr (K == 8) c = __builtin_amdgcn_mfma_f32_32x32x8f16(a, b, c, 0, 0, 0);
    else c = __builtin_amdgcn_mfma_f32_32x32x2f32(a[0], b[0], c, 0, 0, 0);
#pragma unroll
    for (int v = 0; v < 16; ++v) out[(p * 32 + 8 * (v >> 2) + 4 * h + (v & 3)) * 32 + r] = c[v];
}

}  // namespace

extern "C" {

// k: the instruction with that many terms, 16 or 8 of fp16 or 2 of fp32.  All pointers DEVICE; n problems; the default stream, synchronised.
int hclae_probe_mfma(int k, const void *A, const void *B, const float *acc, float *out, int n)
{
    if ((k != 16 && k != 8 && k != 2) || !A || !B || !acc || !out || n < 1) return -1;
    const _Float16 *a = static_cast<const _Float16 *>(A), *b = static_cast<const _Float16 *>(B);
    if (k == 16) hipLaunchKernelGGL((k_probe_mfma<16, _Float16>), dim3(n), dim3(kWave), 0, 0, a, b, acc, out);
    else if (k == 8) hipLaunchKernelGGL((k_probe_mfma<8, _Float16>), dim3(n), dim3(kWave), 0, 0, a, b, acc, out);
    else hipLaunchKernelGGL((k_probe_mfma<2, float>), dim3(n), dim3(kWave), 0, 0, static_cast<const float *>(A),
                            static_cast<const float *>(B), acc, out);
    if (hipGetLastError() != hipSuccess) return -3;
    return hipDeviceSynchronize() == hipSuccess ? 0 : -3;
}

// What the bounds allow one of them, relative to the largest magnitude it adds: half_acc, and the 2^-23 per term of rescore_items.
float hclae_probe_allowance(int k) { return k == 2 ? 2.f * 1.1920929e-7f : kHalfAccUnit; }

// -||c||^2/2 of M dictionaries as k_encode_prep leaves them, out [M][32 kb] with the smallest kb of 1, 2, 4, 8 that holds K; D <= 256.
int hclae_probe_encode_norms(const float *C, int M, int K, int D, float *out)
{
    if (!C || !out || M < 1 || K < 1 || K > 256 || D < 4 || D > 256 || D % 4) return -1;
    const int kb = K <= 32 ? 1 : K <= 64 ? 2 : K <= 128 ? 4 : 8, NC = (D + kChunkD - 1) / kChunkD, nc = NC == 3 ? 4 : NC;
    char *buf = nullptr;
    const size_t img = (size_t)M * nc * kb * 4096, tab = (size_t)M * 32 * kb, mu = (size_t)M * kChunkD * nc;
    if (hipMalloc((void **)&buf, img + sizeof(float) * (2 * tab + mu + M * kEncodeConsts + 4)) != hipSuccess) return -3;
    float *hn = reinterpret_cast<float *>(buf + img), *w = hn + tab, *negmu = w + tab, *consts = negmu + mu;
    hipLaunchKernelGGL(k_encode_prep<true>, dim3(2 * M), dim3(kPrepThreads), 0, 0, C, K, D, kb, nc, buf, hn, w, negmu, consts, out,
                       reinterpret_cast<unsigned *>(consts + M * kEncodeConsts));
    const bool ok = hipGetLastError() == hipSuccess && hipDeviceSynchronize() == hipSuccess;
    (void)hipFree(buf);
    return ok ? 0 : -3;
}

}
