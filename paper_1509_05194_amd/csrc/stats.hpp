// Dictionary ordering and code statistics (Sec. 3.3: dictionaries in descending order of the variance of
// their elements; Sec. 2.2: self-information H(I_m) and mutual information of the code parts).
// Small integer / fp64 kernels.
#pragma once
#include "common.hpp"

namespace hclae {

// var[m] = (1/K) sum_k || c_m(k) - mean_k c_m ||^2, fp64, one block per dictionary.
__global__ __launch_bounds__(256) void k_dictionary_variance(
    const float *__restrict__ C, int K, int D, double *__restrict__ var)
{
    __shared__ double red[256 / kWave];
    const float *Cm = C + (size_t)blockIdx.x * K * D;
    double acc = 0.0;
    for (int d = threadIdx.x; d < D; d += 256) {
        double s = 0.0;
        // one load after the other is all this kernel would be (95 us for M = 8, K = 256, D = 128): unrolled for 32 of them in
        // flight, the additions keep their order (12 us)
#pragma unroll 32
        for (int k = 0; k < K; ++k) s += (double)Cm[(size_t)k * D + d];
        const double mu = s / (double)K;
        double q = 0.0;
#pragma unroll 32
        for (int k = 0; k < K; ++k) {
            const double t = (double)Cm[(size_t)k * D + d] - mu;
            q += t * t;
        }
        acc += q;
    }
    acc = block_sum(acc, red);
    if (threadIdx.x == 0) var[blockIdx.x] = acc / (double)K;
}

// dst[j] = src[order[j]] for whole dictionaries (K*D floats each).
__global__ __launch_bounds__(256) void k_permute_dictionaries(
    const float *__restrict__ src, const int *__restrict__ order, int M, size_t per, float *__restrict__ dst)
{
    const size_t total = (size_t)M * per;
    for (size_t i = (size_t)blockIdx.x * 256 + threadIdx.x; i < total; i += (size_t)gridDim.x * 256) {
        const size_t j = i / per;
        dst[i] = src[(size_t)order[j] * per + (i - j * per)];
    }
}

// codes[n][j] <- codes[n][order[j]] in place, one thread per row (M <= 256 bytes per row).
__global__ __launch_bounds__(256) void k_permute_code_columns(
    uint8_t *__restrict__ codes, const int *__restrict__ order, int64_t N, int M)
{
    for (int64_t n = (int64_t)blockIdx.x * 256 + threadIdx.x; n < N; n += (int64_t)gridDim.x * 256) {
        uint8_t *row = codes + n * M;
        uint8_t tmp[256];
        for (int j = 0; j < M; ++j) tmp[j] = row[order[j]];
        for (int j = 0; j < M; ++j) row[j] = tmp[j];
    }
}

__global__ __launch_bounds__(256) void k_zero_u64(unsigned long long *p, size_t n)
{
    for (size_t i = (size_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (size_t)gridDim.x * 256) p[i] = 0ull;
}

// hist[m][k] += 1 for every code of the columns m0 .. m0 + cols - 1 (gridDim.y groups of `cols` columns); joint[ka][kb] += 1
// for the pair of columns (a, b) when joint != null.  Integer atomics: the result does not depend on the order.
//
// The M K counters are few and every one is hit N / K times: global atomics on them queue (1206 us for N = 1M, M = 8, K = 256),
// so a block counts in LDS and adds its counts once; few blocks, because that is M K global atomics each.  The K x K joint
// counters are many and take their N additions directly.
// A thread's bytes all belong to one column: it strides by a multiple of the row length.  `wide`: a row length that divides 16
// and an aligned array, 16 codes per load; the column of byte j is j mod M.
constexpr int kHistThreads = 1024;
constexpr int kHistBlocks = 64;
constexpr int kHistLds = 64 * 1024;                 // bytes of counters per block
__global__ __launch_bounds__(kHistThreads) void k_code_histograms(
    const uint8_t *__restrict__ codes, int64_t N, int M, int K, int cols, int a, int b, int wide,
    unsigned long long *__restrict__ hist, unsigned long long *__restrict__ joint)
{
    extern __shared__ float4 smem4[];
    unsigned *cnt = reinterpret_cast<unsigned *>(smem4);            // [cols][K]
    const int m0 = blockIdx.y * cols;
    const int mine = min(cols, M - m0);
    for (int i = threadIdx.x; i < mine * K; i += kHistThreads) cnt[i] = 0u;
    __syncthreads();
    const int64_t t = (int64_t)blockIdx.x * kHistThreads + threadIdx.x, threads = (int64_t)gridDim.x * kHistThreads;
    if (wide) {
        const int64_t n16 = N * M >> 4;                             // M divides 16; the last N M mod 16 bytes go one by one
        for (int64_t i0 = t; i0 < n16; i0 += 4 * threads) {
            uint4 w[4];
#pragma unroll
            for (int u = 0; u < 4; ++u)
                w[u] = reinterpret_cast<const uint4 *>(codes)[i0 + u * threads < n16 ? i0 + u * threads : i0];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                if (i0 + u * threads >= n16) break;
                const unsigned v[4] = {w[u].x, w[u].y, w[u].z, w[u].w};
#pragma unroll
                for (int j = 0; j < 16; ++j) atomicAdd(cnt + (j & (M - 1)) * K + ((v[j >> 2] >> (8 * (j & 3))) & 255u), 1u);
            }
        }
        if (blockIdx.x == 0 && 16 * n16 + threadIdx.x < N * M) {
            const int64_t i = 16 * n16 + threadIdx.x;
            atomicAdd(cnt + (i & (M - 1)) * K + codes[i], 1u);
        }
    } else {
        const int64_t rows = threads / mine;                        // rows a sweep of all threads covers
        if (t < rows * mine) {
            const int c = (int)(t % mine);
            for (int64_t n = t / mine; n < N; n += rows) atomicAdd(cnt + c * K + codes[n * M + m0 + c], 1u);
        }
    }
    if (joint && blockIdx.y == 0)
        for (int64_t n = t; n < N; n += threads) atomicAdd(joint + (size_t)codes[n * M + a] * K + codes[n * M + b], 1ull);
    __syncthreads();
    for (int i = threadIdx.x; i < mine * K; i += kHistThreads)
        if (cnt[i]) atomicAdd(hist + (size_t)m0 * K + i, (unsigned long long)cnt[i]);
}

}  // namespace hclae
