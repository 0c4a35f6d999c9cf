// Shared device helpers for the DA kernels (gfx950, wave64).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace hclae {

constexpr int kWave = 64;

typedef float floatx16 __attribute__((ext_vector_type(16)));

__device__ __forceinline__ int lane_id() { return threadIdx.x & (kWave - 1); }

// Butterfly sum over the 64 lanes of a wave; every lane ends with the same value
// (each step adds the same two operands on both partners, so the result is lane-independent).
__device__ __forceinline__ double wave_sum(double v)
{
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, kWave);
    return v;
}

__device__ __forceinline__ long long wave_sum_ll(long long v)
{
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, kWave);
    return v;
}

// Block sum in a fixed order: wave butterflies, then wave 0 adds the per-wave values
// in ascending wave order.  `scratch` holds >= blockDim.x/64 doubles.  Result valid in thread 0.
__device__ __forceinline__ double block_sum(double v, double *scratch)
{
    v = wave_sum(v);
    const int w = threadIdx.x >> 6;
    if (lane_id() == 0) scratch[w] = v;
    __syncthreads();
    double t = 0.0;
    if (threadIdx.x == 0) {
        const int nw = (blockDim.x + kWave - 1) >> 6;
        for (int i = 0; i < nw; ++i) t += scratch[i];
    }
    __syncthreads();
    return t;
}

// First column of the last 4-float piece of a row that starts below D: the clamp for unconditional row loads
// whose out-of-range columns are zeroed at use.  D itself need not be a multiple of 4 (a prefix of the
// coordinates); the row it lies in is, so the piece is inside the row.
__device__ __forceinline__ int last_piece(int D) { return ((D + 3) & ~3) - 4; }

// The largest of a signed integer over the wave, the same in every lane: six DPP steps (a row of 16 in four, then two
// broadcasts across rows), each a few cycles where a shuffle goes through the LDS crossbar.
__device__ __forceinline__ int wave_max_int(int v)
{
    const int low = (int)0x80000000;
    v = max(v, __builtin_amdgcn_update_dpp(low, v, 0x111, 0xf, 0xf, false));   // row_shr:1
    v = max(v, __builtin_amdgcn_update_dpp(low, v, 0x112, 0xf, 0xf, false));   // row_shr:2
    v = max(v, __builtin_amdgcn_update_dpp(low, v, 0x114, 0xf, 0xf, false));   // row_shr:4
    v = max(v, __builtin_amdgcn_update_dpp(low, v, 0x118, 0xf, 0xf, false));   // row_shr:8
    v = max(v, __builtin_amdgcn_update_dpp(low, v, 0x142, 0xa, 0xf, false));   // row_bcast:15 into rows 1 and 3
    v = max(v, __builtin_amdgcn_update_dpp(low, v, 0x143, 0xc, 0xf, false));   // row_bcast:31 into rows 2 and 3
    return __builtin_amdgcn_readlane(v, kWave - 1);
}

// The kVolatile + 1 largest entries of drift[0..K) (K <= 256, none negative), descending, the lowest index first among equal
// ones, with their indices; computed by the first wave of the block into LDS (top[], tk[]; unused slots 0 / -1).  Ends with a
// barrier.  Non-negative floats compare as integers do.
constexpr int kVolatile = 4;
__device__ __forceinline__ void top_drifts(const float *sdrift, int K, float *top, int *tk)
{
    if (threadIdx.x < kWave) {
        const int lane = threadIdx.x;
        int v[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) v[j] = (lane + kWave * j < K) ? __float_as_int(sdrift[lane + kWave * j]) : -1;
#pragma unroll
        for (int i = 0; i <= kVolatile; ++i) {
            const int best = wave_max_int(max(max(v[0], v[1]), max(v[2], v[3])));
            int at = -1;
#pragma unroll
            for (int j = 3; j >= 0; --j) {
                const unsigned long long who = __ballot(v[j] == best);
                if (who) at = __ffsll((unsigned long long)who) - 1 + kWave * j;
            }
            if (lane == 0) { top[i] = best > 0 ? __int_as_float(best) : 0.f; tk[i] = best > 0 ? at : -1; }
#pragma unroll
            for (int j = 0; j < 4; ++j)
                if (at == lane + kWave * j) v[j] = -1;               // struck out
        }
    }
    __syncthreads();
}

}  // namespace hclae
