// Nearest-codeword assignment with the distance contraction on the bf16 matrix cores
// (v_mfma_f32_32x32x16_bf16, 16x the rate of the fp32 MFMA on gfx950), fp32 operands split
// into two bf16 terms each:  x = xh + xl + dx,  c = ch + cl + dc  with |dx| <= 2^-16 |x|.
// The score x.c - ||c||^2/2 is accumulated in fp32 as  xh.ch + xh.cl + xl.ch  (three MFMAs per
// 16 dims); what is dropped, xl.cl + dx.c + x.dc, is bounded by norms the kernel has, and that
// bound joins the rounding bound of the accumulation in the margin of the decision: every codeword
// whose score is within the margin of the best goes to the same fp64 direct-form re-check
// (k_refine) as in the fp32 kernel.  The contraction only pre-selects candidates, so the codes
// are the same fp64 direct-form decisions whichever kernel ran.
//
// Accumulation error of one 32x32x16 bf16 MFMA, measured on gfx950 over 4.6e6 random sums with
// exponent spreads up to 2^+-16: at most 4.9 * 2^-24 * (|C| + sum |a_k b_k|).  The margin assumes
// 2^-21 (8 * 2^-24) per MFMA.
#pragma once
#include "assign.hpp"

namespace hclae {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float floatx2 __attribute__((ext_vector_type(2)));

constexpr int kSplitStep = 16;                      // dims per bf16 MFMA

// (a, b) -> packed bf16 pairs hi = RNE(a, b), lo = RNE(a - hi_a, b - hi_b); element 0 in the low half.
__device__ __forceinline__ void split_pair(float a, float b, uint32_t &hi, uint32_t &lo)
{
    const floatx2 v = {a, b};
    hi = __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2));
    const float ha = __uint_as_float(hi << 16), hb = __uint_as_float(hi & 0xffff0000u);
    const floatx2 rem = {a - ha, b - hb};            // exact: hi keeps the leading 8 bits
    lo = __builtin_bit_cast(uint32_t, __builtin_convertvector(rem, bf16x2));
}

__device__ __forceinline__ void split8(const float4 &u, const float4 &v, uint4 &hi, uint4 &lo)
{
    split_pair(u.x, u.y, hi.x, lo.x);
    split_pair(u.z, u.w, hi.y, lo.y);
    split_pair(v.x, v.y, hi.z, lo.z);
    split_pair(v.z, v.w, hi.w, lo.w);
}

// Per-codeword constants of the split over the first D coordinates (row stride ld), as fp32 rounded up:
//   out[2k] = || cl_k ||  (low part),   out[2k + 1] = || c_k - ch_k - cl_k ||  (what two terms miss).
// One wave per codeword; the assign kernel takes the maxima over k.
__global__ __launch_bounds__(256) void k_split_norms(
    const float *__restrict__ Cm, int K, int D, int ld, float *__restrict__ out)
{
    const int lane = lane_id();
    const int k = blockIdx.x * (256 / kWave) + (threadIdx.x >> 6);
    if (k >= K) return;
    const float *c = Cm + (size_t)k * ld;
    double sl = 0.0, sd = 0.0;
    for (int d = lane; d < D; d += kWave) {
        uint32_t hi, lo;
        split_pair(c[d], 0.f, hi, lo);
        const float ch = __uint_as_float(hi << 16), cl = __uint_as_float(lo << 16);
        const double dc = ((double)c[d] - (double)ch) - (double)cl;
        sl += (double)cl * (double)cl;
        sd += dc * dc;
    }
    sl = wave_sum(sl);
    sd = wave_sum(sd);
    if (lane == 0) {
        out[2 * k] = (float)(sqrt(sl) * 1.000001);
        out[2 * k + 1] = (float)(sqrt(sd) * 1.000001);
    }
}

// LDS image of the split codebook in MFMA operand order.  For step t (16 dims), row block b (32
// codewords), part p (0 = high, 1 = low) and lane l = 32 g + r, the uint4 at ((t*kb + b)*2 + p)*64 + l
// holds the bf16 values of C[32b + r][16t + 8g .. 16t + 8g + 7]: every operand read is one
// contiguous kilobyte, and the reads of one 64-dim chunk are one base address plus constants below 64 KB.
// Coordinates beyond D and rows beyond K are zero.
__device__ __forceinline__ void stage_codebook_split(
    uint4 *lds, const float *__restrict__ Cm, int K, int D, int ld, int kb, int T)
{
    const int total = kb * T * kWave;
    for (int e = threadIdx.x; e < total; e += blockDim.x) {
        const int l = e & 63;
        const int tb = e >> 6;
        const int b = tb % kb;
        const int t = tb / kb;
        const int row = 32 * b + (l & 31);
        const int col = kSplitStep * t + 8 * (l >> 5);
        const float4 u = load_row_piece(Cm, row, col, K, D, ld);
        const float4 v = load_row_piece(Cm, row, col + 4, K, D, ld);
        uint4 hi, lo;
        split8(u, v, hi, lo);
        lds[(size_t)(tb * 2 + 0) * kWave + l] = hi;
        lds[(size_t)(tb * 2 + 1) * kWave + l] = lo;
    }
}

// The 64-dim chunk q of a row in B-operand order: lane (g, r) gets, for step t = 0..3, the eight
// floats x'[row r][64q + 16t + 8g .. + 7] as x[2t], x[2t + 1].
__device__ __forceinline__ void load_x_chunk_split(
    float4 (&x)[8], const float *__restrict__ xrow, int q, int g, int D)
{
#pragma unroll
    for (int t = 0; t < 4; ++t) {
        const int col = kChunkD * q + kSplitStep * t + 8 * g;
        x[2 * t] = (col < D) ? *reinterpret_cast<const float4 *>(xrow + col) : make_float4(0.f, 0.f, 0.f, 0.f);
        x[2 * t + 1] = (col + 4 < D) ? *reinterpret_cast<const float4 *>(xrow + col + 4) : make_float4(0.f, 0.f, 0.f, 0.f);
    }
}

template <int KB>
__device__ __forceinline__ void mfma_chunk_split(
    floatx16 (&acc)[KB], const float4 (&x)[8], const uint4 *__restrict__ lds, int q, int T, int lane,
    float &xsq, float &amax)
{
    constexpr int GB = KB < 4 ? KB : 4;              // codeword blocks whose operands are in registers at once
    const uint4 *chunk = lds + (size_t)(4 * q) * KB * 2 * kWave + lane;
    (void)T;
#pragma unroll
    for (int t = 0; t < 4; ++t) {
        const float4 u = x[2 * t], v = x[2 * t + 1];
        xsq = fmaf(u.x, u.x, xsq);
        xsq = fmaf(u.y, u.y, xsq);
        xsq = fmaf(u.z, u.z, xsq);
        xsq = fmaf(u.w, u.w, xsq);
        xsq = fmaf(v.x, v.x, xsq);
        xsq = fmaf(v.y, v.y, xsq);
        xsq = fmaf(v.z, v.z, xsq);
        xsq = fmaf(v.w, v.w, xsq);
        amax = fmaxf(fmaxf(amax, fabsf(u.x)), fabsf(u.y));      // one v_max3_f32 per two elements
        amax = fmaxf(fmaxf(amax, fabsf(u.z)), fabsf(u.w));
        amax = fmaxf(fmaxf(amax, fabsf(v.x)), fabsf(v.y));
        amax = fmaxf(fmaxf(amax, fabsf(v.z)), fabsf(v.w));
        uint4 xh4, xl4;
        split8(u, v, xh4, xl4);
        const bf16x8 xh = __builtin_bit_cast(bf16x8, xh4), xl = __builtin_bit_cast(bf16x8, xl4);
#pragma unroll
        for (int b0 = 0; b0 < KB; b0 += GB) {
            bf16x8 ch[GB], cl[GB];
#pragma unroll
            for (int b = 0; b < GB; ++b) {
                const uint4 *at = chunk + ((t * KB + b0 + b) * 2) * kWave;      // compile-time offset
                ch[b] = __builtin_bit_cast(bf16x8, at[0]);
                cl[b] = __builtin_bit_cast(bf16x8, at[kWave]);
            }
#pragma unroll
            for (int b = 0; b < GB; ++b) acc[b0 + b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(cl[b], xh, acc[b0 + b], 0, 0, 0);
#pragma unroll
            for (int b = 0; b < GB; ++b) acc[b0 + b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ch[b], xl, acc[b0 + b], 0, 0, 0);
#pragma unroll
            for (int b = 0; b < GB; ++b) acc[b0 + b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ch[b], xh, acc[b0 + b], 0, 0, 0);
        }
    }
}

// ---- the same contraction for dimensions whose codebook does not fit LDS ---------------------------------

// Split codebook in the order the D-chunked split kernel stages it: the slice of 64-dim chunk q is KB * 512
// uint4 laid out as in stage_codebook_split with chunk-local steps t = 0..3 (element ((t*KB + b)*2 + p)*64 + l),
// slices one after the other.  Same size as the fp32 image of k_codebook_image.
__global__ __launch_bounds__(256) void k_codebook_image_split(
    const float *__restrict__ Cm, int K, int D, int ld, int kb, int NC, uint4 *__restrict__ img)
{
    const int total = NC * 4 * kb * kWave;                          // (q, t, b, l)
    for (int e = blockIdx.x * 256 + threadIdx.x; e < total; e += gridDim.x * 256) {
        const int l = e & 63;
        int tb = e >> 6;
        const int b = tb % kb;
        tb /= kb;
        const int t = tb & 3, q = tb >> 2;
        const int row = 32 * b + (l & 31);
        const int col = kChunkD * q + kSplitStep * t + 8 * (l >> 5);
        const float4 u = load_row_piece(Cm, row, col, K, D, ld);
        const float4 v = load_row_piece(Cm, row, col + 4, K, D, ld);
        uint4 hi, lo;
        split8(u, v, hi, lo);
        uint4 *dst = img + (size_t)q * kb * 8 * kWave + (size_t)((t * kb + b) * 2) * kWave + l;
        dst[0] = hi;
        dst[kWave] = lo;
    }
}

// One 64-dim chunk of the D-chunked split kernel (see mfma_chunk_refill): contracts x with the slice in `cur`
// while the next slice and the next chunk of x' arrive.  Each 16-dim step fetches its share of the thread's KB
// pieces of the next slice (src: its uint4 of piece 0; pieces are 8 * 64 uint4 apart) at its start and stores
// them to `nxt` late in the step; x[2t], x[2t+1] are refilled from xnext as soon as step t has them.
template <int KB>
__device__ __forceinline__ void mfma_chunk_split_refill(
    floatx16 (&acc)[KB], float4 (&x)[8], const uint4 *__restrict__ cur, uint4 *__restrict__ nxt,
    const uint4 *__restrict__ src, const float *__restrict__ xnext, int q, int qn, int D, int lane, int wave,
    float &xsq, float &amax)
{
    constexpr int GB = KB < 4 ? KB : 4;
    constexpr int PP = (KB + 3) / 4;                                // pieces fetched per step
    const int g = lane >> 5;
    const uint4 *chunk = cur + lane;
#pragma unroll
    for (int t = 0; t < 4; ++t) {
        // Fetched as relaxed atomics (two 64-bit halves) and fenced for the scheduler: an ordinary load would be
        // moved down next to its use, where its latency is no longer covered.
        unsigned long long piece[PP][2];
#pragma unroll
        for (int i = 0; i < PP; ++i)
            if (t * PP + i < KB) {
                const unsigned long long *s64 = reinterpret_cast<const unsigned long long *>(src + (t * PP + i) * 8 * kWave);
                piece[i][0] = __hip_atomic_load(s64, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
                piece[i][1] = __hip_atomic_load(s64 + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
            }
        __builtin_amdgcn_sched_barrier(0x10f);
        float4 u = x[2 * t], v = x[2 * t + 1];
        {
            // columns past D are zeroed at use; the refill is unconditional, its address clamped into the row
            const int col = kChunkD * q + kSplitStep * t + 8 * g;
            if (col >= D) u = make_float4(0.f, 0.f, 0.f, 0.f);
            if (col + 4 >= D) v = make_float4(0.f, 0.f, 0.f, 0.f);
            const int coln = kChunkD * qn + kSplitStep * t + 8 * g;
            x[2 * t] = *reinterpret_cast<const float4 *>(xnext + min(coln, last_piece(D)));
            x[2 * t + 1] = *reinterpret_cast<const float4 *>(xnext + min(coln + 4, last_piece(D)));
        }
        xsq = fmaf(u.x, u.x, xsq);
        xsq = fmaf(u.y, u.y, xsq);
        xsq = fmaf(u.z, u.z, xsq);
        xsq = fmaf(u.w, u.w, xsq);
        xsq = fmaf(v.x, v.x, xsq);
        xsq = fmaf(v.y, v.y, xsq);
        xsq = fmaf(v.z, v.z, xsq);
        xsq = fmaf(v.w, v.w, xsq);
        amax = fmaxf(fmaxf(amax, fabsf(u.x)), fabsf(u.y));
        amax = fmaxf(fmaxf(amax, fabsf(u.z)), fabsf(u.w));
        amax = fmaxf(fmaxf(amax, fabsf(v.x)), fabsf(v.y));
        amax = fmaxf(fmaxf(amax, fabsf(v.z)), fabsf(v.w));
        uint4 xh4, xl4;
        split8(u, v, xh4, xl4);
        const bf16x8 xh = __builtin_bit_cast(bf16x8, xh4), xl = __builtin_bit_cast(bf16x8, xl4);
#pragma unroll
        for (int b0 = 0; b0 < KB; b0 += GB) {
            bf16x8 ch[GB], cl[GB];
#pragma unroll
            for (int b = 0; b < GB; ++b) {
                const uint4 *at = chunk + ((t * KB + b0 + b) * 2) * kWave;      // compile-time offset
                ch[b] = __builtin_bit_cast(bf16x8, at[0]);
                cl[b] = __builtin_bit_cast(bf16x8, at[kWave]);
            }
#pragma unroll
            for (int b = 0; b < GB; ++b) acc[b0 + b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(cl[b], xh, acc[b0 + b], 0, 0, 0);
#pragma unroll
            for (int b = 0; b < GB; ++b) acc[b0 + b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ch[b], xl, acc[b0 + b], 0, 0, 0);
            if (b0 + GB >= KB) {
                // the stores (and the waits for their loads) stay behind most of the step's MFMAs
                __builtin_amdgcn_sched_barrier(0x10f);
#pragma unroll
                for (int i = 0; i < PP; ++i)
                    if (t * PP + i < KB) {
                        uint4 v4;
                        v4.x = (uint32_t)piece[i][0]; v4.y = (uint32_t)(piece[i][0] >> 32);
                        v4.z = (uint32_t)piece[i][1]; v4.w = (uint32_t)(piece[i][1] >> 32);
                        nxt[((t * PP + i) * 8 + wave) * kWave + lane] = v4;
                    }
            }
#pragma unroll
            for (int b = 0; b < GB; ++b) acc[b0 + b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ch[b], xh, acc[b0 + b], 0, 0, 0);
        }
    }
}

}  // namespace hclae
