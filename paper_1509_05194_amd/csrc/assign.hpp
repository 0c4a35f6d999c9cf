// What the nearest-codeword assignments share (assign_half.hpp holds their kernels), the fp32 contraction of the rotation, and the
// distance bounds of a stage.
//
// argmin_k ||x' - c_k||^2 = argmax_k ( x'.c_k - ||c_k||^2/2 ).  The right-hand score is a dense K x D by D x N contraction.
// The product is oriented codewords x vectors, so a lane ends up holding scores of many codewords for ONE vector and the
// argmax never leaves the wave (one exchange between lane l and lane l+32 at the end).
#pragma once
#include "common.hpp"

namespace hclae {

constexpr int kAssignThreads = 512;                 // 8 waves: 2 per SIMD
constexpr int kAssignWaves = kAssignThreads / kWave;
constexpr int kTileVec = 32;                        // vectors per wave tile (N side of the MFMA)
constexpr int kChunkD = 64;                         // dims per register-resident chunk of x'

// Exact pruning of the assignments of one stage (x' fixed, only the dictionary moves).  For every vector
// the stage keeps an upper bound bu on the distance to its own codeword and a lower bound bl on the
// distance to every other one, both widened by the rounding bound of the scores.  When
// the dictionary moves, bu grows by the drift of the own codeword and bl shrinks by the largest drift
// of another one (triangle inequality); while bu < bl the own codeword is still the unique nearest
// and the vector is not recomputed.  The others are listed (k_bounds_step) and go through the same
// contraction and decision as before, which also renews their bounds.  The codes are
// therefore exactly those of full assignments.
//   PRUNE 0: plain assignment.  1: all vectors, and store their bounds.  2: only active[0..*active_count),
//   and store their bounds.
struct PruneArgs {
    float *bu, *bl;                    // [N]
    const uint32_t *active;            // [*active_count] vector indices (PRUNE 2)
    const unsigned *active_count;
    float slack;                       // rounding of ||x'||^2 and of the bound arithmetic, relative: grows with D
};

// -||c_k||^2 / 2 in fp32 (computed in fp64) over the first D coordinates of rows of stride ld, for
// k < K; -inf for the padding rows up to kpad.
// One wave per codeword.  Also resets the two counters the assign that follows will fill
// (refine_count[0]: vectors its scores leave undecided, refine_count[1]: bits of max |x'|).
// keep_absmax 2: max |x'| was left by the row pass that wrote x', spread over amax_parts[0..64) (block_absmax): the
// largest word becomes refine_count[1] and the words are cleared for the next such pass.
// entry_copy (or nullptr): receives the K x D dictionary as it is now (the carried bounds price a stage by how far
// it moves from here); zero_word (or nullptr): a counter cleared for the kernel that follows.
__global__ __launch_bounds__(256) void k_codeword_norms(
    const float *__restrict__ Cm, int K, int D, int ld, int kpad, float *__restrict__ hneg,
    unsigned *__restrict__ refine_count, int keep_absmax,
    unsigned *__restrict__ amax_parts = nullptr, float *__restrict__ entry_copy = nullptr,
    unsigned *__restrict__ zero_word = nullptr)
{
    const int lane = lane_id();
    const int k = blockIdx.x * (256 / kWave) + (threadIdx.x >> 6);
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        refine_count[0] = 0u;                      // undecided vectors
        if (!keep_absmax) refine_count[1] = 0u;    // bits of max |x'|
        if (keep_absmax == 2) {
            unsigned mx = 0u;
            for (int i = 0; i < 64; ++i) {
                mx = max(mx, amax_parts[i]);
                amax_parts[i] = 0u;
            }
            refine_count[1] = mx;
        }
        if (zero_word) *zero_word = 0u;
    }
    if (k >= kpad) return;
    if (k >= K) {
        if (lane == 0) hneg[k] = -__builtin_inff();
        return;
    }
    const float *c = Cm + (size_t)k * ld;
    double s = 0.0;
    for (int d = lane; d < D; d += kWave) {
        const float v = c[d];
        s += (double)v * (double)v;
        if (entry_copy) entry_copy[(size_t)k * D + d] = v;
    }
    s = wave_sum(s);
    if (lane == 0) hneg[k] = -(float)(0.5 * s);
}

// Four coordinates of a row from column col: zero beyond the first D coordinates and beyond the first K rows (stride ld), so that
// whatever the other operand holds there contributes nothing to a product.
__device__ __forceinline__ float4 load_row_piece(const float *__restrict__ base, int row, int col, int K, int D, int ld)
{
    float4 v = make_float4(0.f, 0.f, 0.f, 0.f);
    if (row < K && col < D) {
        v = *reinterpret_cast<const float4 *>(base + (size_t)row * ld + col);
        if (col + 3 >= D) {                        // D need not be a multiple of 4
            if (col + 1 >= D) v.y = 0.f;
            if (col + 2 >= D) v.z = 0.f;
            v.w = 0.f;
        }
    }
    return v;
}

// Loads the 64-dim chunk q of the wave's 32-vector tile into B-operand order:
// lane (h, r) gets x'[row r][64q + 8s + 4h .. +3] for s = 0..7.
// PREFIX: only the first `steps` 8-dim steps of the chunk are wanted (the others are not contracted either).
template <bool PREFIX = false>
__device__ __forceinline__ void load_x_chunk(
    float4 (&x)[8], const float *__restrict__ xrow, int q, int h, int D, int steps = 8)
{
    if (!PREFIX && kChunkD * (q + 1) <= D) {               // a whole chunk (uniform): no lane masks around the loads
        const float4 *p = reinterpret_cast<const float4 *>(xrow + kChunkD * q + 4 * h);
#pragma unroll
        for (int s = 0; s < 8; ++s) x[s] = p[2 * s];
        return;
    }
#pragma unroll
    for (int s = 0; s < 8; ++s) {
        const int col = kChunkD * q + 8 * s + 4 * h;
        x[s] = (col < D && (!PREFIX || s < steps)) ? *reinterpret_cast<const float4 *>(xrow + col)
                                                   : make_float4(0.f, 0.f, 0.f, 0.f);
    }
}

// One chunk of the fp32 contraction: lds holds the rows of the other operand in MFMA order (for row block b, 8-dim step s and lane
// l = 32 h + r the float4 at (b S + s) 64 + l is row 32 b + r, dims 8 s + 4 h .. + 3; component j contracts dims 8 s + j, 8 s + 4 + j).
template <int KB>
__device__ __forceinline__ void mfma_chunk(
    floatx16 (&acc)[KB], const float4 (&x)[8], const float4 *__restrict__ lds, int S, int lane)
{
#pragma unroll
    for (int s = 0; s < 8; ++s) {
        float4 a[KB];
#pragma unroll
        for (int b = 0; b < KB; ++b) a[b] = lds[(b * S + s) * kWave + lane];
        const float4 xv = x[s];
#pragma unroll
        for (int b = 0; b < KB; ++b) acc[b] = __builtin_amdgcn_mfma_f32_32x32x2f32(a[b].x, xv.x, acc[b], 0, 0, 0);
#pragma unroll
        for (int b = 0; b < KB; ++b) acc[b] = __builtin_amdgcn_mfma_f32_32x32x2f32(a[b].y, xv.y, acc[b], 0, 0, 0);
#pragma unroll
        for (int b = 0; b < KB; ++b) acc[b] = __builtin_amdgcn_mfma_f32_32x32x2f32(a[b].z, xv.z, acc[b], 0, 0, 0);
#pragma unroll
        for (int b = 0; b < KB; ++b) acc[b] = __builtin_amdgcn_mfma_f32_32x32x2f32(a[b].w, xv.w, acc[b], 0, 0, 0);
    }
}

// Accumulator start: element v of block b in lane (h, r) belongs to codeword
// 32b + 8(v/4) + 4h + v%4 (the 32x32 fp32 MFMA result layout).
template <int KB>
__device__ __forceinline__ void init_acc(floatx16 (&acc)[KB], const float *hneg_lds, int h)
{
#pragma unroll
    for (int b = 0; b < KB; ++b) {
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            const float4 t = *reinterpret_cast<const float4 *>(hneg_lds + 32 * b + 8 * g + 4 * h);
            acc[b][4 * g + 0] = t.x;
            acc[b][4 * g + 1] = t.y;
            acc[b][4 * g + 2] = t.z;
            acc[b][4 * g + 3] = t.w;
        }
    }
}

// Between two assignments of a stage: age the bounds by the drift of the dictionary (drift[k] >= the
// distance codeword k moved in the centroid update, 0 for a kept one) and list the vectors that have to be
// recomputed.  A block takes kBoundThreads U consecutive vectors, stages its entries in LDS and claims its stretch
// of the list with one counter add (*count must be zero on entry; order is free).
//
// One codeword that moves far (a cluster of few members) costs every vector its lower bound.  When the
// largest drift stands out from the (kVolatile+1)-th, the block looks again at those of its unsettled vectors
// that the drift of the REST alone would leave settled (if they are many), with the kVolatile codewords that
// moved most treated apart: the lower bound ages by the largest drift of the rest, and the distance to each of
// those few is computed afresh from x' (expanded form in fp32 with its rounding bound) and joins the lower bound.
// Vectors that this settles get their aged bounds and leave the list.  Eight lanes share a vector.
// Dynamic LDS: kVolatile rows of D floats.
// U, the vectors per thread: the fewest of 1, 2 and 4 with which no CU has a second block (4 beyond).  The ranking of the drifts is a prologue
// that every block pays for, so fewer and larger blocks win once they would run one after another; below that the second look, a chain of
// gathers, wants the CUs.  Measured, us with 1 / 2 / 4 (two sweeps of four dictionaries, D = 128, K = 256, 256 CUs): N = 150k 9.4 / 9.7 / 11.7,
// 300k 11.0 / 9.1 / 9.3, 400k 12.0 / 9.5 / 9.6, 524k 13.3 / 10.6 / 10.3, 600k 14.4 / 12.2 / 10.2, 800k 17.7 / 14.0 / 11.6, 1M 20.9 / 15.7 /
// 13.6, 2.2M 35.8 / 24.9 / 22.0; D = 32, K = 64: 300k 11.2 / 9.1 / 9.3, 600k 14.9 / 12.2 / 10.4.  Smaller blocks (512 x 2, 256 x 4 at 250k) and
// two vectors at a time per eight lanes in the second look are slower.
constexpr int kBoundThreads = 1024;
template <int U>
__global__ __launch_bounds__(kBoundThreads) void k_bounds_step(
    const uint8_t *__restrict__ codes, int64_t N, int M, int m, const float *__restrict__ drift, int K,
    float *__restrict__ bu, float *__restrict__ bl, uint32_t *__restrict__ list, unsigned *__restrict__ count,
    const float *__restrict__ xp, int D, const float *__restrict__ Cm)
{
    constexpr int SPAN = kBoundThreads * U;
    extern __shared__ float4 smem4[];
    float *vrow = reinterpret_cast<float *>(smem4);
    __shared__ uint32_t found[SPAN], kept[SPAN];
    __shared__ float sdrift[256];
    __shared__ unsigned nfound, nkept, base;
    __shared__ float s_vnorm[kVolatile], s_top[kVolatile + 1];
    __shared__ int s_tk[kVolatile + 1];
    if (threadIdx.x < 256) sdrift[threadIdx.x] = (int)threadIdx.x < K ? drift[threadIdx.x] : 0.f;
    if (threadIdx.x == 0) { nfound = 0u; nkept = 0u; }
    const int64_t n0 = (int64_t)blockIdx.x * SPAN;
    int c[U];
    float u[U], l[U];
#pragma unroll
    for (int j = 0; j < U; ++j) {                                   // all loads first: in flight during the ranking
        const int64_t n = n0 + j * kBoundThreads + threadIdx.x;
        const int64_t nn = n < N ? n : N - 1;
        c[j] = codes[nn * M + m];
        u[j] = bu[nn];
        l[j] = bl[nn];
    }
    __syncthreads();
    top_drifts(sdrift, K, s_top, s_tk);
    const float d1 = s_top[0], d2 = s_top[1], drest = s_top[kVolatile];
    const int k1 = s_tk[0];
    // The second look can only settle a vector whose upper bound stays below its lower bound aged by the drift
    // of the rest: the others are kept without it (found: worth the second look; kept: to recompute).
    const bool outlier = K > kVolatile + 1 && d1 > 3.0f * drest;
    {
#pragma unroll
        for (int j = 0; j < U; ++j) {
            const int64_t n = n0 + j * kBoundThreads + threadIdx.x;
            if (n < N) {
                const float un = (u[j] + sdrift[c[j]]) * 1.000001f;  // rounded up
                const float ln = (l[j] - ((c[j] == k1) ? d2 : d1)) * 0.999999f;   // rounded down while positive
                if (un < ln) {
                    bu[n] = un;
                    bl[n] = ln;
                } else if (outlier && un < (l[j] - drest) * 0.999999f) {
                    found[atomicAdd(&nfound, 1u)] = (uint32_t)n;      // its bounds stay as they were
                } else {
                    kept[atomicAdd(&nkept, 1u)] = (uint32_t)n;        // likewise
                }
            }
        }
    }
    __syncthreads();
    const unsigned nf = nfound;
    // worth a gather of those rows of x'?
    const bool apart = nf * 8u > (unsigned)SPAN;
    if (!apart) {
        const unsigned nk0 = nkept;
        if (threadIdx.x == 0 && nf + nk0) base = atomicAdd(count, nf + nk0);
        __syncthreads();
        for (unsigned i = threadIdx.x; i < nk0; i += kBoundThreads) list[base + i] = kept[i];
        for (unsigned i = threadIdx.x; i < nf; i += kBoundThreads) list[base + nk0 + i] = found[i];
        return;
    }
    for (int e = threadIdx.x; e < kVolatile * D; e += kBoundThreads) {
        const int j = e / D;
        vrow[e] = s_tk[j] >= 0 ? Cm[(size_t)s_tk[j] * D + (e - j * D)] : 0.f;
    }
    __syncthreads();
    {
        static_assert(kBoundThreads / kWave >= kVolatile, "a wave per row");
        const int w = threadIdx.x >> 6;                             // the first kVolatile waves, one row each
        if (w < kVolatile) {
            double q = 0.0;
            for (int d = lane_id(); d < D; d += kWave) q += (double)vrow[w * D + d] * (double)vrow[w * D + d];
            q = wave_sum(q);
            if (lane_id() == 0) s_vnorm[w] = (float)q;
        }
    }
    __syncthreads();
    const int sub = threadIdx.x & 7;
    const int d4n = D >> 2;
    // fp32 rounding of ||x'||^2 - 2 x'.c + ||c||^2 (D/8 chained fmas per lane, three shuffle adds, the final
    // sums) as a fraction of ||x'||^2 + 2|x'.c| + ||c||^2
    const float slack = (float)(D / 8 + 8) * 1.2e-7f;
    for (unsigned i0 = 0; i0 < nf; i0 += kBoundThreads / 8) {
        const unsigned e = i0 + (threadIdx.x >> 3);
        const bool ok = e < nf;
        const int64_t n = found[ok ? e : nf - 1];
        const float4 *row = reinterpret_cast<const float4 *>(xp + n * D);
        float x2 = 0.f, dot[kVolatile];
#pragma unroll
        for (int j = 0; j < kVolatile; ++j) dot[j] = 0.f;
#pragma unroll 4
        for (int q = sub; q < d4n; q += 8) {
            const float4 x = row[q];
            x2 = fmaf(x.x, x.x, fmaf(x.y, x.y, fmaf(x.z, x.z, fmaf(x.w, x.w, x2))));
#pragma unroll
            for (int j = 0; j < kVolatile; ++j) {
                const float4 c = *reinterpret_cast<const float4 *>(vrow + j * D + 4 * q);
                dot[j] = fmaf(x.x, c.x, fmaf(x.y, c.y, fmaf(x.z, c.z, fmaf(x.w, c.w, dot[j]))));
            }
        }
#pragma unroll
        for (int o = 1; o < 8; o <<= 1) {
            x2 += __shfl_xor(x2, o, kWave);
#pragma unroll
            for (int j = 0; j < kVolatile; ++j) dot[j] += __shfl_xor(dot[j], o, kWave);
        }
        if (ok && sub == 0) {
            const int c = codes[n * M + m];
            const float u = (bu[n] + sdrift[c]) * 1.000001f;
            float l = (bl[n] - drest) * 0.999999f;                   // the rest moved by at most drest
#pragma unroll
            for (int j = 0; j < kVolatile; ++j) {
                if (s_tk[j] >= 0 && s_tk[j] != c) {
                    const float mag = x2 + 2.f * fabsf(dot[j]) + s_vnorm[j];
                    const float dj2 = (x2 - 2.f * dot[j] + s_vnorm[j]) - slack * mag;
                    l = fminf(l, sqrtf(fmaxf(dj2, 0.f)) * 0.999999f);
                }
            }
            if (u < l) {
                bu[n] = u;
                bl[n] = l;
            } else {
                kept[atomicAdd(&nkept, 1u)] = (uint32_t)n;
            }
        }
    }
    __syncthreads();
    const unsigned nk = nkept;
    if (threadIdx.x == 0 && nk) base = atomicAdd(count, nk);
    __syncthreads();
    for (unsigned i = threadIdx.x; i < nk; i += kBoundThreads) list[base + i] = kept[i];
}

constexpr int kBoundSpan = 4096;                     // of k_bounds_carry

// ---- Distance bounds carried from one sweep to the next (several sweeps in one call, plain Lloyd cool-down) ----
// When a sweep comes back to stage m, C_m and column m of the codes are as the stage's last visit left them
// (Sec. 3.1: a stage changes its own dictionary and code only); x' alone has moved, in exact arithmetic by
//   x'_new - x'_old = - sum over the stages j visited in between of d_j,   d_j = c_j,new(i_j,new) - c_j,old(i_j,old),
// the change of stage j's part of the reconstruction.  The bounds the last visit ended with therefore still hold
// once the upper one has grown and the lower one has shrunk by delta >= ||x'_new - x'_old||, and a vector they still
// settle keeps its code without being assigned again.  delta is taken per vector as the sum of ||d_j|| (triangle
// inequality), read from a K x K table per stage, plus a bound on the fp32 roundings of the passes in between:
// 2M results of magnitude <= 2A per coordinate (A = largest |x'| or |codeword| coordinate seen), each off by at
// most 2^-24 of itself, i.e. at most 3M 2^-24 sqrt(D) A in norm; (8M + 16) 2^-24 sqrt(D) A is used.

// T[a][b] = ||C_now[b] - C_entry[a]||, rounded up: how far the reconstruction part of a vector moved whose code went
// from a (dictionary as the stage found it) to b (as it leaves it).  One block per a; dynamic LDS: D floats.
__global__ __launch_bounds__(256) void k_pair_table(
    const float *__restrict__ Centry, const float *__restrict__ Cm, int K, int D, float *__restrict__ T)
{
    extern __shared__ float4 smem4[];
    const int a = blockIdx.x;
    const int d4 = D >> 2;
    for (int d = threadIdx.x; d < d4; d += 256) smem4[d] = reinterpret_cast<const float4 *>(Centry + (size_t)a * D)[d];
    __syncthreads();
    // a thread per b: its row of the dictionary against the row in LDS (every lane reads the same LDS address)
    for (int b = threadIdx.x; b < K; b += 256) {
        const float4 *cb = reinterpret_cast<const float4 *>(Cm + (size_t)b * D);
        double s0 = 0.0, s1 = 0.0;
#pragma unroll 4
        for (int d = 0; d < d4; ++d) {
            const float4 x = cb[d], y = smem4[d];
            const double t0 = (double)x.x - (double)y.x, t1 = (double)x.y - (double)y.y;
            const double t2 = (double)x.z - (double)y.z, t3 = (double)x.w - (double)y.w;
            s0 += t0 * t0 + t2 * t2;
            s1 += t1 * t1 + t3 * t3;
        }
        T[(size_t)a * K + b] = (float)(sqrt(s0 + s1) * 1.000001);
    }
}

// End of stage m: path[n] += T[code at entry][code now]; snap[n] = path[n] (the stage's mark on the running path
// length: when it is visited again, path - snap is the sum of ||d_j|| over the stages in between).  Also folds the
// stage's max |x'| (refine_count[1]) into the running maximum.
__global__ __launch_bounds__(256) void k_path_step(
    const uint8_t *__restrict__ entry, const uint8_t *__restrict__ codes, int64_t N, int M, int m,
    const float *__restrict__ T, int K, double *__restrict__ path, double *__restrict__ snap,
    unsigned *__restrict__ refine_count, unsigned *__restrict__ amax_run)
{
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        const unsigned a = refine_count[1];
        if (a > *amax_run) *amax_run = a;
    }
    for (int64_t n = (int64_t)blockIdx.x * 256 + threadIdx.x; n < N; n += (int64_t)gridDim.x * 256) {
        const double s = path[n] + (double)T[(size_t)entry[n] * K + codes[n * M + m]];
        path[n] = s;
        snap[n] = s;
    }
}

// Entry of a stage whose bounds were kept: widen them by delta and list the vectors they no longer settle
// (*count must be zero on entry; order is free), as k_bounds_step does after a centroid update.
__global__ __launch_bounds__(kBoundThreads) void k_bounds_carry(
    const double *__restrict__ path, const double *__restrict__ snap, int64_t N, double slack_unit,
    const unsigned *__restrict__ amax_run, const unsigned *__restrict__ amax_now,
    float *__restrict__ bu, float *__restrict__ bl, uint32_t *__restrict__ list, unsigned *__restrict__ count)
{
    __shared__ uint32_t kept[kBoundSpan];
    __shared__ unsigned nkept, base;
    if (threadIdx.x == 0) nkept = 0u;
    __syncthreads();
    const unsigned abits = max(*amax_run, *amax_now);
    const double slack = slack_unit * (double)__uint_as_float(abits);
    const int64_t n0 = (int64_t)blockIdx.x * kBoundSpan;
    constexpr int U = kBoundSpan / kBoundThreads;
#pragma unroll
    for (int j = 0; j < U; ++j) {
        const int64_t n = n0 + j * kBoundThreads + threadIdx.x;
        if (n < N) {
            const double delta = (path[n] - snap[n]) * (1.0 + 1e-9) + slack;
            const float un = (float)((double)bu[n] + delta) * 1.000001f;    // rounded up
            const float ln = (float)((double)bl[n] - delta) * 0.999999f;    // rounded down while positive
            if (un < ln) {
                bu[n] = un;
                bl[n] = ln;
            } else {
                kept[atomicAdd(&nkept, 1u)] = (uint32_t)n;                  // its bounds stay; the assignment renews them
            }
        }
    }
    __syncthreads();
    const unsigned nk = nkept;
    if (threadIdx.x == 0 && nk) base = atomicAdd(count, nk);
    __syncthreads();
    for (unsigned i = threadIdx.x; i < nk; i += kBoundThreads) list[base + i] = kept[i];
}

__global__ void k_zero_words(unsigned *__restrict__ p, int n)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = 0u;
}

}  // namespace hclae
