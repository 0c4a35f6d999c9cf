// Greedy encoding (Sec. 3.3, Eq. 3 with one path) of dictionaries that fit fp16 operand registers, in one kernel: a block
// takes 32 vectors through ALL M dictionaries, the residual rows staying in registers in between.
//
// Dictionary by dictionary the greedy encoder launches 3 M kernels and reads and writes every row M times; a few thousand
// vectors pay for nothing but launches that way (D = 128, M = 8: 158 us for 64 vectors, 202 us for 10k).  Here a row is read
// and written once, and the two launches are k_encode_prep, which lays out the fp16 dictionaries, and k_encode_fused: 51 us
// and 90 us.  What bounds it is the chain of a dictionary's steps (round, contract, decide, subtract, with two or four
// barriers): about 4.5 us each, eight waves waiting for each other, which is why large calls do not come here
// (encoder(); k_encode_wave takes most of them).
//
// Wave b of the block keeps codewords 32 b .. 32 b + 31 of the running dictionary as MFMA operands in registers (its next
// operands travel while the vectors are decided); the 32 rows are rounded to fp16 once by all threads and shared through
// LDS.  Scores, bounds and decisions are those of k_assign_half (assign_half.hpp), so the codes are the same fp64 direct-form
// decisions and the residuals the same fp32 subtractions as dictionary by dictionary.
#pragma once
#include "assign_half.hpp"

namespace hclae {

constexpr int kPrepThreads = 1024;
constexpr int kEncodeConsts = 8;                    // floats per dictionary: scale, h, rho, acc, hx, cmax

// Tiles of N < 2^31 vectors, and the blocks that take them: one each up to 2^20, which stride beyond (a launch holds less than
// 2^32 threads, and a block has up to 512).
__host__ __device__ constexpr int64_t encode_tiles(int64_t N) { return (N + kTileVec - 1) / kTileVec; }
__host__ __device__ constexpr int64_t encode_blocks(int64_t N) { return encode_tiles(N) < (1 << 20) ? encode_tiles(N) : (1 << 20); }

// One block per dictionary: fp16 image in the order of half_slot, k-step by k-step; -||C||^2/2 and w per codeword; -mu; the
// constants (half_constants has the reasons).  Also clears the counters of undecided vectors and of tiles given up (k_encode_wave).
// NORMS: a second block per dictionary leaves -||c||^2/2 of the codewords as they are, from 64-bit sums (-inf beyond K), for scores from
// the fp32 matrix cores; within the other blocks the same sums cost small calls, which never ask for such scores, 1 %.
template <bool NORMS>
__global__ __launch_bounds__(kPrepThreads) void k_encode_prep(
    const float *__restrict__ C, int K, int D, int kb, int NC, char *__restrict__ img, float *__restrict__ hn,
    float *__restrict__ wtab, float *__restrict__ negmu, float *__restrict__ consts, float *__restrict__ hneg,
    unsigned *__restrict__ refine_count)
{
    __shared__ float s_sq[256], s_dsq[256], s_red[2][kPrepThreads / kWave];
    constexpr int waves = kPrepThreads / kWave;
    const int M = NORMS ? gridDim.x / 2 : gridDim.x, m = NORMS && (int)blockIdx.x >= M ? blockIdx.x - M : blockIdx.x;
    const int lane = lane_id(), wave = threadIdx.x >> 6;
    const int kpad = 32 * kb;
    const float *Cm = C + (size_t)m * K * D;
    if (NORMS && (int)blockIdx.x >= M) {
        for (int row = wave; row < kpad; row += waves) {
            const float4 v = load_row_piece(Cm, row, 4 * lane, K, D, D);
            const double s = wave_sum((double)v.x * v.x + (double)v.y * v.y + (double)v.z * v.z + (double)v.w * v.w);
            if (lane == 0) hneg[(size_t)m * kpad + row] = row < K ? -(float)(0.5 * s) : -__builtin_inff();
        }
        return;
    }
    img += (size_t)m * NC * kb * 4096;
    if (m == 0 && threadIdx.x == 0) refine_count[0] = refine_count[2] = refine_count[3] = 0u;
    // a lane keeps its float4 column (NC <= 4), a wave takes rows wave, wave + 16, ..., eight of them in flight
    constexpr int U = 8;
    const int p = lane;
    const bool live = p < 16 * NC;
    float4 mu = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
    for (int i = 0; i < kMuRows; ++i) {
        const float4 w = load_row_piece(Cm, (int)((unsigned)(i * K) / kMuRows), 4 * p, K, D, D);
        mu.x += w.x;
        mu.y += w.y;
        mu.z += w.z;
        mu.w += w.w;
    }
    // the largest norm sets the scale (see half_shift)
    float big = 0.f;
    for (int r0 = wave; r0 < K; r0 += U * waves) {
        float s[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const float4 v = load_row_piece(Cm, r0 + u * waves, 4 * p, K, D, D);
            s[u] = v.x * v.x + v.y * v.y + v.z * v.z + v.w * v.w;
        }
        big = fmaxf(big, group_sums<U, 64>(s));
    }
#pragma unroll
    for (int o = 1; o < U; o <<= 1) big = fmaxf(big, __shfl_xor(big, o, kWave));
    if (lane == 0) s_red[0][wave] = big;
    __syncthreads();
    for (int i = 0; i < waves; ++i) big = fmaxf(big, s_red[0][i]);
    const float scale = ldexpf(1.f, half_exponent(0.5f * big));
    const float f = -scale / kMuRows;
    const float4 neg = make_float4(mu.x * f, mu.y * f, mu.z * f, mu.w * f);
    if (wave == 0 && live) reinterpret_cast<float4 *>(negmu + (size_t)m * kChunkD * NC)[p] = neg;
    for (int r0 = wave; r0 < kpad; r0 += U * waves) {
        float4 v[U];
        float s[2 * U];
#pragma unroll
        for (int u = 0; u < U; ++u) v[u] = load_row_piece(Cm, r0 + u * waves, 4 * p, K, D, D);
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int row = r0 + u * waves;
            float4 w = scaled(v[u], scale, neg);
            if (row >= K || !live) w = make_float4(0.f, 0.f, 0.f, 0.f);
            s[2 * u] = s[2 * u + 1] = 0.f;
            const halfx4 q = half4(w, s[2 * u], s[2 * u + 1]);
            const int t = p >> 2, g = p & 1, hi = (p >> 1) & 1;
            if (live && row < kpad)
                *reinterpret_cast<halfx4 *>(img + (size_t)(t * kb + (row >> 5)) * 1024 + half_slot(t, g, row & 31) + 8 * hi) = q;
        }
        const float mine = group_sums<2 * U, 64>(s);                // lane i: value i
        const int row = r0 + (lane >> 1) * waves;
        if (lane < 2 * U && row < kpad) ((lane & 1) ? s_dsq : s_sq)[row] = mine;
    }
    __syncthreads();
    float hm = 0.f;
    for (int k = lane; k < kpad; k += kWave) hm = fmaxf(hm, s_sq[k]);
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) hm = fmaxf(hm, __shfl_xor(hm, o, kWave));
    const float cmax = sqrtf(hm) * 1.001f;
    float rho = 0.f;
    for (int k = threadIdx.x; k < kpad; k += kPrepThreads) {
        const float wk = half_floor(s_sq[k], cmax);
        rho = half_rho(s_dsq[k], wk, cmax);
        hn[(size_t)m * kpad + k] = k < K ? -0.5f * s_sq[k] : -1e38f;
        wtab[(size_t)m * kpad + k] = k < K ? (float)half_up(wk) : 0.f;
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) rho = fmaxf(rho, __shfl_xor(rho, o, kWave));
    if (lane == 0) s_red[1][wave] = rho;
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int i = 0; i < waves; ++i) rho = fmaxf(rho, s_red[1][i]);
        float *c = consts + (size_t)m * kEncodeConsts;
        c[0] = scale;
        c[2] = rho;
        c[3] = half_acc(NC);
        c[1] = half_loss(c[3], hm, cmax);
        c[4] = half_loss_x(c[3], cmax);
        c[5] = cmax;
    }
}

// The j-th candidate (bit i of mask[b]: codeword 32 b + i), -1 beyond the last.
template <int KB>
__device__ __forceinline__ int nth_candidate(const unsigned *mask, int j)
{
    int k = -1;
    for (int w = 0; w < KB; ++w) {
        unsigned q = mask[w];
        const int c = __popc(q);
        if (j >= 0 && j < c) {
            for (int i = 0; i < j; ++i) q &= q - 1u;
            k = 32 * w + __ffs(q) - 1;
        }
        j -= c;
    }
    return k;
}

// The nearest of a vector's candidates in fp64, by one wave, a lane per candidate; row: its fp32 residual in LDS.
template <int KB>
__device__ __forceinline__ int encode_decide_fp64(const float *__restrict__ row, const float *__restrict__ Cm, const unsigned *mask, int D, int lane)
{
    const int d4 = D >> 2;
    int total = 0;
    for (int b = 0; b < KB; ++b) total += __popc(mask[b]);
    double dbest = __builtin_inf();
    int k64 = 0x7fffffff;
    for (int j0 = 0; j0 < total; j0 += kWave) {
        const int k = nth_candidate<KB>(mask, j0 + lane);
        if (k < 0) continue;
        const float4 *c4 = reinterpret_cast<const float4 *>(Cm + (size_t)k * D);
        double s = 0.0;
#pragma unroll 2
        for (int d = 0; d < d4; ++d) {
            const float4 u = reinterpret_cast<const float4 *>(row)[d], v = c4[d];
            const double t0 = (double)u.x - (double)v.x, t1 = (double)u.y - (double)v.y;
            const double t2 = (double)u.z - (double)v.z, t3 = (double)u.w - (double)v.w;
            s += t0 * t0;
            s += t1 * t1;
            s += t2 * t2;
            s += t3 * t3;
        }
        if (s < dbest || (s == dbest && k < k64)) { dbest = s; k64 = k; }
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        const double os = __shfl_xor(dbest, o, kWave);
        const int ok = __shfl_xor(k64, o, kWave);
        if (os < dbest || (os == dbest && ok < k64)) { dbest = os; k64 = ok; }
    }
    return k64 == 0x7fffffff ? 0 : k64;
}

// The nearest of a vector's candidates (bit i of mask[b]: codeword 32 b + i), by one wave; row: its fp32 residual in LDS.
// As decide_items: fp32 direct form where the two best are further apart than its error, then fp64 in ascending dimension
// order, lowest index on exact ties.
// Four candidates at a time: bound by the latency of a round, so sixteen lanes (two loads each at D = 128) take one rather than
// a half wave (two at a time: vectors with many candidates pay twice the rounds; 10k rows with lognormal norms, D = 64, K = 64,
// M = 4: 143 us, 224 with a half wave, 64 queries at D = 128 49.4 / 51.5) or eight lanes (115 us, but registers spill at
// D = 256, K = 128: 920 us for 200k rows instead of 775).
template <int KB>
__device__ __forceinline__ int encode_decide(const float *__restrict__ row, const float *__restrict__ Cm, const unsigned *mask, int D, int lane)
{
    const int d4 = D >> 2;
    // fp32: four candidates at a time, sixteen lanes each
    const int sub = lane & 15;
    const float eta = (float)(4 * ((d4 + 15) >> 4) + 8) * 6.1e-8f;
    float best = __builtin_inff(), second = __builtin_inff();
    int kbest = 0, total = 0;
    for (int b = 0; b < KB; ++b) total += __popc(mask[b]);
    for (int j0 = 0; j0 < total; j0 += 4) {
        const int k = nth_candidate<KB>(mask, j0 + (lane >> 4));
        const float4 *c4 = reinterpret_cast<const float4 *>(Cm + (size_t)(k < 0 ? 0 : k) * D);
        float s = 0.f;
#pragma unroll 2
        for (int d = sub; d < d4; d += 16) {
            const float4 u = reinterpret_cast<const float4 *>(row)[d], v = c4[d];
            const float e0 = u.x - v.x, e1 = u.y - v.y, e2 = u.z - v.z, e3 = u.w - v.w;
            s = fmaf(e3, e3, fmaf(e2, e2, fmaf(e1, e1, fmaf(e0, e0, s))));
        }
#pragma unroll
        for (int o = 1; o < 16; o <<= 1) s += __shfl_xor(s, o, kWave);
        if (k < 0) s = __builtin_inff();
        second = s < best ? best : fminf(second, s);
        if (s < best) { best = s; kbest = k; }
    }
#pragma unroll
    for (int o = 16; o < kWave; o <<= 1) {
        const float ob = __shfl_xor(best, o, kWave), os = __shfl_xor(second, o, kWave);
        const int ok = __shfl_xor(kbest, o, kWave);
        second = fminf(fmaxf(best, ob), fminf(second, os));
        if (ob < best) { best = ob; kbest = ok; }
    }
    if (best * (1.f + eta) < second * (1.f - eta) && second > 1e-25f) return kbest;
    return encode_decide_fp64<KB>(row, Cm, mask, D, lane);
}
// LDS of k_encode_fused.
struct EncodeLds {
    int rows16, rows32, best, w, rsq, mask, code, misc, total;      // byte offsets
};
__host__ __device__ constexpr EncodeLds encode_lds(int kb, int nc)
{
    EncodeLds l = {};
    l.rows16 = 0;                                                   // 32 rows of 64 nc halves, operand order
    l.rows32 = l.rows16 + 4096 * nc;                                // 32 rows of 64 nc floats: the undecided ones
    l.best = l.rows32 + 8192 * nc;                                  // [kb][32] {best key, second key, code}
    l.w = l.best + kb * 32 * 16;                                    // [32 kb]
    l.rsq = l.w + 32 * kb * 4;                                      // [32][2] ||X||^2, ||X - X^||^2
    l.mask = l.rsq + 256;                                           // [32][kb] candidates of block b, bit 8 (v / 4) + 4 h + v % 4
    l.code = l.mask + 32 * kb * 4;                                  // [32]
    l.misc = l.code + 128;
    l.total = l.misc + 64;
    return l;
}

// NC: 64-dim chunks, 1, 2 or 4 (a row length between rounds up).  A block is KB waves.
template <int KB, int NC>
__global__ __launch_bounds__(64 * KB, 2) void k_encode_fused(
    const float *__restrict__ X, const float *__restrict__ C, int N, int D, int K, int M,
    const char *__restrict__ img, const float *__restrict__ hn, const float *__restrict__ wtab, const float *__restrict__ negmu,
    const float *__restrict__ consts, uint8_t *__restrict__ codes, float *__restrict__ residue,
    unsigned *__restrict__ refine_count, unsigned long long *__restrict__ work)
{
    extern __shared__ float4 smem4[];
    char *lds = reinterpret_cast<char *>(smem4);
    constexpr EncodeLds L = encode_lds(KB, NC);
    constexpr int COLS = 16 * NC;                                   // float4 columns of a padded row: that many lanes share a row
    constexpr int RSTEP = 64 * KB / COLS;                           // rows the block covers at a time
    constexpr int R = 32 / RSTEP;                                   // rows (one float4 each) per thread
    constexpr int T = 4 * NC;                                       // 16-dim steps
    const int lane = lane_id(), wave = threadIdx.x >> 6, h = lane >> 5, r = lane & 31;
    const int p = threadIdx.x % COLS, row0 = threadIdx.x / COLS;
    const bool col_live = 4 * p < D;
    float4 *best = reinterpret_cast<float4 *>(lds + L.best);
    float *lds_w = reinterpret_cast<float *>(lds + L.w);
    float *rsq = reinterpret_cast<float *>(lds + L.rsq);
    unsigned *masks = reinterpret_cast<unsigned *>(lds + L.mask);
    unsigned *final_code = reinterpret_cast<unsigned *>(lds + L.code);
    unsigned rechecked = 0u, rechecked_last = 0u;                   // counted by wave 0

    uint4 a[T];                                                     // this wave's codewords of the running dictionary
    float4 hn4[4];
    float wl;
    float4 mu;
    auto fetch = [&](int m) {
        const char *src = img + ((size_t)m * T * KB + wave) * 1024 ;
#pragma unroll
        for (int t = 0; t < T; ++t) a[t] = *reinterpret_cast<const uint4 *>(src + (size_t)t * KB * 1024 + half_slot(t, h, r));
        const float *q = hn + (size_t)m * 32 * KB + 32 * wave;
#pragma unroll
        for (int g = 0; g < 4; ++g) hn4[g] = *reinterpret_cast<const float4 *>(q + 8 * g + 4 * h);
        wl = wtab[(size_t)m * 32 * KB + 32 * wave + r];
        mu = reinterpret_cast<const float4 *>(negmu + (size_t)m * kChunkD * NC)[p];
    };
    const int ntiles = (int)encode_tiles(N);
    fetch(0);
    for (int tile = blockIdx.x; tile < ntiles; tile += gridDim.x) {
        const int n0 = tile * kTileVec;
        float4 x[R];
#pragma unroll
        for (int i = 0; i < R; ++i) {
            const int n = min(n0 + row0 + i * RSTEP, N - 1);        // the ragged tail re-reads the last row
            x[i] = make_float4(0.f, 0.f, 0.f, 0.f);
            if (col_live) x[i] = *reinterpret_cast<const float4 *>(X + (size_t)n * D + 4 * p);
        }
        for (int m = 0; m < M; ++m) {
            const float *cc = consts + (size_t)m * kEncodeConsts;
            HalfConsts c;
            c.scale = cc[0];
            c.h = cc[1];
            c.rho = cc[2];
            c.acc = cc[3];
            c.hx = cc[4];
            // ---- the rows as fp16 operands, with their norms
            const int t16 = p >> 2, g16 = p & 1, hi = (p >> 1) & 1;
            float s[2 * R];
#pragma unroll
            for (int i = 0; i < R; ++i) {
                const int row = row0 + i * RSTEP;
                s[2 * i] = s[2 * i + 1] = 0.f;
                const halfx4 q = half4(scaled(x[i], c.scale, mu), s[2 * i], s[2 * i + 1]);
                *reinterpret_cast<halfx4 *>(lds + L.rows16 + t16 * 1024 + half_slot(t16, g16, row) + 8 * hi) = q;
            }
            const float mine = group_sums<2 * R, COLS>(s);          // lane i of a row's lanes: value i
            if (p < 2 * R) rsq[2 * (row0 + (p >> 1) * RSTEP) + (p & 1)] = mine;
            __syncthreads();
            // ---- scores of this wave's 32 codewords
            floatx16 acc;
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                acc[4 * g] = hn4[g].x;
                acc[4 * g + 1] = hn4[g].y;
                acc[4 * g + 2] = hn4[g].z;
                acc[4 * g + 3] = hn4[g].w;
            }
#pragma unroll
            for (int t = 0; t < T; ++t) {
                const halfx8 bfrag = *reinterpret_cast<const halfx8 *>(lds + L.rows16 + t * 1024 + half_slot(t, h, r));
                acc = __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(halfx8, a[t]), bfrag, acc, 0, 0, 0);
            }
            const float x2 = rsq[2 * r];
            const float xn = sqrtf(x2) * 1.001f;
            const float e = half_bound(x2, rsq[2 * r + 1], xn, c);
            {
                const halfx4 aw = {h == 0 ? (_Float16)wl : (_Float16)0.f, (_Float16)0.f, (_Float16)0.f, (_Float16)0.f};
                const halfx4 bw = {(_Float16)e, (_Float16)0.f, (_Float16)0.f, (_Float16)0.f};
                acc = __builtin_amdgcn_mfma_f32_32x32x8f16(aw, bw, acc, 0, 0, 0);
            }
            if (h == 0) lds_w[32 * wave + r] = wl;
            fetch(m + 1 < M ? m + 1 : 0);                           // the next dictionary's operands travel from here on
            {
                const float inf = opaque(__builtin_inff());
                float mx = -__builtin_inff(), m2 = -__builtin_inff();
#pragma unroll
                for (int v = 0; v < 16; ++v) {
                    const float key = __uint_as_float((__float_as_uint(acc[v]) & ~15u) | (unsigned)v);
                    m2 = __builtin_amdgcn_fmed3f(mx, m2, key);
                    mx = __builtin_amdgcn_fmed3f(mx, key, inf);
                }
                const int v = (int)(__float_as_uint(mx) & 15u);
                int code = 32 * wave + 8 * (v >> 2) + 4 * h + (v & 3);
                const float mxo = __shfl_xor(mx, 32, kWave), m2o = __shfl_xor(m2, 32, kWave);
                const int co = __shfl_xor(code, 32, kWave);
                m2 = fmaxf(fminf(mx, mxo), fmaxf(m2, m2o));
                if (mxo > mx) code = co;
                mx = fmaxf(mx, mxo);
                if (h == 0) best[32 * wave + r] = make_float4(mx, m2, __int_as_float(code), 0.f);
            }
            __syncthreads();
            // ---- best and second best over all codewords, the same in every wave
            float mx = -__builtin_inff(), m2 = -__builtin_inff();
            int code = 0;
#pragma unroll
            for (int b = 0; b < KB; ++b) {
                const float4 o = best[32 * b + r];
                m2 = fmaxf(fminf(mx, o.x), fmaxf(m2, o.y));
                if (o.x > mx) code = __float_as_int(o.z);
                mx = fmaxf(mx, o.x);
            }
            code = code < K ? code : 0;
            const float hh = fmaf(c.hx, xn, fmaf(2.1e-6f, fabsf(mx), c.h)) + 1e-36f;
            const float thr = mx - 2.f * e * lds_w[code] - 2.f * hh;
            const bool big = !(x2 < kHalfMaxNorm * kHalfMaxNorm && fabsf(thr) < 1e37f);
            const bool amb = K > 1 && n0 + r < N && (big || !(m2 < thr));
            unsigned who = (unsigned)__ballot(amb);                 // low half: vector r; the same in every wave
            if (who) {
                // ---- candidates of the undecided vectors, their rows in fp32, and the decision: a wave per vector
                unsigned bits = 0u;
#pragma unroll
                for (int v = 0; v < 16; ++v) bits |= acc[v] >= thr || big ? 1u << (8 * (v >> 2) + 4 * h + (v & 3)) : 0u;
                bits |= (unsigned)__shfl_xor((int)bits, 32, kWave);
                const int left = K - 32 * wave;
                if (left < 32) bits &= left > 0 ? (1u << left) - 1u : 0u;
                if (h == 0) masks[r * KB + wave] = bits;
                if (wave == 0 && h == 0) final_code[r] = (unsigned)code;
#pragma unroll
                for (int i = 0; i < R; ++i) {
                    const int row = row0 + i * RSTEP;
                    if ((who >> row) & 1u) reinterpret_cast<float4 *>(lds + L.rows32)[row * COLS + p] = x[i];
                }
                __syncthreads();
                const float *Cm = C + (size_t)m * K * D;
                unsigned mine = who;
                for (int skip = wave; mine; ) {                     // wave w takes the w-th, (w + KB)-th, ... undecided vector
                    for (; skip > 0 && mine; --skip) mine &= mine - 1u;
                    if (!mine) break;
                    const int v = __ffs(mine) - 1;
                    mine &= mine - 1u;
                    skip = KB - 1;
                    const int k = encode_decide<KB>(reinterpret_cast<const float *>(lds + L.rows32) + v * 4 * COLS, Cm, masks + v * KB, D, lane);
                    if (lane == 0) final_code[v] = (unsigned)k;
                }
                if (wave == 0) {
                    rechecked += (unsigned)__popc(who);
                    if (m == M - 1) rechecked_last += (unsigned)__popc(who);
                }
                __syncthreads();
                code = (int)final_code[r];
            }
            // ---- codes, and the residual rows
            if (wave == 0 && h == 0 && n0 + r < N) codes[(size_t)(n0 + r) * M + m] = (uint8_t)code;
#pragma unroll
            for (int i = 0; i < R; ++i) {
                const int k = __shfl(code, row0 + i * RSTEP, kWave);
                if (col_live) {
                    const float4 q = *reinterpret_cast<const float4 *>(C + ((size_t)m * K + k) * D + 4 * p);
                    x[i] = make_float4(x[i].x - q.x, x[i].y - q.y, x[i].z - q.z, x[i].w - q.w);
                }
            }
        }
#pragma unroll
        for (int i = 0; i < R; ++i) {
            const int n = n0 + row0 + i * RSTEP;
            if (n < N && col_live) *reinterpret_cast<float4 *>(residue + (size_t)n * D + 4 * p) = x[i];
        }
    }
    if (threadIdx.x == 0) {
        if (rechecked_last) atomicAdd(refine_count, rechecked_last);
        if (rechecked) atomicAdd(work + 2, (unsigned long long)rechecked);
        if (blockIdx.x == 0) {
            work[0] += (unsigned long long)M;                       // launches on one stream follow one another
            work[1] += (unsigned long long)M * (unsigned long long)N;
        }
    }
}

}  // namespace hclae
