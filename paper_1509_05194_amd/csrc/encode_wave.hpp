// Greedy encoding (Sec. 3.3, Eq. 3 with one path) of large calls with rows of up to 128 coordinates, in one kernel: a wave takes 32
// vectors through ALL M dictionaries, the residual rows staying in its registers in between.
//
// Dictionary by dictionary a row crosses HBM three times per dictionary (assignment, residue in, residue out), which is what holds
// those kernels (N = 1M, D = 128, M = 8, K = 256: 24 passes of 512 MB).  Here it is read once and written once.  The fp16 dictionaries
// (k_encode_prep) pass through LDS, two of them held: while one is contracted the next travels from L2 into the other by direct
// loads, for all eight waves of the block together, one barrier per dictionary.  An undecided vector is decided at once, by the two
// lanes that hold its row, a candidate a round.  Scores, bounds and decisions are those of k_assign_half (assign_half.hpp), so the codes are the same fp64 direct-form
// decisions and the residuals the same fp32 subtractions as dictionary by dictionary.
//
// Measured (D = 128, M = 8, K = 256, us dictionary by dictionary / here): N = 1M 2451 / 1560, 200k 620 / 424, 49k 317 / 137; D = 64, 100k
// 286 / 140.  Of the 1560, 930 are the arithmetic (MFMAs and VALU in turn, two waves to a SIMD), some 250 the rows to subtract (gathered
// from L2, 16 bytes a lane; through LDS with contiguous reads it is no faster), 230 the dictionaries' way into LDS and the barriers,
// 200 the undecided vectors.  Data whose vectors have many candidates each take the second launch and are up to 1.5 times as
// slow as dictionary by dictionary (N = 200k, M = 2: groups 30 standard deviations apart 384 / 523, lognormal norms 2567 / 3773,
// codewords 1e-4 of the vectors 594 / 762, a dictionary of zeros 8046 / 9820).
#pragma once
#include "encode.hpp"

namespace hclae {

// LDS of k_encode_wave.
struct WaveLds {
    int img, hn, w, mu, rows, masks, total;                         // byte offsets; img, hn, w, mu twice
    int img_size, hn_size, mu_size;
};
__host__ __device__ constexpr WaveLds wave_lds(int kb, int nc)
{
    WaveLds l = {};
    l.img_size = kb * nc * 4096;
    l.hn_size = 32 * kb * 4;
    l.mu_size = 64 * nc * 4;
    l.img = 0;
    l.hn = 2 * l.img_size;
    l.w = l.hn + 2 * l.hn_size;
    l.mu = l.w + 2 * l.hn_size;
    l.rows = l.mu + 2 * l.mu_size;                                  // a row per wave, for the decision in fp64
    l.masks = l.rows + kAssignWaves * 64 * nc * 4;                  // [wave][kb]
    l.total = l.masks + kAssignWaves * kb * 4;
    return l;
}

// 16 bytes per lane from global memory into LDS without passing through registers: lane i's to `to` + 16 i.
__device__ __forceinline__ void load_to_lds(const void *from, void *to)
{
    __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void *)from, (__attribute__((address_space(3))) void *)to,
                                     16, 0, 0);
}

// Narrows the candidates mk of the wave's 32 vectors by scores from the fp32 matrix cores, as rescore_items does and with its bound, but
// for rows in registers.  hneg: -||c||^2/2 of the dictionary's codewords, -inf beyond K.
template <int KB, int S>
__device__ __forceinline__ void rescore_rows(uint32_t (&mk)[4], const float4 (&x)[S], const float *__restrict__ Cm,
                                             const float *__restrict__ hneg, int D, int K, int lane)
{
    const int h = lane >> 5, r = lane & 31;
    float hmax = 0.f;
    for (int k = lane; k < K; k += kWave) hmax = fmaxf(hmax, -hneg[k]);
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) hmax = fmaxf(hmax, __shfl_xor(hmax, o, kWave));
    floatx16 acc[KB];
    init_acc<KB>(acc, hneg, h);
    float x2 = 0.f;
#pragma unroll
    for (int s = 0; s < S; ++s) {
        float4 a[KB];
#pragma unroll
        for (int b = 0; b < KB; ++b) a[b] = load_row_piece(Cm, 32 * b + r, 8 * s + 4 * h, K, D, D);
        x2 = fmaf(x[s].x, x[s].x, fmaf(x[s].y, x[s].y, fmaf(x[s].z, x[s].z, fmaf(x[s].w, x[s].w, x2))));
#pragma unroll
        for (int b = 0; b < KB; ++b) {
            acc[b] = __builtin_amdgcn_mfma_f32_32x32x2f32(a[b].x, x[s].x, acc[b], 0, 0, 0);
            acc[b] = __builtin_amdgcn_mfma_f32_32x32x2f32(a[b].y, x[s].y, acc[b], 0, 0, 0);
            acc[b] = __builtin_amdgcn_mfma_f32_32x32x2f32(a[b].z, x[s].z, acc[b], 0, 0, 0);
            acc[b] = __builtin_amdgcn_mfma_f32_32x32x2f32(a[b].w, x[s].w, acc[b], 0, 0, 0);
        }
        __builtin_amdgcn_sched_barrier(0);
    }
    x2 += __shfl_xor(x2, 32, kWave);
    float mx = -__builtin_inff();
#pragma unroll
    for (int b = 0; b < KB; ++b)
#pragma unroll
        for (int v = 0; v < 16; ++v) mx = fmaxf(mx, acc[b][v]);
    mx = fmaxf(mx, __shfl_xor(mx, 32, kWave));
    const float eps = 2.02f * (float)(8 * S + 2) * 1.1920929e-7f;
    const float thr = mx - eps * (hmax + sqrtf(x2) * sqrtf(2.f * hmax) * 1.000001f);
    uint32_t now[4];
    reaching<KB>(now, acc, thr);
    if (fabsf(thr) < 1e37f) {                                       // else the sums may have left fp32's range
#pragma unroll
        for (int i = 0; i < 4; ++i) mk[i] &= now[i];
    }
}

// Candidates of a vector from which its tile is scored again in fp32: that takes as long as some twenty rounds of one candidate each.
constexpr unsigned kWaveMany = 20;

// FULL: D == 64 NC.
// MANY: the tiles that the launch before gave up (given[0 .. *given_count)) because a vector had that many candidates, with fp32 scores where
// it has.  An instance of its own, since the registers of those scores cost the ordinary tiles a seventh of their time (1553 ->
// 1768 us for N = 1M; as a call, which puts the rows into memory, 2683); without such tiles the launch is over at once.
template <int KB, int NC, bool FULL, bool MANY>
__global__ __launch_bounds__(kAssignThreads) void k_encode_wave(
    const float *__restrict__ X, const float *__restrict__ C, int N, int D, int K, int M,
    const char *__restrict__ img, const float *__restrict__ hn, const float *__restrict__ wtab, const float *__restrict__ negmu,
    const float *__restrict__ consts, const float *__restrict__ hneg, uint8_t *__restrict__ codes, float *__restrict__ residue,
    unsigned *__restrict__ refine_count, unsigned long long *__restrict__ work, uint32_t *__restrict__ given,
    unsigned *__restrict__ given_count)
{
    extern __shared__ float4 smem4[];
    char *lds = reinterpret_cast<char *>(smem4);
    constexpr WaveLds L = wave_lds(KB, NC);
    constexpr int S = 8 * NC;                                       // float4 pieces of a row per lane
    constexpr int T = 4 * NC;                                       // 16-dim steps
    constexpr int CHUNKS = L.img_size / 1024;                       // kilobytes of an image, one per wave and load
    const int lane = lane_id(), wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), h = lane >> 5, r = lane & 31;
    const float inf = __builtin_inff();
    unsigned rechecked = 0u, rechecked_last = 0u;

    // dictionary m into half b of LDS: asynchronous but for the tables
    auto stage = [&](int m, int b) {
        const char *from = img + (size_t)m * L.img_size + 16 * lane;
        char *to = lds + L.img + b * L.img_size;
#pragma unroll
        for (int i = 0; i < (CHUNKS + kAssignWaves - 1) / kAssignWaves; ++i) {
            const int at = (i * kAssignWaves + wave) * 1024;
            if (CHUNKS % kAssignWaves == 0 || at < L.img_size) load_to_lds(from + at, to + at);
        }
        if ((int)threadIdx.x < 32 * KB) {
            reinterpret_cast<float *>(lds + L.hn + b * L.hn_size)[threadIdx.x] = hn[(size_t)m * 32 * KB + threadIdx.x];
            reinterpret_cast<float *>(lds + L.w + b * L.hn_size)[threadIdx.x] = wtab[(size_t)m * 32 * KB + threadIdx.x];
        }
        if ((int)threadIdx.x < 64 * NC) reinterpret_cast<float *>(lds + L.mu + b * L.mu_size)[threadIdx.x] = negmu[(size_t)m * 64 * NC + threadIdx.x];
    };
    auto landed = [&]() {                                           // what this wave sent for has arrived, and everybody's
        __builtin_amdgcn_s_waitcnt(0x0f70);                         // vmcnt(0)
        __syncthreads();
    };
    auto piece = [&](const float *row, int s) {
        if (FULL || 8 * s + 4 * h < D) return *reinterpret_cast<const float4 *>(row + 8 * s + 4 * h);
        return make_float4(0.f, 0.f, 0.f, 0.f);
    };

    const unsigned ntiles = MANY ? *given_count : ((unsigned)N + kTileVec - 1) / kTileVec;
    const int nbt = (int)((ntiles + kAssignWaves - 1) / kAssignWaves);
    int b = 0;
    if ((int)blockIdx.x < nbt) {
        stage(0, 0);
        landed();
    }
    for (int bt = blockIdx.x; bt < nbt; bt += gridDim.x) {
        unsigned tile = (unsigned)bt * kAssignWaves + wave;
        const bool mine = tile < ntiles;                            // the others keep the block's barriers
        if (MANY) tile = given[mine ? tile : 0];
        const unsigned at = tile * kTileVec + r;
        const bool live = mine && at < (unsigned)N;
        bool given_up = false;
        unsigned open = 0u;
        const size_t n = at < (unsigned)N ? at : N - 1;                         // the ragged tail re-reads the last row
        float4 x[S];
#pragma unroll
        for (int s = 0; s < S; ++s) x[s] = piece(X + n * D, s);
        for (int m = 0; m < M; ++m, b ^= 1) {
            const float *lds_h = reinterpret_cast<const float *>(lds + L.hn + b * L.hn_size);
            const float *lds_w = reinterpret_cast<const float *>(lds + L.w + b * L.hn_size);
            const float4 *mu4 = reinterpret_cast<const float4 *>(lds + L.mu + b * L.mu_size) + h;
            const float *cc = consts + (size_t)m * kEncodeConsts;
            HalfConsts c;
            c.scale = cc[0];
            c.h = cc[1];
            c.rho = cc[2];
            c.acc = cc[3];
            c.hx = cc[4];
            c.cmax = cc[5];
            const bool more = m + 1 < M || bt + (int)gridDim.x < nbt;
            if (more) stage(m + 1 < M ? m + 1 : 0, b ^ 1);
            if (given_up) {
                landed();
                continue;
            }
            floatx16 acc[KB];
            init_acc<KB>(acc, lds_h, h);
            float xsq = 0.f, dsq = 0.f;
            contract_half<KB, T>(acc, lds + L.img + b * L.img_size, h, r, T,
                [&](int t) {
                    const halfx4 lo = half4(scaled(x[2 * t], c.scale, mu4[4 * t]), xsq, dsq);
                    const halfx4 hi = half4(scaled(x[2 * t + 1], c.scale, mu4[4 * t + 2]), xsq, dsq);
                    return __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
                },
                [](int) {});
            float x2, xn, e;
            {
                const uint2 a = both_halves(__float_as_uint(xsq)), d = both_halves(__float_as_uint(dsq));
                x2 = __uint_as_float(a.x) + __uint_as_float(a.y);
                xn = sqrtf(x2) * 1.001f;
                e = half_bound(x2, __uint_as_float(d.x) + __uint_as_float(d.y), xn, c);
            }
            {
                const halfx4 w = {(_Float16)e, (_Float16)0.f, (_Float16)0.f, (_Float16)0.f};
#pragma unroll
                for (int i = 0; i < KB; ++i) {
                    const halfx4 a = {h == 0 ? (_Float16)lds_w[32 * i + r] : (_Float16)0.f, (_Float16)0.f, (_Float16)0.f, (_Float16)0.f};
                    acc[i] = __builtin_amdgcn_mfma_f32_32x32x8f16(a, w, acc[i], 0, 0, 0);
                }
            }
            // the best, the threshold and the candidates: decide_half has the reasons
            float mx = -inf;
            int code = 0;
            {
                int blk = 0;
#pragma unroll
                for (int i = 0; i < KB; ++i) {
                    const float k = block_key(acc[i]);
                    blk = k > mx ? i : blk;
                    mx = __builtin_elementwise_maximum(mx, k);
                }
                const int v = (int)(__float_as_uint(mx) & 15u);
                code = 32 * blk + 8 * (v >> 2) + 4 * h + (v & 3);
                const uint2 s = both_halves(__float_as_uint(mx)), k = both_halves((unsigned)code);
                const float lo = __uint_as_float(s.x), hi = __uint_as_float(s.y);
                mx = __builtin_elementwise_maximum(lo, hi);
                code = (int)(lo >= hi ? k.x : k.y);
                code = code < K ? code : 0;
            }
            const float *Cm = C + (size_t)m * K * D;
            const float hh = fmaf(c.hx, xn, fmaf(4.3e-6f, fabsf(mx), fmaf(4.4e-6f * e, c.cmax, c.h))) + 1e-9f;
            const float thr = mx - 2.f * e * lds_w[code] - 2.f * hh;
            const bool big = !(x2 < kHalfMaxNorm * kHalfMaxNorm && fabsf(thr) < kHalfMaxThr);
            subtract_half<KB>(acc, thr, h);
            uint32_t mk[4];
            not_negative<KB>(mk, acc);
            const uint2 count = both_halves((unsigned)(__popc(mk[0]) + __popc(mk[1]) + __popc(mk[2]) + __popc(mk[3])));
            const bool amb = K > 1 && live && (big || count.x + count.y != 1u);
            landed();                                               // the next dictionary is there, this one is free
            if (big) {
#pragma unroll
                for (int i = 0; i < (KB + 1) / 2; ++i) {
                    uint32_t all = 0u;
#pragma unroll 1
                    for (int p = 0; p < 32; ++p) all |= (64 * i + 8 * (p >> 2) + 4 * h + (p & 3) < K) ? 1u << p : 0u;
                    mk[i] = all;
                }
            }
            if (__ballot(amb && (big || count.x + count.y >= kWaveMany))) {
                if (!MANY) {
                    given_up = true;
                    continue;
                }
                rescore_rows<KB, S>(mk, x, Cm, hneg + (size_t)m * 32 * KB, D, K, lane);
            }
            const unsigned who = (unsigned)__ballot(amb);
            if (who) {
                open += (unsigned)__popc(who);
                if (m == M - 1) rechecked_last += (unsigned)__popc(who);
                auto term = [](float s, const float4 &u, const float4 &q) {
                    const float a = u.x - q.x, g = u.y - q.y, w = u.z - q.z, v = u.w - q.w;
                    return fmaf(v, v, fmaf(w, w, fmaf(g, g, fmaf(a, a, s))));
                };
                auto total = [](float s) {                          // of the two lanes that share the row
                    const uint2 p = both_halves(__float_as_uint(s));
                    return __uint_as_float(p.x) + __uint_as_float(p.y);
                };
                uint32_t left[4];                                   // candidates not yet compared, of the lane's half of the codewords
#pragma unroll
                for (int i = 0; i < 4; ++i) left[i] = amb ? mk[i] : 0u;
                float best = inf, second = inf;
                while (__ballot((left[0] | left[1] | left[2] | left[3]) != 0u)) {
                    // the lane's first candidate; the vector's is the low half's while it has one
                    int i = 0;
                    uint32_t word = left[0];
#pragma unroll
                    for (int j = 1; j < (KB + 1) / 2; ++j)
                        if (!word) { word = left[j]; i = j; }
                    const int p = __ffs(word) - 1;
                    const uint2 k2 = both_halves(word ? (unsigned)(64 * i + 8 * (p >> 2) + 4 * h + (p & 3)) : 256u);
                    const int k = (int)(k2.x < 256u ? k2.x : k2.y);
                    if (word && (h == 0 || k2.x == 256u)) {
#pragma unroll
                        for (int j = 0; j < (KB + 1) / 2; ++j)
                            if (j == i) left[j] &= left[j] - 1u;
                    }
                    const float *row = Cm + (size_t)(k < 256 ? k : 0) * D;
                    float d = 0.f;
#pragma unroll
                    for (int s0 = 0; s0 < S; s0 += 8) {             // eight pieces in flight
                        float4 q[8];
#pragma unroll
                        for (int s = 0; s < 8; ++s) q[s] = piece(row, s0 + s);
#pragma unroll
                        for (int s = 0; s < 8; ++s) d = term(d, x[s0 + s], q[s]);
                        __builtin_amdgcn_sched_barrier(0);
                    }
                    d = total(d);
                    if (k >= 256) d = inf;
                    second = d < best ? best : fminf(second, d);
                    if (d < best) {
                        best = d;
                        code = k;
                    }
                }
                const float eta = (float)(4 * S + 6) * 6.1e-8f;
                const bool sure = best * (1.f + eta) < second * (1.f - eta) && second > 1e-25f;
                unsigned hard = (unsigned)__ballot(amb && !sure);   // exact and nearly exact ties: one after another, in fp64
                while (hard) {
                    const int v = __ffs(hard) - 1;
                    hard &= hard - 1u;
                    float4 *row = reinterpret_cast<float4 *>(lds + L.rows) + wave * 16 * NC;
                    unsigned *masks = reinterpret_cast<unsigned *>(lds + L.masks) + wave * KB;
#pragma unroll
                    for (int i = 0; i < KB; ++i) {
                        const unsigned bits = mk[i >> 1] >> (16 * (i & 1)) & 0xffffu;
                        unsigned spread = 0u;
#pragma unroll
                        for (int j = 0; j < 4; ++j) spread |= (bits >> (4 * j) & 15u) << (8 * j + 4 * h);
                        const uint2 o = both_halves(spread);
                        if (lane == v) masks[i] = o.x | o.y;
                    }
                    if (r == v) {
#pragma unroll
                        for (int s = 0; s < S; ++s) row[2 * s + h] = x[s];
                    }
                    wave_lds_fence();
                    const int k = encode_decide_fp64<KB>(reinterpret_cast<const float *>(row), Cm, masks, D, lane);
                    wave_lds_fence();
                    if (r == v) code = k;
                }
            }
            if (h == 0 && live) codes[n * M + m] = (uint8_t)code;
#pragma unroll
            for (int s = 0; s < S; ++s) {
                const float4 q = piece(Cm + (size_t)code * D, s);
                x[s] = make_float4(x[s].x - q.x, x[s].y - q.y, x[s].z - q.z, x[s].w - q.w);
            }
        }
        if (!given_up) rechecked += open;
        if (given_up && lane == 0) given[atomicAdd(given_count, 1u)] = tile;
        if (live && !given_up) {
#pragma unroll
            for (int s = 0; s < S; ++s)
                if (FULL || 8 * s + 4 * h < D) *reinterpret_cast<float4 *>(residue + n * D + 8 * s + 4 * h) = x[s];
        }
    }
    if (lane == 0) {
        if (rechecked_last) atomicAdd(refine_count, rechecked_last);
        if (rechecked) atomicAdd(work + 2, (unsigned long long)rechecked);
        if (!MANY && blockIdx.x == 0 && wave == 0) {
            work[0] += (unsigned long long)M;                       // launches on one stream follow one another
            work[1] += (unsigned long long)M * (unsigned long long)N;
        }
    }
}

}  // namespace hclae
