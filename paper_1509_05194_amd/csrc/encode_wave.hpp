// Greedy encoding (Sec. 3.3, Eq. 3 with one path) of large calls with rows of up to 128 coordinates, in one kernel: a wave takes 32
// vectors through ALL M dictionaries, the residual rows staying in its registers in between (K > 128 and D > 64: but for 13 to 15 registers'
// worth in scratch memory).
//
// Dictionary by dictionary a row crosses HBM three times per dictionary (assignment, residue in, residue out), which is what holds
// those kernels (N = 1M, D = 128, M = 8, K = 256: 24 passes of 512 MB).  Here it is read once and written once.  The fp16 dictionaries
// (k_encode_prep) pass through LDS, two of them held: while one is contracted the next travels from L2 into the other by direct
// loads, for all eight waves of the block together, one barrier per dictionary.  An undecided vector is decided at once, by the two
// lanes that hold its row, a candidate a round.  Scores, bounds and decisions are those of k_assign_half (assign_half.hpp), so the codes are the same fp64 direct-form
// decisions and the residuals the same fp32 subtractions as dictionary by dictionary.
//
// Measured (D = 128, M = 8, K = 256, us dictionary by dictionary / here): N = 1M 2480 / 1630, 200k 620 / 420, 49k 237 / 131; D = 64, 100k
// 288 / 140 (calls in a row; the kernel alone 1690 when it runs once).  Of the 1630, 930 are the arithmetic (MFMAs and VALU in turn, two waves to a SIMD), some 250 the rows to subtract (gathered
// from L2, 16 bytes a lane; through LDS with contiguous reads it is no faster), 230 the dictionaries' way into LDS and the barriers,
// 200 the undecided vectors.  Tiles whose vectors have many candidates go on in a second launch (k_encode_rest), which decides them with all
// the waves of a block; data that consist of such (N = 200k, M = 8, us dictionary by dictionary / here): groups 30 standard deviations apart
// 847 / 664, lognormal norms 8548 / 7202, codewords 1e-4 of the vectors 2301 / 2131, a dictionary of zeros 4562 / 4102.
#pragma once
#include "beam.hpp"
#include "encode.hpp"

namespace hclae {

// LDS of k_encode_wave.
struct WaveLds {
    int img, hn, w, mu, rows, masks, early, total;                  // byte offsets; img, hn, w, mu twice
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
    l.early = l.masks + kAssignWaves * kb * 4;
    l.total = l.early + 16;
    return l;
}

// 16 bytes per lane from global memory into LDS without passing through registers: lane i's to `to` + 16 i.
__device__ __forceinline__ void load_to_lds(const void *from, void *to)
{
    __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void *)from, (__attribute__((address_space(3))) void *)to,
                                     16, 0, 0);
}

// Candidates of a vector from which its tile is given up to k_encode_rest: a round takes one candidate of every vector.
constexpr unsigned kWaveMany = 20;

// FULL: D == 64 NC.
// given[0 .. counts[0]): tiles left to k_encode_rest, each with the first dictionary that it still needs.  A tile goes there as it stands when
// one of its vectors has kWaveMany candidates: its residual rows are in `residue` (at the first dictionary they are X), its codes so
// far in `codes`.  Where most tiles go before half of the dictionaries are done (counts[1] of them so far), the block leaves
// all it has not begun to that kernel and ends.
template <int KB, int NC, bool FULL>
__global__ __launch_bounds__(kAssignThreads) void k_encode_wave(
    const float *__restrict__ X, const float *__restrict__ C, int N, int D, int K, int M,
    const char *__restrict__ img, const float *__restrict__ hn, const float *__restrict__ wtab, const float *__restrict__ negmu,
    const float *__restrict__ consts, uint8_t *__restrict__ codes, float *__restrict__ residue,
    unsigned *__restrict__ refine_count, unsigned long long *__restrict__ work, uint2 *__restrict__ given,
    unsigned *__restrict__ counts)
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

    // dictionary m into a half of LDS: asynchronous but for the tables
    auto stage = [&](int m, int to_half) {
        const char *from = img + (size_t)m * L.img_size + 16 * lane;
        char *to = lds + L.img + to_half * L.img_size;
#pragma unroll
        for (int i = 0; i < (CHUNKS + kAssignWaves - 1) / kAssignWaves; ++i) {
            const int at = (i * kAssignWaves + wave) * 1024;
            if (CHUNKS % kAssignWaves == 0 || at < L.img_size) load_to_lds(from + at, to + at);
        }
        if ((int)threadIdx.x < 32 * KB) {
            reinterpret_cast<float *>(lds + L.hn + to_half * L.hn_size)[threadIdx.x] = hn[(size_t)m * 32 * KB + threadIdx.x];
            reinterpret_cast<float *>(lds + L.w + to_half * L.hn_size)[threadIdx.x] = wtab[(size_t)m * 32 * KB + threadIdx.x];
        }
        if ((int)threadIdx.x < 64 * NC) reinterpret_cast<float *>(lds + L.mu + to_half * L.mu_size)[threadIdx.x] = negmu[(size_t)m * 64 * NC + threadIdx.x];
    };
    int b = 0;                                                      // the half of LDS with the running dictionary
    unsigned *lds_early = reinterpret_cast<unsigned *>(lds + L.early);
    auto landed = [&]() {                                           // what this wave sent for has arrived, and everybody's
        __builtin_amdgcn_s_waitcnt(0x0f70);                         // vmcnt(0)
        __syncthreads();
    };
    auto piece = [&](const float *row, int s) {
        if (FULL || 8 * s + 4 * h < D) return *reinterpret_cast<const float4 *>(row + 8 * s + 4 * h);
        return make_float4(0.f, 0.f, 0.f, 0.f);
    };

    const unsigned ntiles = ((unsigned)N + kTileVec - 1) / kTileVec;
    const int nbt = (int)((ntiles + kAssignWaves - 1) / kAssignWaves);
    if ((int)blockIdx.x < nbt) {
        stage(0, 0);
        landed();
    }
    for (int bt = blockIdx.x; bt < nbt; bt += gridDim.x) {
        const unsigned tile = (unsigned)bt * kAssignWaves + wave, at = tile * kTileVec + r;     // beyond the last: for the barriers
        const bool live = at < (unsigned)N;
        int given_up = -1;                                          // at which dictionary
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
            // the counter as it is in memory (sc1): a copy that the block reads behind the next barrier and before the one after it
            if (m == M - 1 && threadIdx.x == 0)
                __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void *)(counts + 1),
                                                 (__attribute__((address_space(3))) void *)(lds_early + b), 4, 0, 16);
            if (more) stage(m + 1 < M ? m + 1 : 0, b ^ 1);
            if (given_up >= 0) {
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
            float mx;
            int code = best_half<KB>(acc, h, K, mx);
            const float *Cm = C + (size_t)m * K * D;
            const float hh = margin_half(c, mx, xn, e);
            const float thr = mx - 2.f * e * lds_w[code] - 2.f * hh;
            const bool big = !(x2 < kHalfMaxNorm * kHalfMaxNorm && fabsf(thr) < kHalfMaxThr);
            subtract_half<KB>(acc, thr, h);
            uint32_t mk[4];
            not_negative<KB>(mk, acc);
            const uint2 count = both_halves((unsigned)(__popc(mk[0]) + __popc(mk[1]) + __popc(mk[2]) + __popc(mk[3])));
            const bool amb = K > 1 && live && (big || count.x + count.y != 1u);
            landed();                                               // the next dictionary is there, this one is free
            if (__ballot(amb && (big || count.x + count.y >= kWaveMany))) {
                given_up = m;
                if (2 * m < M && lane == 0) atomicAdd(counts + 1, 1u);
                continue;
            }
            const unsigned who = (unsigned)__ballot(amb);
            if (who) {
                rechecked += (unsigned)__popc(who);
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
        if (given_up >= 0 && lane == 0) given[atomicAdd(counts, 1u)] = make_uint2(tile, (unsigned)given_up);
        if (live && given_up != 0) {
#pragma unroll
            for (int s = 0; s < S; ++s)
                if (FULL || 8 * s + 4 * h < D) *reinterpret_cast<float4 *>(residue + n * D + 8 * s + 4 * h) = x[s];
        }
        // tiles begun so far, at most: every block is in its round or behind
        if ((unsigned)kAssignWaves * (unsigned)(bt - (int)blockIdx.x + (int)gridDim.x) < 2u * lds_early[b ^ 1]) {
            const unsigned next = tile + (unsigned)kAssignWaves * gridDim.x, step = (unsigned)kAssignWaves * gridDim.x;
            const unsigned rest = next < ntiles ? (ntiles - next + step - 1) / step : 0u;
            unsigned to = 0u;
            if (lane == 0 && rest) to = atomicAdd(counts, rest);
            to = __builtin_amdgcn_readfirstlane(to);
            for (unsigned i = lane; i < rest; i += kWave) given[to + i] = make_uint2(next + i * step, 0u);
            break;
        }
    }
    if (lane == 0) {
        if (rechecked_last) atomicAdd(refine_count, rechecked_last);
        if (rechecked) atomicAdd(work + 2, (unsigned long long)rechecked);
        if (blockIdx.x == 0 && wave == 0) {
            work[0] += (unsigned long long)M;                       // launches on one stream follow one another
            work[1] += (unsigned long long)M * (unsigned long long)N;
        }
    }
}

// The tiles that k_encode_wave gives up, dictionary by dictionary as k_assign_half and the row pass take them, in one launch: the tiles of a block
// are its own from one dictionary to the next, so that its barriers are all there is between the steps.  The dictionaries come as
// k_encode_prep left them; hneg: -||c||^2/2 of their codewords as they are.  What bounds it are the gathers of decide_items, as there: all tiles
// of N = 1M in it, M = 2, lognormal norms 11.0 ms (dictionary by dictionary 10.7), a dictionary of zeros 18.0 (17.9).
template <int KB, int NC>
__global__ __launch_bounds__(kAssignThreads) void k_encode_rest(
    const float *X, const float *__restrict__ C, int N, int D, int K, int M,
    const char *__restrict__ img, const float *__restrict__ hn, const float *__restrict__ wtab, const float *__restrict__ negmu,
    const float *__restrict__ consts, const float *__restrict__ hneg, uint8_t *codes, float *residue,
    unsigned *__restrict__ refine_count, unsigned long long *__restrict__ work, const uint2 *__restrict__ given,
    const unsigned *__restrict__ counts, HalfItem *items)
{
    extern __shared__ float4 smem4[];
    char *lds = reinterpret_cast<char *>(smem4);
    constexpr HalfLds L = half_lds(KB, NC, NC);
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const float *lds_h = reinterpret_cast<const float *>(lds + L.hneg);
    const int ntiles = (int)counts[0];
    if ((int)blockIdx.x >= ntiles) return;
    HalfWave w = half_wave(lds, L, items + (size_t)half_share(ntiles, gridDim.x, -1) * kTileVec * blockIdx.x);
    const int places = half_tiles_of(blockIdx.x, wave, ntiles, gridDim.x, -1);
    auto entry = [&](int j) { return given[half_tile(blockIdx.x, wave + kAssignWaves * j, gridDim.x, -1)]; };
    int *first = reinterpret_cast<int *>(lds + L.misc);             // dictionary that some tile of the block needs
    if (threadIdx.x == 0) *first = M;
    __syncthreads();
    for (int j = lane_id(); j < places; j += kWave) atomicMin(first, (int)entry(j).y);
    __syncthreads();
    const int m0 = *first;
    unsigned rechecked = 0u, rechecked_last = 0u;
    for (int m = m0; m < M; ++m) {
        const float *src = m == 0 ? X : residue, *Cm = C + (size_t)m * K * D;
        // (lane numbers anew for every dictionary: what the compiler derives from them once and keeps is spilled, 31 registers instead of 8)
        int lane = lane_id();
        asm volatile("" : "+v"(lane));
        const int h = lane >> 5, r = lane & 31;
        {
            const uint4 *from = reinterpret_cast<const uint4 *>(img + (size_t)m * KB * NC * 4096);
            uint4 *to = reinterpret_cast<uint4 *>(lds + L.img);
#pragma unroll 4
            for (int i = threadIdx.x; i < KB * NC * 256; i += kAssignThreads) to[i] = from[i];
            if ((int)threadIdx.x < 32 * KB) {
                const int row = threadIdx.x;
                const float up = wtab[(size_t)m * 32 * KB + row];   // fp16 numbers; 0 beyond K
                const halfx2 pair = {(_Float16)up, (_Float16)0.f};
                reinterpret_cast<float *>(lds + L.hneg)[row] = hn[(size_t)m * 32 * KB + row];
                reinterpret_cast<float *>(lds + L.w)[row] = up;
                unsigned *aug = reinterpret_cast<unsigned *>(lds + L.waug) + 64 * (row >> 5) + (row & 31);
                aug[0] = __builtin_bit_cast(unsigned, pair);
                aug[32] = 0u;
            }
            if ((int)threadIdx.x < 64 * NC) reinterpret_cast<float *>(lds + L.mu)[threadIdx.x] = negmu[(size_t)m * 64 * NC + threadIdx.x];
            if (threadIdx.x == 0) *w.open = HalfOpen{0u, 0u, 0u};
        }
        const float *cc = consts + (size_t)m * kEncodeConsts;
        HalfConsts c;
        c.scale = cc[0];
        c.inv = 1.f;                                                // of bounds that nobody keeps here
        c.h = cc[1];
        c.rho = cc[2];
        c.acc = cc[3];
        c.hx = cc[4];
        c.cmax = cc[5];
        __syncthreads();
        // the wave's next tile that needs this dictionary
        auto skip = [&](int j) {
            while (j < places && (int)entry(j).y > m) ++j;
            return j;
        };
        auto vec_of = [&](int j) { return (int)min(entry(j).x * kTileVec + r, (unsigned)N); };
        auto row_ptr = [&](int n) { return src + (size_t)(n < N ? n : N - 1) * D; };
        int j = skip(0);
        if (j < places) {
            int n = vec_of(j), q = 0;
            float4 x[8];
            load_x_chunk<false>(x, row_ptr(n), 0, h, D);
            floatx16 acc[KB];
            float xsq = 0.f, dsq = 0.f;
            init_acc<KB>(acc, lds_h, h);
            while (j < places) {
                const int q_n = q + 1 == NC ? 0 : q + 1, j_n = q_n ? j : skip(j + 1);
                const int n_n = q_n ? n : vec_of(j_n < places ? j_n : j);       // after the last step the row again: unused
                mfma_chunk_refill<KB, 1>(acc, x, lds + L.img, reinterpret_cast<const float *>(lds + L.mu), q, lane, c.scale, xsq, dsq, row_ptr(n_n), q_n, D);
                if (q_n == 0) {
                    const float x2 = xsq + __shfl_xor(xsq, 32, kWave), norm = sqrtf(x2) * 1.001f;
                    const float e = mfma_bound_half<KB>(acc, reinterpret_cast<const unsigned *>(lds + L.waug), x2,
                                                        dsq + __shfl_xor(dsq, 32, kWave), norm, c, lane);
                    decide_half<KB, 0>(acc, x2, norm, e, c, reinterpret_cast<const float *>(lds + L.w), lane, n, N, D, K, M, m, 0u, codes,
                                       PruneArgs{}, w, nullptr, nullptr);
                    init_acc<KB>(acc, lds_h, h);
                    xsq = 0.f;
                    dsq = 0.f;
                }
                n = n_n;
                j = j_n;
                q = q_n;
            }
        }
        decide_items<KB, 0>(w, src, Cm, hneg + (size_t)m * 32 * KB, D, D, K, M, m, codes, PruneArgs{}, nullptr, nullptr);
        __syncthreads();                                            // the codes are there
        rechecked += w.open->items;
        if (m == M - 1) rechecked_last = w.open->items;
        // the rows of the wave's tiles: 16 NC lanes a row
        constexpr int W = 16 * NC, RP = kWave / W, U = 8;
        const int p = lane & (W - 1);
        if (4 * p < D) {
            for (j = skip(0); j < places; j = skip(j + 1)) {
                const unsigned n0 = entry(j).x * kTileVec;
#pragma unroll 1
                for (int i0 = 0; i0 < kTileVec; i0 += U * RP) {
                    float4 x[U], q[U];
                    int k[U];
#pragma unroll
                    for (int u = 0; u < U; ++u) {
                        const size_t row = min(n0 + i0 + u * RP + lane / W, (unsigned)N - 1u);
                        k[u] = codes[row * M + m];
                        x[u] = reinterpret_cast<const float4 *>(src + row * D)[p];
                    }
                    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                    for (int u = 0; u < U; ++u) q[u] = reinterpret_cast<const float4 *>(Cm + (size_t)k[u] * D)[p];
                    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                    for (int u = 0; u < U; ++u) {
                        const unsigned row = n0 + i0 + u * RP + lane / W;
                        if (row < (unsigned)N)
                            reinterpret_cast<float4 *>(residue + (size_t)row * D)[p] =
                                make_float4(x[u].x - q[u].x, x[u].y - q[u].y, x[u].z - q[u].z, x[u].w - q[u].w);
                    }
                }
            }
        }
        __syncthreads();                                            // rows and counters are free
    }
    if (threadIdx.x == 0) {
        if (rechecked_last) atomicAdd(refine_count, rechecked_last);
        if (rechecked) atomicAdd(work + 2, (unsigned long long)rechecked);
    }
}

}  // namespace hclae
