// Assignments of a stage from a copy of x' in fp16 operands (Sec. 3.1: within a stage x' is fixed, only the dictionary moves).
//
// The assignment of assign_half.hpp reads x' in fp32, centres, scales and rounds it, every time: up to eleven times a stage, and it
// is the reads that hold it (N = 1M, D = 128: 512 MB of an HBM pass, 85 of some 150 us).  A stage that keeps distance bounds
// therefore has the pass that writes x' write the rounded rows X^ beside it, with ||X||^2 and ||X - X^||^2 per vector (25 to
// 29 % more bytes in that pass), and all its assignments read those: half of the bytes and no conversion.  The centre mu and the scale are those of the
// dictionary as the stage finds it and stay for the stage: the bounds hold for any.  The dictionary's image follows from them too,
// codeword by codeword, so the merge writes it where it writes the codeword, and an assignment copies 64 KB into LDS instead of
// rounding 128 KB in every block.  Undecided vectors are decided from x' in fp32 as before: the codes are the same.
// Measured, before / with them: pruned assignments of a training at N = 1M, D = 128, K = 256 110 us / 80 us on average, the first of a
// stage 138 / 101; N = 250k 31.9 / 23.2; N = 200k, D = 960 185 / 148; trainings of the four sizes 8 to 13 % shorter, boundary pass and all.
//
// Row n of X^: 16 ceil(D / 16) halfs, k-step t in halfs 16 t .. 16 t + 15, of which lane half h of the product reads 8 h .. 8 h + 7:
// dims 16 t + 4 h .. + 3 and 16 t + 8 + 4 h .. + 3 (assign_half.hpp).  Halfs beyond D are zero from the allocation on.
#pragma once
#include "assign_half.hpp"
#include "stream.hpp"

namespace hclae {

constexpr int kRefSamples = 64;                     // vectors whose norms count for the scale
enum { kWordAmax = 0, kWordCmax = kAmaxSlots, kWordXmax, kWordTicket, kWords16 };

__host__ __device__ constexpr int rows16_ld(int D) { return (D + 15) & ~15; }

// Before the pass that writes x'' of stage j: its centre and scale, from what will be the stage's dictionary: Cj as it is, or the
// rows of x'' that seed it (idx), formed here as the pass forms them.  src, Cm: the pass is the stage boundary (x'' = (src - c_m) + c_j)
// or, with Cm null, the heat pass (x'' = src + c_j).
// Scale: the power of two that brings the larger of the codewords' and the sampled vectors' norms into [2^9, 2^10): the centroids to come
// are no longer than the vectors they are means of, whatever the dictionary is now, vectors up to 64 times those stay in fp16's range
// (kHalfMaxNorm), and coordinates down to 2^-23 of them are normal numbers.  A wave per row; the last block to finish writes the
// result and clears the words.
__global__ __launch_bounds__(256) void k_rows16_ref(
    const float *__restrict__ src, const uint8_t *__restrict__ codes, const float *__restrict__ Cm, const float *__restrict__ Cj,
    int64_t N, int D, int K, int M, int m, int j, int NC, const int64_t *__restrict__ idx, float *__restrict__ ref,
    float *__restrict__ negmu, float *__restrict__ consts, unsigned *__restrict__ words)
{
    __shared__ bool last;
    const int lane = lane_id(), item = blockIdx.x * 4 + (threadIdx.x >> 6);
    const int d4 = D >> 2;
    if (item < K + kRefSamples) {
        const bool sample = item >= K;
        const bool row = sample || idx;
        const int64_t n = sample ? (int64_t)(item - K) * N / kRefSamples : idx ? idx[item] : 0;
        const float4 *from = reinterpret_cast<const float4 *>(row ? src + n * D : Cj + (size_t)item * D);
        const float4 *a = reinterpret_cast<const float4 *>(row && Cm ? Cm + (size_t)codes[n * M + m] * D : nullptr);
        const float4 *b = reinterpret_cast<const float4 *>(row ? Cj + (size_t)codes[n * M + j] * D : nullptr);
        float s = 0.f;
        for (int p = lane; p < d4; p += kWave) {
            float4 v = from[p];
            if (a) {
                const float4 w = a[p];
                v = make_float4(v.x - w.x, v.y - w.y, v.z - w.z, v.w - w.w);
            }
            if (b) {
                const float4 w = b[p];
                v = make_float4(v.x + w.x, v.y + w.y, v.z + w.z, v.w + w.w);
            }
            s = fmaf(v.x, v.x, fmaf(v.y, v.y, fmaf(v.z, v.z, fmaf(v.w, v.w, s))));
            if (row && !sample) reinterpret_cast<float4 *>(ref + (size_t)item * D)[p] = v;
        }
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) s += __shfl_xor(s, o, kWave);
        if (lane == 0) atomicMax(words + (sample ? kWordXmax : kWordCmax), __float_as_uint(s));
    }
    __threadfence();
    __syncthreads();
    if (threadIdx.x == 0) last = atomicAdd(words + kWordTicket, 1u) == gridDim.x - 1;
    __syncthreads();
    if (!last) return;
    __threadfence();
    const float c2 = __uint_as_float(atomicAdd(words + kWordCmax, 0u)), x2 = __uint_as_float(atomicAdd(words + kWordXmax, 0u));
    __syncthreads();
    const int e = half_exponent(0.5f * fmaxf(c2, x2)) + 3;
    const float f = -ldexpf(1.f, e) / kMuRows;
    const float *C = idx ? ref : Cj;
    for (int p = threadIdx.x; p < 16 * NC; p += 256) {
        float4 mu = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
        for (int i = 0; i < kMuRows; ++i) {
            const float4 w = load_row_piece(C, (int)((unsigned)(i * K) / kMuRows), 4 * p, K, D, D);
            mu.x += w.x;
            mu.y += w.y;
            mu.z += w.z;
            mu.w += w.w;
        }
        reinterpret_cast<float4 *>(negmu)[p] = make_float4(mu.x * f, mu.y * f, mu.z * f, mu.w * f);
    }
    if (threadIdx.x == 0) {
        consts[0] = ldexpf(1.f, e);
        consts[1] = ldexpf(1.f, -e);
    }
    if (threadIdx.x < kWords16) words[threadIdx.x] = 0u;
}

// The dictionary's image in the stage's centre and scale, with the sums its constants come from, and what k_codeword_norms does at
// the beginning of a stage.  A wave per row of the padded dictionary; later changes of a codeword are written by the merge.
__global__ __launch_bounds__(256) void k_rows16_image(
    const float *__restrict__ Cm, int K, int D, int kb, int NC, const float *__restrict__ negmu, const float *__restrict__ consts,
    char *__restrict__ img, float *__restrict__ sums, float *__restrict__ hneg, unsigned *__restrict__ refine_count,
    unsigned *__restrict__ words, float *__restrict__ entry_copy, unsigned *__restrict__ zero_word)
{
    const int lane = lane_id(), row = blockIdx.x * 4 + (threadIdx.x >> 6);
    if (blockIdx.x == 0 && threadIdx.x < kWave) {
        static_assert(kAmaxSlots == kWave, "a word per lane");
        unsigned mx = words[kWordAmax + lane];
        words[kWordAmax + lane] = 0u;
        mx = (unsigned)wave_max_int((int)mx);                       // bits of non-negative floats
        if (lane == 0) {
            refine_count[0] = 0u;
            refine_count[1] = mx;
            if (zero_word) *zero_word = 0u;
        }
    }
    const float scale = consts[0];
    float sq = 0.f, dsq = 0.f;
    double s = 0.0;
    for (int p = lane; p < 16 * NC; p += kWave) {
        const float4 v = load_row_piece(Cm, row, 4 * p, K, D, D);
        s += (double)v.x * v.x + (double)v.y * v.y + (double)v.z * v.z + (double)v.w * v.w;
        if (entry_copy && row < K && 4 * p < D) reinterpret_cast<float4 *>(entry_copy + (size_t)row * D)[p] = v;
        float4 w = scaled(v, scale, reinterpret_cast<const float4 *>(negmu)[p]);
        if (row >= K) w = make_float4(0.f, 0.f, 0.f, 0.f);
        const halfx4 q = half4(w, sq, dsq);
        const int t = p >> 2, g = p & 1, hi = (p >> 1) & 1;
        *reinterpret_cast<halfx4 *>(img + (size_t)(t * kb + (row >> 5)) * 1024 + half_slot(t, g, row & 31) + 8 * hi) = q;
    }
    s = wave_sum(s);
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        sq += __shfl_xor(sq, o, kWave);
        dsq += __shfl_xor(dsq, o, kWave);
    }
    if (lane == 0) {
        sums[2 * row] = sq;
        sums[2 * row + 1] = dsq;
        hneg[row] = row < K ? -(float)(0.5 * s) : -__builtin_inff();
    }
}

// The largest centred codeword norm that fits fp16 in the stage's units for certain: beyond (a cluster of an outlier 32 times as long as
// what set the scale) every codeword is a candidate of every vector until the stage ends.
constexpr float kRows16MaxNorm = 32000.f;

// Rows, code and norms behind a column of a tile.
struct Rows16Args {
    const _Float16 *rows;                           // [N][ld]
    const float2 *norm;                             // [N] {||X||^2, ||X - X^||^2}
    const float *consts;                            // scale, 1 / scale
    const char *img;                                // the dictionary, in the order of half_slot
    const float *sums;                              // [32 kb][2]
    int ld, steps;                                  // halfs of a row; 16-dim steps of it
};

// k_assign_half over the fp16 rows, the dictionary resident in LDS.  A wave owns tiles of 32 vectors; up to eight k-steps (128 dims)
// of a row, 256 bytes, are in flight while the ones before are contracted.  UNIT: so many, 8 where the row's steps are a multiple of it, else 4.
template <int KB, int PRUNE, int UNIT>
__global__ __launch_bounds__(kAssignThreads) void k_assign_rows16(
    const float *__restrict__ xp, const float *__restrict__ Cm, const float *__restrict__ hneg, Rows16Args x16,
    int N, int D, int K, int M, int m, int NC,
    uint8_t *__restrict__ codes, unsigned *__restrict__ refine_count, PruneArgs pa,
    unsigned long long *__restrict__ moved_list, unsigned *__restrict__ moved_count, unsigned long long *__restrict__ work,
    HalfItem *__restrict__ items)
{
    extern __shared__ float4 smem4[];
    char *lds = reinterpret_cast<char *>(smem4);
    const HalfLds L = half_lds(KB, NC, NC);
    const int lane = lane_id(), wave = threadIdx.x >> 6, h = lane >> 5, r = lane & 31;
    const float *lds_h = reinterpret_cast<const float *>(lds + L.hneg);
    const bool want_moved = moved_list != nullptr;

    const int listed = PRUNE == 2 ? (int)*pa.active_count : N;
    const bool gather = PRUNE == 2 && listed < N - (N >> 5);
    const int rows = gather ? listed : N;
    const int ntiles = (int)(((unsigned)rows + kTileVec - 1) / kTileVec);
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        work[0] += 1ull;                                            // launches on one stream follow one another
        work[1] += (unsigned long long)listed;
    }
    if ((int)blockIdx.x >= ntiles) return;                      // no tile for any wave of this block

    const int tstride = (int)gridDim.x * kAssignWaves;
    const int t0 = (int)blockIdx.x + (int)gridDim.x * wave;     // with few tiles, a block each before any block gets two
    HalfWave w = half_wave(lds, L, items + (size_t)((ntiles + tstride - 1) / tstride) * kTileVec * kAssignWaves * blockIdx.x);
    const int my_tiles = t0 < ntiles ? (ntiles - t0 + tstride - 1) / tstride : 0;
    const int NU = (x16.steps + UNIT - 1) / UNIT;                   // units of so many steps
    const int64_t G = (int64_t)my_tiles * NU;

    auto vec_of = [&](int tile) -> int {                            // N (= "none") for the columns of the ragged tail
        const unsigned i = (unsigned)tile * kTileVec + r;
        if (i >= (unsigned)rows) return N;
        return gather ? (int)pa.active[i] : (int)i;
    };
    auto real = [&](int n) { return n < N ? n : gather ? (int)pa.active[rows - 1] : N - 1; };   // tail columns re-read the last row
    auto unit = [&](int n, int u) { return reinterpret_cast<const uint4 *>(x16.rows + (size_t)real(n) * x16.ld) + 2 * UNIT * u + h; };
    // steps beyond the row re-read its last one: they are not contracted
    auto fetch = [&](const uint4 *p, int u, int t) { return p[2 * (UNIT == 8 ? t : min(t, x16.steps - 1 - UNIT * u))]; };
    int tile = t0, n = N;
    unsigned old = 0u;
    float2 nv = make_float2(0.f, 0.f);
    uint4 x[UNIT];
    if (G > 0) {                                                    // the first unit travels while the dictionary is staged
        n = vec_of(t0);
        const uint4 *p = unit(n, 0);
#pragma unroll
        for (int t = 0; t < UNIT; ++t) x[t] = fetch(p, 0, t);
        nv = x16.norm[real(n)];
        if (want_moved && n < N) old = codes[(size_t)n * M + m];
    }
    {
        const int pieces = KB * NC * 256;                           // of 16 bytes
        const uint4 *from = reinterpret_cast<const uint4 *>(x16.img);
        uint4 *to = reinterpret_cast<uint4 *>(lds);
#pragma unroll 4
        for (int i = threadIdx.x; i < pieces; i += kAssignThreads) to[i] = from[i];
    }
    const bool holder = (int)threadIdx.x < 32 * KB;
    const HalfConsts c = half_constants<KB>(lds, L, holder ? x16.sums[2 * threadIdx.x] : 0.f, holder ? x16.sums[2 * threadIdx.x + 1] : 0.f,
                                            threadIdx.x, holder, K, NC, x16.consts[0], x16.consts[1]);
    const float lost = c.cmax <= kRows16MaxNorm ? 0.f : __builtin_inff();
    if (G > 0) {
        floatx16 acc[KB];
        int u = 0;
        init_acc<KB>(acc, lds_h, h);
        for (int64_t g = 0; g < G; ++g) {
            const bool more = g + 1 < G;
            int tile_n = tile, n_n = n, u_n = u + 1;
            unsigned old_n = old;
            float2 nv_n = nv;
            if (u_n == NU) {
                u_n = 0;
                tile_n = tile + tstride;
                if (more) {
                    n_n = vec_of(tile_n);
                    nv_n = x16.norm[real(n_n)];
                    if (want_moved) old_n = n_n < N ? codes[(size_t)n_n * M + m] : 0u;
                }
            }
            const uint4 *next = more ? unit(n_n, u_n) : unit(n, u);     // the last unit re-reads itself: unused
            const int u_f = more ? u_n : u;
            contract_half<KB, UNIT>(acc, lds + (size_t)u * UNIT * KB * 1024, h, r, UNIT == 8 ? 8 : x16.steps - UNIT * u,
                                    [&](int t) { return __builtin_bit_cast(halfx8, x[t]); },
                                    [&](int t) { x[t] = fetch(next, u_f, t); });
            if (u == NU - 1) {
                const float xn1 = sqrtf(nv.x) * 1.001f;
                const float e = mfma_bound_half<KB>(acc, reinterpret_cast<const unsigned *>(lds + L.waug), nv.x, nv.y, xn1, c, lane);
                decide_half<KB, PRUNE>(acc, nv.x + lost, xn1, e, c, reinterpret_cast<const float *>(lds + L.w), lane, n, N, D, K, M, m, old,
                                       codes, pa, w, moved_list, moved_count);
                init_acc<KB>(acc, lds_h, h);                        // here and not where the next tile begins: dead until now
            }
            tile = tile_n;
            n = n_n;
            u = u_n;
            old = old_n;
            nv = nv_n;
        }
    }
    decide_items<KB, PRUNE>(w, xp, Cm, hneg, D, D, K, M, m, codes, pa, moved_list, moved_count);
    half_finish<2>(lds, L, w, 0.f, refine_count, moved_list, moved_count, work);
}

// k_assign_half_chunked over the fp16 rows: the dictionary passes through LDS in 64-dim slices, two of them held; a lane's part of
// two slices of its row is in registers, each refilled two slices ahead.
template <int KB, int PRUNE>
__global__ __launch_bounds__(kAssignThreads) void k_assign_rows16_chunked(
    const float *__restrict__ xp, const float *__restrict__ Cm, const float *__restrict__ hneg, Rows16Args x16,
    int N, int D, int K, int M, int m, int NC,
    uint8_t *__restrict__ codes, unsigned *__restrict__ refine_count, PruneArgs pa,
    unsigned long long *__restrict__ moved_list, unsigned *__restrict__ moved_count, unsigned long long *__restrict__ work,
    HalfItem *__restrict__ items)
{
    extern __shared__ float4 smem4[];
    char *lds = reinterpret_cast<char *>(smem4);
    const HalfLds L = half_lds(KB, NC, 2);
    constexpr int SLICE = KB * 4096, PIECES = SLICE / 16;
    const int lane = lane_id(), wave = threadIdx.x >> 6, h = lane >> 5, r = lane & 31;
    const float *lds_h = reinterpret_cast<const float *>(lds + L.hneg);

    const int listed = PRUNE == 2 ? (int)*pa.active_count : N;
    const bool gather = PRUNE == 2 && listed < N - (N >> 5);
    const int rows = gather ? listed : N;
    const int nbt = (int)(((unsigned)rows + kTileVec * kAssignWaves - 1) / (kTileVec * kAssignWaves));   // block tiles
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        work[0] += 1ull;                                            // launches on one stream follow one another
        work[1] += (unsigned long long)listed;
    }
    if ((int)blockIdx.x >= nbt) return;

    auto vec_of = [&](int bt) -> int {                              // N (= "none") in the ragged tail
        const unsigned i = ((unsigned)bt * kAssignWaves + wave) * kTileVec + r;
        if (i >= (unsigned)rows) return N;
        return gather ? (int)pa.active[i] : (int)i;
    };
    auto real = [&](int n) { return n < N ? n : gather ? (int)pa.active[rows - 1] : N - 1; };   // tail columns re-read the last row
    // the slice that is fetched next: fq of the row frow of the block tile fbt
    int fbt = blockIdx.x, fq = 0;
    int n = vec_of(fbt), n_n = n;
    const uint4 *frow = reinterpret_cast<const uint4 *>(x16.rows + (size_t)real(n) * x16.ld) + h;
    float2 nv = x16.norm[real(n)], nv_n = nv;
    unsigned old = moved_list && n < N ? codes[(size_t)n * M + m] : 0u, old_n = old;
    // steps beyond the row re-read its last one: the dictionary is zero there
    auto fetch = [&](uint4 &x, int t) { x = frow[2 * min(4 * fq + t, x16.steps - 1)]; };
    auto advance = [&]() {
        if (++fq < NC) return;
        fq = 0;
        fbt += gridDim.x;
        if (fbt >= nbt) return;                                     // the last tile's row again: unused
        n_n = vec_of(fbt);
        frow = reinterpret_cast<const uint4 *>(x16.rows + (size_t)real(n_n) * x16.ld) + h;
        nv_n = x16.norm[real(n_n)];
        if (moved_list) old_n = n_n < N ? codes[(size_t)n_n * M + m] : 0u;
    };
    uint4 xa[4], xb[4];
#pragma unroll
    for (int t = 0; t < 4; ++t) fetch(xa[t], t);
    advance();
#pragma unroll
    for (int t = 0; t < 4; ++t) fetch(xb[t], t);
    advance();

    for (int i = threadIdx.x; i < PIECES; i += kAssignThreads)
        reinterpret_cast<uint4 *>(lds)[i] = reinterpret_cast<const uint4 *>(x16.img)[i];
    const bool holder = (int)threadIdx.x < 32 * KB;
    const HalfConsts c = half_constants<KB>(lds, L, holder ? x16.sums[2 * threadIdx.x] : 0.f, holder ? x16.sums[2 * threadIdx.x + 1] : 0.f,
                                            threadIdx.x, holder, K, NC, x16.consts[0], x16.consts[1]);
    const float lost = c.cmax <= kRows16MaxNorm ? 0.f : __builtin_inff();
    HalfWave w = half_wave(lds, L, items + (size_t)((nbt + gridDim.x - 1) / gridDim.x) * kTileVec * kAssignWaves * blockIdx.x);

    floatx16 acc[KB];
    init_acc<KB>(acc, lds_h, h);
    int q = 0, par = 0;
    // contracts slice q of the tile with x and refills x two slices on; the next dictionary slice comes in behind the MFMAs
    auto step = [&](uint4 (&x)[4]) {
        constexpr int GB = KB < 4 ? KB : 4;
        const int qn = q + 1 == NC ? 0 : q + 1;
        const uint4 *src = reinterpret_cast<const uint4 *>(x16.img + (size_t)qn * SLICE);
        const char *cur = lds + par * SLICE;
        uint4 *nxt = reinterpret_cast<uint4 *>(lds + (par ^ 1) * SLICE);
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            const int at = t * kAssignThreads + (int)threadIdx.x;
            uint4 piece = make_uint4(0u, 0u, 0u, 0u);
            if ((t + 1) * kAssignThreads <= PIECES || (t * kAssignThreads < PIECES && at < PIECES)) piece = src[at];
            const halfx8 b16 = __builtin_bit_cast(halfx8, x[t]);
            fetch(x[t], t);
            const char *base = cur + half_slot(t, h, r);
#pragma unroll
            for (int b0 = 0; b0 < KB; b0 += GB) {
                halfx8 a[GB];
#pragma unroll
                for (int b = 0; b < GB; ++b) a[b] = *reinterpret_cast<const halfx8 *>(base + (t * KB + b0 + b) * 1024);
#pragma unroll
                for (int b = 0; b < GB; ++b) acc[b0 + b] = __builtin_amdgcn_mfma_f32_32x32x16_f16(a[b], b16, acc[b0 + b], 0, 0, 0);
            }
            // the store (and the wait for its load) stays behind the step's MFMAs
            __builtin_amdgcn_sched_barrier(0x10f);
            if ((t + 1) * kAssignThreads <= PIECES || (t * kAssignThreads < PIECES && at < PIECES)) nxt[at] = piece;
        }
        __syncthreads();                                            // slice q consumed by all, slice qn complete
        par ^= 1;
        if (q + 1 == NC) {
            const float xn1 = sqrtf(nv.x) * 1.001f;
            const float e = mfma_bound_half<KB>(acc, reinterpret_cast<const unsigned *>(lds + L.waug), nv.x, nv.y, xn1, c, lane);
            decide_half<KB, PRUNE>(acc, nv.x + lost, xn1, e, c, reinterpret_cast<const float *>(lds + L.w), lane, n, N, D, K, M, m, old,
                                   codes, pa, w, moved_list, moved_count);
            init_acc<KB>(acc, lds_h, h);
            n = n_n;
            nv = nv_n;
            old = old_n;
        }
        q = qn;
        advance();
    };
    const int my_tiles = (nbt - (int)blockIdx.x + (int)gridDim.x - 1) / (int)gridDim.x;
    const int64_t G = (int64_t)my_tiles * NC;                       // the same in every wave of the block
    for (int64_t g = 0; g < G; g += 2) {
        step(xa);
        if (g + 1 >= G) break;
        step(xb);
    }
    decide_items<KB, PRUNE>(w, xp, Cm, hneg, D, D, K, M, m, codes, pa, moved_list, moved_count);
    half_finish<2>(lds, L, w, 0.f, refine_count, moved_list, moved_count, work);
}

}  // namespace hclae
