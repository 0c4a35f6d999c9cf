// Multi-path encoding (Sec. 3.3, Eq. 3): for every vector keep the L best sums a_l of codewords
// of the dictionaries seen so far; for the next dictionary score all K * L sums a_l + c(k) by
// || x - a_l - c(k) ||^2 and keep the L smallest.
//
// The beam is stored as residuals r_l = x - a_l (fp32 rows), so a candidate's error is || r_l - c(k) ||^2 and scoring a
// dictionary is the same codewords x vectors contraction as the nearest-codeword assignment, over N * L rows.  Two kernels per
// dictionary:
//   k_beam_score_*  fp16 matrix cores with the bounds of assign_half.hpp; per vector finds a value that the lower bounds of
//                   at least L candidates reach and writes, per beam row, the bitmap of codewords whose upper bound reaches
//                   it (so the L best in exact arithmetic are in it);
//   k_beam_expand   evaluates the listed candidates in fp64 in the direct form, sorts them by (error, l, k), keeps the first
//                   L and writes their residuals, errors and code prefixes.
// The decision is therefore an fp64 direct-form decision, as in the assignment kernels.
#pragma once
#include "assign_half.hpp"

namespace hclae {

constexpr int kBeamMaxL = 32;        // a vector's beam rows must fit one 32-column MFMA tile

// Candidate codewords of one beam row: bit p of w[h][i] is codeword 64 i + 8 (p >> 2) + 4 h + (p & 3).
struct BeamMask {
    uint32_t w[2][4];
};

// Threshold and bitmaps from a wave's upper scores U_k (assign_half.hpp).  Lane (h, r) holds those of beam row r of the tile
// for half of the codewords.  Half a candidate's squared distance is ||X||^2/2 - S_k, so candidates of one vector are ranked
// by S_k - ||X||^2/2 of their own row X (larger is better).
//   1. per lane, the maximum of each 16-score accumulator block, taken down to a lower bound of that candidate's rank
//      value: less 2 e cmax, h and the rounding of ||X||^2/2;
//   2. Ln rounds of "take the largest value of the vector's group of lanes and strike it out": the value taken in the last
//      round is reached by at least Ln distinct candidates (ties struck together only lower it);
//   3. every candidate whose upper bound reaches that value is marked.
// slack: rounding of ||X||^2 relative to it.  next[i]: lane that is 2^i rows further round the vector's group of Lc lanes.
constexpr int kBeamHops = 5;                        // 2^5 >= kBeamMaxL
template <int KB>
__device__ __forceinline__ void beam_select(
    const floatx16 (&acc)[KB], float x2, float xn, float e, const HalfConsts &c, float slack,
    int lane, const int (&next)[kBeamHops], int hops, int Ln, bool valid, BeamMask *__restrict__ out)
{
    const float ninf = -__builtin_inff();
    const float half_x2 = 0.5f * x2;
    float bm[KB], top = ninf;
#pragma unroll
    for (int b = 0; b < KB; ++b) {
        bm[b] = block_max(acc[b]);
        top = fmaxf(top, bm[b]);
    }
    const float round = c.h + c.acc * 6.2e-5f * xn + 2.4e-7f * (fabsf(top) + xn * c.cmax) + slack * x2 + 1e-36f;
    const float down = half_x2 + 2.f * e * (c.cmax * 1.01f + 1.2e-7f) + round;
    const bool big = !(x2 < kHalfMaxNorm * kHalfMaxNorm && down < 1e37f);     // may not fit fp16: all codewords are candidates
#pragma unroll
    for (int b = 0; b < KB; ++b) bm[b] = valid && !big ? bm[b] - down : ninf;

    float tau = ninf;
    for (int it = 0; it < Ln; ++it) {
        float g = bm[0];
#pragma unroll
        for (int b = 1; b < KB; ++b) g = fmaxf(g, bm[b]);
        g = fmaxf(g, __shfl_xor(g, 32, kWave));
#pragma unroll
        for (int i = 0; i < kBeamHops; ++i)
            if (i < hops) g = fmaxf(g, __shfl(g, next[i], kWave));
        tau = g;
#pragma unroll
        for (int b = 0; b < KB; ++b) bm[b] = (bm[b] == g) ? ninf : bm[b];
    }
    const float thr = (tau - round) + half_x2;           // back to the lane's scores

    // (the threshold is subtracted here and not on the matrix cores as in decide_half: they are the busier of the two)
    uint32_t mk[4];
    reaching<KB>(mk, acc, thr);
    if (big || !(thr > ninf))                            // (bits of codewords beyond K are dropped by the reader)
        mk[0] = mk[1] = mk[2] = mk[3] = ~0u;
    if (valid) *reinterpret_cast<uint4 *>(&out->w[lane >> 5][0]) = make_uint4(mk[0], mk[1], mk[2], mk[3]);
}

// What the scoring kernels share: tiles of V = 32 / Lc whole vectors = V Lc consecutive beam rows; the remaining columns of
// the 32 idle.
struct BeamTile {
    int rt, hops;                                       // beam rows per tile; doublings that cover a group
    int next[kBeamHops];
    __device__ __forceinline__ BeamTile(int lane, int Lc)
    {
        const int r = lane & 31;
        rt = (kTileVec / Lc) * Lc;
        const int base = r < rt ? (r / Lc) * Lc : 0, at = r < rt ? r - base : 0;
        hops = 0;
        while ((1 << hops) < Lc) ++hops;
#pragma unroll
        for (int i = 0; i < kBeamHops; ++i) next[i] = (lane & 32) + base + (at + (1 << i)) % Lc;
    }
};

// mfma_chunk_half with the dictionary's operands read ahead (contract_half) and x refilled in place, with chunk qn of row `next`, as soon
// as it has been converted: addresses are clamped into the row, and what lies past D is multiplied by zero (mu and the dictionary are
// zero there).  Here, where ten rows a vector keep the matrix cores busy, it saves a fiftieth of the call (N = 200k, L = 10, D = 128:
// 6.26 -> 6.14 ms, with the block maxima two scores a step).  For K > 128 only: with fewer codewords a step has too few MFMAs to hide what it
// sends for, and two buffers are shorter (a launch, N = 100k, L = 10, us so / two buffers: K = 21, D = 92 96 / 78, D = 128 110 / 104, K = 54, D = 92
// 88 / 79, K = 100, D = 192 157 / 153); k_assign_half, which waits for its rows, is 3 % slower with it.
// USE: an instance for each kernel that has it; shared with k_encode_rest the compiler puts it together in another order, and this kernel's
// calls take 1 % longer (5.95 -> 6.00 ms).
template <int KB, int USE = 0>
__device__ __forceinline__ void mfma_chunk_refill(
    floatx16 (&acc)[KB], float4 (&x)[8], const char *__restrict__ img, const float *__restrict__ negmu, int q, int lane,
    float scale, float &xsq, float &dsq, const float *__restrict__ next, int qn, int D)
{
    const int g = lane >> 5, r = lane & 31, last = last_piece(D);
    const float4 *mu4 = reinterpret_cast<const float4 *>(negmu) + 16 * q + g;
    auto fetch = [&](int s) { return *reinterpret_cast<const float4 *>(next + min(kChunkD * qn + 8 * s + 4 * g, last)); };
    contract_half<KB, 4>(acc, img + (size_t)q * 4 * KB * 1024, g, r, 4,
        [&](int t) {
            const int col = kChunkD * q + 16 * t + 4 * g;
            const halfx4 lo = half4(scaled(x[2 * t], col < D ? scale : 0.f, mu4[4 * t]), xsq, dsq);
            const halfx4 hi = half4(scaled(x[2 * t + 1], col + 8 < D ? scale : 0.f, mu4[4 * t + 2]), xsq, dsq);
            return __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
        },
        [&](int t) {
            x[2 * t] = fetch(2 * t);
            x[2 * t + 1] = fetch(2 * t + 1);
        });
}

// Scoring with the dictionary resident in LDS as fp16: staging, streaming and bounds of k_assign_half.
template <int KB>
__global__ __launch_bounds__(kAssignThreads) void k_beam_score_half(
    const float *__restrict__ rows, const float *__restrict__ Cm, const float *__restrict__ hneg,
    int64_t N, int Lc, int Ln, int D, int K, int NC, float slack, BeamMask *__restrict__ masks)
{
    extern __shared__ float4 smem4[];
    char *lds = reinterpret_cast<char *>(smem4);
    const HalfLds L = half_lds(KB, NC, NC);
    const int lane = lane_id(), wave = threadIdx.x >> 6, h = lane >> 5, r = lane & 31;
    const float *lds_h = reinterpret_cast<const float *>(lds + L.hneg);
    const float *lds_mu = reinterpret_cast<const float *>(lds + L.mu);
    const BeamTile bt(lane, Lc);
    const int64_t nrows = N * Lc;
    const int64_t ntiles = (nrows + bt.rt - 1) / bt.rt;
    const int64_t nslots = (int64_t)gridDim.x * 4, tstride = 2 * nslots;
    const int64_t t0 = (int64_t)blockIdx.x * 4 + (wave & 3) + nslots * (wave >> 2);
    const int64_t my_tiles = t0 < ntiles ? (ntiles - t0 + tstride - 1) / tstride : 0;
    const int64_t G = my_tiles * NC;
    auto row_ptr = [&](int64_t tile) {
        int64_t n = tile * bt.rt + r;
        if (r >= bt.rt || n >= nrows) n = nrows - 1;     // idle columns re-read the last row
        return rows + n * D;
    };
    float4 x[8];
    if (G > 0) load_x_chunk(x, row_ptr(t0), 0, h, D);    // travels while the dictionary is staged
    const HalfConsts c = stage_half<KB>(lds, L, Cm, hneg, K, D, D, NC);
    if (G == 0) return;
    floatx16 acc[KB];
    float xsq = 0.f, dsq = 0.f;
    int64_t tile = t0;
    int q = 0;
    init_acc<KB>(acc, lds_h, h);
    // one step: contract x (chunk q of the tile), with the chunk after it on its way into xn, and select where it was the tile's last
    auto step = [&](float4 (&x)[8], float4 (&xn)[8], bool more) {
        const int q_n = q + 1 == NC ? 0 : q + 1;
        const int64_t tile_n = q_n ? tile : tile + tstride;
        if constexpr (KB == 8) {                         // xn is x; the last step re-reads itself: unused
            mfma_chunk_refill<KB>(acc, x, lds + L.img, lds_mu, q, lane, c.scale, xsq, dsq, row_ptr(more ? tile_n : tile), more ? q_n : q, D);
        } else {
            float unused = 0.f;
            if (more) load_x_chunk(xn, row_ptr(tile_n), q_n, h, D);
            mfma_chunk_half<KB, false, false>(acc, x, lds + L.img, lds_mu, q, lane, c.scale, xsq, dsq, unused, 4);
        }
        if (q == NC - 1) {
            const float x2 = xsq + __shfl_xor(xsq, 32, kWave), norm = sqrtf(x2) * 1.001f;
            const float e = mfma_bound_half<KB>(acc, reinterpret_cast<const unsigned *>(lds + L.waug), x2,
                                                dsq + __shfl_xor(dsq, 32, kWave), norm, c, lane);
            const int64_t row = tile * bt.rt + r;
            const bool valid = r < bt.rt && row < nrows;
            beam_select<KB>(acc, x2, norm, e, c, slack, lane, bt.next, bt.hops, Ln, valid, masks + (valid ? row : 0));
            init_acc<KB>(acc, lds_h, h);
            xsq = 0.f;
            dsq = 0.f;
        }
        tile = tile_n;
        q = q_n;
    };
    if constexpr (KB == 8) {
        for (int64_t i = 0; i < G; ++i) step(x, x, i + 1 < G);
    } else {
        float4 y[8];
        for (int64_t i = 0; i < G; i += 2) {
            step(x, y, i + 1 < G);
            if (i + 1 >= G) break;
            step(y, x, i + 2 < G);
        }
    }
}

// Scoring for dictionaries that do not fit LDS: the slices of k_assign_half_chunked (laid out by k_half_image).
template <int KB, bool EXACT>
__global__ __launch_bounds__(kAssignThreads) void k_beam_score_half_chunked(
    const float *__restrict__ rows, const float *__restrict__ hneg, const char *__restrict__ img, const float *__restrict__ sums,
    const float *__restrict__ negmu, int64_t N, int Lc, int Ln, int D, int K, int NC, float slack, BeamMask *__restrict__ masks)
{
    extern __shared__ float4 smem4[];
    char *lds = reinterpret_cast<char *>(smem4);
    const HalfLds L = half_lds(KB, NC, 2);
    constexpr int SLICE = KB * 4096;
    const int lane = lane_id(), wave = threadIdx.x >> 6, h = lane >> 5, r = lane & 31;
    const float *lds_h = reinterpret_cast<const float *>(lds + L.hneg);
    float *lds_mu = reinterpret_cast<float *>(lds + L.mu);
    const BeamTile bt(lane, Lc);
    const int64_t nrows = N * Lc;
    const int64_t ntiles = (nrows + bt.rt - 1) / bt.rt;
    const int64_t nbt = (ntiles + kAssignWaves - 1) / kAssignWaves;
    if ((int64_t)blockIdx.x >= nbt) return;
    // beam row this lane feeds for block tile i (idle lanes and waves re-read the last row)
    auto tile_row = [&](int64_t i, bool &valid) -> int64_t {
        const int64_t row = (i * kAssignWaves + wave) * bt.rt + r;
        valid = r < bt.rt && row < nrows;
        return valid ? row : nrows - 1;
    };
    bool valid;
    int64_t row = tile_row(blockIdx.x, valid);
    const float *xrow = rows + row * D;
    float4 x[8];
#pragma unroll
    for (int s = 0; s < 8; ++s) x[s] = *reinterpret_cast<const float4 *>(xrow + min(8 * s + 4 * h, last_piece(D)));
    for (int i = threadIdx.x; i < SLICE / 16; i += kAssignThreads)
        reinterpret_cast<uint4 *>(lds)[i] = reinterpret_cast<const uint4 *>(img)[i];
    for (int d = threadIdx.x; d < kChunkD * NC; d += kAssignThreads) lds_mu[d] = negmu[d];
    const int s = half_shift(hneg, K);
    const bool holder = (int)threadIdx.x < 32 * KB;
    const HalfConsts c = half_constants<KB>(lds, L, holder ? sums[2 * threadIdx.x] : 0.f, holder ? sums[2 * threadIdx.x + 1] : 0.f,
                                            threadIdx.x, holder, K, NC, ldexpf(1.f, s), ldexpf(1.f, -s));
    floatx16 acc[KB];
    float unused = 0.f;
    int par = 0;
    for (int64_t i = blockIdx.x; i < nbt; i += gridDim.x) {
        bool valid_n = valid;
        int64_t row_n = row;
        if (i + gridDim.x < nbt) row_n = tile_row(i + gridDim.x, valid_n);
        const float *xrow_n = rows + row_n * D;
        float xsq = 0.f, dsq = 0.f;
        init_acc<KB>(acc, lds_h, h);
#pragma unroll 1
        for (int q = 0; q < NC; ++q) {
            const bool last = q + 1 == NC;
            const int qn = last ? 0 : q + 1;
            mfma_slice_half_refill<KB, false, EXACT>(acc, x, lds + par * SLICE, lds + (par ^ 1) * SLICE, img + (size_t)qn * SLICE,
                                                     last ? xrow_n : xrow, lds_mu, q, qn, D, lane, c.scale, xsq, dsq, unused);
            __syncthreads();
            par ^= 1;
        }
        const float x2 = xsq + __shfl_xor(xsq, 32, kWave), norm = sqrtf(x2) * 1.001f;
        const float e = mfma_bound_half<KB>(acc, reinterpret_cast<const unsigned *>(lds + L.waug), x2, dsq + __shfl_xor(dsq, 32, kWave),
                                            norm, c, lane);
        beam_select<KB>(acc, x2, norm, e, c, slack, lane, bt.next, bt.hops, Ln, valid, masks + (valid ? row : 0));
        row = row_n;
        valid = valid_n;
        xrow = xrow_n;
    }
}

constexpr int kExpandChunk = 32;     // candidates evaluated and ranked at a time
constexpr int kExpandList = 512;     // candidates listed in LDS at a time

// (error, id) order of the candidates: smaller error first, equal errors by id = (l << 8) | k.
__device__ __forceinline__ bool beam_before(double ea, int ia, double eb, int ib)
{
    return (ea < eb) || (ea == eb && ia < ib);
}

// Exact evaluation and selection for one dictionary; one wave (a 64-thread block) per vector.
// The vector's marked candidates are listed in LDS (kExpandList at a time).  kExpandChunk at a time they
// are evaluated in fp64 in the direct form, four lanes per candidate, and land one per lane in
// lanes 0..31; lanes 32..63 hold the best Ln found so far.  Every lane counts how many of the
// others come before it in (error, l, k) order: that rank is its position, and ranks below Ln are
// the new best list (kept in LDS).  After the last chunk the list is the next beam: residual rows
// r_l - c(k) rounded to fp32, their fp64 errors, and the parent's code prefix extended by k.
//   rows_c [N*Lc] stride ldc -> rows_n [N*Ln] stride ldn;  pre_c [N][Lc][M] -> pre_n [N][Ln][M]
//   (bytes 0..m-1 copied, byte m = k);  err_n, parent, code: [N*Ln], each may be null.
__global__ __launch_bounds__(kWave) void k_beam_expand(
    const float *__restrict__ rows_c, int ldc, const BeamMask *__restrict__ masks,
    const float *__restrict__ Cm, int K, int D, int64_t N, int Lc, int Ln,
    const uint8_t *__restrict__ pre_c, uint8_t *__restrict__ pre_n, int M, int m,
    float *__restrict__ rows_n, int ldn, double *__restrict__ err_n,
    uint8_t *__restrict__ parent, uint8_t *__restrict__ code)
{
    __shared__ uint16_t list[kExpandList];
    __shared__ double win_e[kBeamMaxL];
    __shared__ int win_id[kBeamMaxL];
    const int lane = lane_id();
    const int d4n = D >> 2;
    // words of a vector: j = 8 l + 4 h + i; a lane takes j = lane + 64 t, so (h, i) is fixed per lane
    const int wh = (lane >> 2) & 1, wi = lane & 3;
    uint32_t vm = 0u;                                   // bits of real codewords (k < K)
    for (int p = 0; p < 32; ++p)
        if (64 * wi + 8 * (p >> 2) + 4 * wh + (p & 3) < K) vm |= 1u << p;
    const uint32_t *mw = reinterpret_cast<const uint32_t *>(masks);
    const int nwords = 8 * Lc;
    const double inf = __builtin_inf();
    const int none = 0x7fffffff;

    uint32_t Wn[4];                                      // bitmap words of the next vector, fetched ahead
#pragma unroll
    for (int t = 0; t < 4; ++t) {
        const int j = lane + 64 * t;
        Wn[t] = (j < nwords && (int64_t)blockIdx.x < N) ? mw[(size_t)blockIdx.x * nwords + j] : 0u;
    }
    for (int64_t n = blockIdx.x; n < N; n += gridDim.x) {
        uint32_t W[4];
        int cnt = 0;
        const int64_t nn = n + gridDim.x;
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            const int j = lane + 64 * t;
            W[t] = Wn[t] & vm;
            cnt += __popc(W[t]);
            Wn[t] = (j < nwords && nn < N) ? mw[(size_t)nn * nwords + j] : 0u;
        }
        int incl = cnt;
#pragma unroll
        for (int o = 1; o < kWave; o <<= 1) {
            const int y = __shfl_up(incl, o, kWave);
            if (lane >= o) incl += y;
        }
        const int total = __shfl(incl, kWave - 1, kWave);
        const int off = incl - cnt;                      // list position of the lane's first candidate
        if (lane < kBeamMaxL) { win_e[lane] = inf; win_id[lane] = none; }
        __syncthreads();

        int nwin = 0;                                    // entries of the best list so far
        for (int lbase = 0; lbase < total; lbase += kExpandList) {
        {   // list the candidates lbase .. lbase + kExpandList - 1 (any order: the ranking key is total)
            int at = off - lbase;
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                uint32_t bits = W[t];
                const int l = (lane + 64 * t) >> 3;
                while (bits) {
                    const int p = __ffs(bits) - 1;
                    bits &= bits - 1;
                    if (at >= 0 && at < kExpandList)
                        list[at] = (uint16_t)((l << 8) | (64 * wi + 8 * (p >> 2) + 4 * wh + (p & 3)));
                    ++at;
                }
            }
        }
        __syncthreads();
        const int nl = min(kExpandList, total - lbase);
        for (int base = 0; base < nl; base += kExpandChunk) {
            const int nc = min(kExpandChunk, nl - base);
            // evaluate: pass p covers candidates base + 16 p + (lane >> 2), four lanes each
            double e_mine = inf;
            int id_mine = none;
#pragma unroll 1
            for (int p = 0; p < 2; ++p) {
                if (16 * p >= nc) break;                 // uniform
                const int c = 16 * p + (lane >> 2);
                const int ent = (c < nc) ? (int)list[base + c] : 0;
                const float4 *a = reinterpret_cast<const float4 *>(rows_c + ((size_t)n * Lc + (ent >> 8)) * ldc);
                const float4 *b = reinterpret_cast<const float4 *>(Cm + (size_t)(ent & 255) * D);
                double s0 = 0.0, s1 = 0.0;
                auto term = [&](const float4 &u, const float4 &v) {
                    const double t0 = (double)u.x - (double)v.x, t1 = (double)u.y - (double)v.y;
                    const double t2 = (double)u.z - (double)v.z, t3 = (double)u.w - (double)v.w;
                    s0 = fma(t0, t0, s0);
                    s1 = fma(t1, t1, s1);
                    s0 = fma(t2, t2, s0);
                    s1 = fma(t3, t3, s1);
                };
                int d = lane & 3;
                for (; d + 12 < d4n; d += 16) {          // four float4 pairs in flight per lane
                    const float4 u0 = a[d], u1 = a[d + 4], u2 = a[d + 8], u3 = a[d + 12];
                    const float4 v0 = b[d], v1 = b[d + 4], v2 = b[d + 8], v3 = b[d + 12];
                    term(u0, v0);
                    term(u1, v1);
                    term(u2, v2);
                    term(u3, v3);
                }
                for (; d < d4n; d += 4) term(a[d], b[d]);
                double s = s0 + s1;
                s += __shfl_xor(s, 1, kWave);
                s += __shfl_xor(s, 2, kWave);
                if (!(s == s)) s = inf;                  // non-finite input sorts last
                // candidate 16 p + q sits in lanes 4 q .. 4 q + 3; bring it to lane 16 p + q
                const double sq = __shfl(s, 4 * (lane & 15), kWave);
                const int iq = __shfl(ent, 4 * (lane & 15), kWave);
                if ((lane >> 4) == p && lane < nc) { e_mine = sq; id_mine = iq; }
            }
            if (lane >= 32) {                            // the best so far
                const int i = lane - 32;
                if (i < nwin) { e_mine = win_e[i]; id_mine = win_id[i]; }
            }
            __syncthreads();                             // win_* read before it is rewritten
            // rank among the nc new candidates and the nwin kept ones
            int rank = 0;
            for (int j = 0; j < nc; ++j) {
                const double ej = __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(e_mine), j),
                                                   __builtin_amdgcn_readlane(__double2loint(e_mine), j));
                const int ij = __builtin_amdgcn_readlane(id_mine, j);
                rank += beam_before(ej, ij, e_mine, id_mine) ? 1 : 0;
            }
            for (int j = 32; j < 32 + nwin; ++j) {
                const double ej = __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(e_mine), j),
                                                   __builtin_amdgcn_readlane(__double2loint(e_mine), j));
                const int ij = __builtin_amdgcn_readlane(id_mine, j);
                rank += beam_before(ej, ij, e_mine, id_mine) ? 1 : 0;
            }
            const bool live = (lane < nc) || (lane >= 32 && lane - 32 < nwin);
            if (live && rank < Ln) { win_e[rank] = e_mine; win_id[rank] = id_mine; }
            nwin = min(Ln, nwin + nc);
            __syncthreads();
        }
        }

        // the next beam: eight rows per pass, eight lanes each
        const int sub = lane & 7;
        for (int i0 = 0; i0 < Ln; i0 += 8) {
            const int i = i0 + (lane >> 3);
            if (i < Ln) {
                int id = win_id[i];
                if (id == none) id = 0;                  // fewer candidates than Ln: non-finite input only
                const int l = id >> 8, k = id & 255;
                const size_t src = (size_t)n * Lc + l, slot = (size_t)n * Ln + i;
                const float4 *a = reinterpret_cast<const float4 *>(rows_c + src * ldc);
                const float4 *b = reinterpret_cast<const float4 *>(Cm + (size_t)k * D);
                float4 *o = reinterpret_cast<float4 *>(rows_n + slot * ldn);
                int d = sub;
                for (; d + 24 < d4n; d += 32) {
                    const float4 u0 = a[d], u1 = a[d + 8], u2 = a[d + 16], u3 = a[d + 24];
                    const float4 v0 = b[d], v1 = b[d + 8], v2 = b[d + 16], v3 = b[d + 24];
                    o[d] = make_float4(u0.x - v0.x, u0.y - v0.y, u0.z - v0.z, u0.w - v0.w);
                    o[d + 8] = make_float4(u1.x - v1.x, u1.y - v1.y, u1.z - v1.z, u1.w - v1.w);
                    o[d + 16] = make_float4(u2.x - v2.x, u2.y - v2.y, u2.z - v2.z, u2.w - v2.w);
                    o[d + 24] = make_float4(u3.x - v3.x, u3.y - v3.y, u3.z - v3.z, u3.w - v3.w);
                }
                for (; d < d4n; d += 8) {
                    const float4 u = a[d], v = b[d];
                    o[d] = make_float4(u.x - v.x, u.y - v.y, u.z - v.z, u.w - v.w);
                }
                if (pre_n) {
                    for (int j = sub; j < m; j += 8) pre_n[slot * M + j] = pre_c[src * M + j];
                    if (sub == 0) pre_n[slot * M + m] = (uint8_t)k;
                }
                if (sub == 0) {
                    if (err_n) err_n[slot] = win_e[i];
                    if (parent) parent[slot] = (uint8_t)l;
                    if (code) code[slot] = (uint8_t)k;
                }
            }
        }
        __syncthreads();                                 // list and win_* are reused by the next vector
    }
}

}  // namespace hclae
