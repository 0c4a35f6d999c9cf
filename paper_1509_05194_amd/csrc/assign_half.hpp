// Nearest-codeword assignment (Sec. 3.1/3.2; the per-dictionary step of Eq. 3 with one path) whose scores come from the
// fp16 matrix cores (v_mfma_f32_32x32x16_f16, 16 times the rate of the fp32 MFMA on gfx950) and whose decisions are
// those of fp64.
//
//   argmin_k ||x - c_k||^2 = argmax_k ( (x - mu).(c_k - mu) - ||c_k - mu||^2 / 2 )          for any mu
//
// The scores only pre-select.  Both operands, centred on mu (the mean of a few codewords) and scaled by a power of two,
// are rounded to fp16; what that rounding can do to a score is bounded by norms that are MEASURED, per vector and per
// codeword, and every codeword whose score can still be the best within its own bound is a candidate.  One candidate: it
// is the nearest codeword, whatever the rounding did.  Several: the wave itself decides among them from the fp32 data, with
// direct-form distances (decide_items).  The codes are therefore fp64 direct-form decisions on the fp32 data, the same
// ones an fp32 contraction with its own (narrower) margin leads to.
//
// Bound on the score of codeword k, in the scaled and centred units X, C (X^, C^ the fp16 values that enter the product):
//   |X.C_k - X^.C^_k| <= ||X - X^|| ||C^_k|| + ||X|| ||C_k - C^_k||  (rounding)
//                      + A (max||C||^2/2 + ||X|| ||C^_k|| + t (||X|| + max||C||) + t^2)   (accumulation),
// A = (D/16 + 3) 17 2^-23, t = 2^-14.  The rounding part is measured and rigorous.  The accumulation part holds if an MFMA, which
// adds 16 exact products and the accumulator, loses no more than 17 addends do when each is truncated to 24 bits of the largest,
// where a product counts as if its factors were not below fp16's smallest normal number t (subnormal ones are aligned so).  No
// document says that; measured on an MI355X over random and adversarial sums it loses less than a quarter of it.  With w_k >= ||C_k||, rho = max ||C_k - C^_k|| / w_k:
//   E_k = e w_k + h,   e = ||X - X^|| (1 + rho) + ||X|| (rho + A (1 + rho)),   h = A (max||C||^2/2 + t (||X|| + max||C||) + t^2).
// The matrix cores add e w_k themselves, as one more dimension of the product (X^: e, C^: w_k, both rounded up), so that the
// accumulators end with U_k, U_k + h an upper bound of the true score; the best one's lower bound is U - 2 e w - h.
// Per-codeword bounds instead of the largest norm for all leave a third of the undecided vectors (SIFT-shaped data, later
// stages: 1.5 % instead of 4.5 %).
#pragma once
#include "assign.hpp"

namespace hclae {

typedef _Float16 halfx8 __attribute__((ext_vector_type(8)));
typedef _Float16 halfx4 __attribute__((ext_vector_type(4)));
typedef _Float16 halfx2 __attribute__((ext_vector_type(2)));
typedef float floatv2 __attribute__((ext_vector_type(2)));

constexpr int kHalfStep = 16;                       // dims per fp16 MFMA
constexpr int kWaveMoved = 128;                     // vectors that changed cluster a wave keeps before it lists them
constexpr int kRefineLanes = 4;                     // lanes that share an undecided vector in the fp64 decision
// Candidates in one word of an undecided vector's bitmap (32 codewords, 16 of the smallest dictionaries) from which it is scored
// again in fp32 (rescore_items): six are rare with fewer than some 16 in all, and a look at the words costs no exchange.  The fp32
// bound grows with D, and for long rows it leaves out little unless fp16 said nothing.
__host__ __device__ constexpr int rescore_from(int kb, int D) { return D <= 256 ? 6 : kb == 1 ? 13 : 24; }
constexpr int kMuRows = 8;                          // codewords whose mean centres the scores
constexpr float kHalfMaxNorm = 64000.f;             // a scaled row beyond this may not fit fp16: all codewords are candidates

// One undecided vector: its candidates (bit p of mask[h][i] is codeword 64 i + 8 (p >> 2) + 4 h + (p & 3)), a lower bound
// on the distance to every codeword that is not among them, and the code it had.
struct HalfItem {
    uint32_t mask[2][4];
    uint32_t n, old;
    float lrest;
    uint32_t pad;
};

// Every block lists its undecided vectors in a stretch of its own of one array in global memory, 32 per tile of its share; entries the
// array needs for launches over at most N vectors with at most `waves` waves: a wave's share is rounded up to whole tiles,
// ceil(N / 32 / waves) of them, which leaves less than a tile per wave unused.
__host__ __device__ constexpr int64_t half_list_entries(int64_t N, int64_t waves) { return N + (waves + 1) * kTileVec; }
// Blocks of k_assign_half over N vectors: with few tiles, four each (one per SIMD).  k_assign_half_chunked, whose blocks take eight tiles
// at once, never has more.
__host__ __device__ constexpr int64_t half_blocks(int64_t N, int cus)
{
    const int64_t blocks = ((N + kTileVec - 1) / kTileVec + 3) / 4;
    return blocks < cus ? blocks : cus;
}

// Which tile a block of k_assign_half takes in its slot-th place (wave w has the places w, w + 8, ...).  ls < 0: tiles in order over the
// blocks, so that with few of them every block has one before any has two.  ls >= 0: so within each XCD, and a stretch of 2^ls tiles
// belongs to the XCD whose row-pass blocks take those rows (blocks go round the eight XCDs in order): what the pass left in that L2 is
// read from there, and the other way round.  A chunk of the online learner, D = 128, us in order / so: N = 49k, K = 20 534 / 466, K = 256
// 752 / 702; N = 1M, K = 256, beyond the L2s, 4596 / 4593; encoding N = 60k, D = 192, K = 256 438 / 406.
__host__ __device__ constexpr int half_tile(int block, int slot, int grid, int ls)
{
    if (ls < 0) return block + grid * slot;
    const int i = slot * (grid >> 3) + (block >> 3);
    return ((((i >> ls) << 3) | (block & 7)) << ls) | (i & ((1 << ls) - 1));
}
// Tiles below ntiles among the places of a wave.
__host__ __device__ constexpr int half_tiles_of(int block, int wave, int ntiles, int grid, int ls)
{
    int first = block + grid * wave, end = ntiles, step = grid;
    if (ls >= 0) {
        const int rounds = ntiles >> (ls + 3), rest = ntiles - (rounds << (ls + 3)) - ((block & 7) << ls);
        step = grid >> 3;
        first = wave * step + (block >> 3);
        end = (rounds << ls) + (rest < 0 ? 0 : rest < (1 << ls) ? rest : 1 << ls);      // tiles of the block's XCD
    }
    step *= kAssignWaves;
    return first < end ? (end - first + step - 1) / step : 0;
}
// No block has more tiles than this.
__host__ __device__ constexpr int half_share(int ntiles, int grid, int ls)
{
    if (ls < 0) return (ntiles + grid - 1) / grid;
    const int step = grid >> 3;
    return ((((ntiles >> (ls + 3)) + 1) << ls) + step - 1) / step;
}
// ls of a launch: with a block on every CU, if a stretch is no larger than half a round of blocks (half_list_entries has room for the
// tiles that one XCD may have more than another).  pass_rows: consecutive rows that a block of the row pass takes.
__host__ __device__ constexpr int half_order(int grid, int cus, int pass_rows)
{
    if (grid != cus || grid % 8 || pass_rows < kTileVec || 2 * (pass_rows / kTileVec) > grid) return -1;
    int ls = 0;
    while ((2 << ls) * kTileVec <= pass_rows) ++ls;
    return ls;
}

// LDS of the kernels: the fp16 dictionary (or two slices of it), then per-codeword constants, mu, and the waves' buffers.
struct HalfLds {
    int img, hneg, w, waug, mu, moved, misc, open, total;   // byte offsets
};
// slices: 64-dim slices of the dictionary held at a time (all nc of them, or the two of k_assign_half_chunked).
__host__ __device__ constexpr HalfLds half_lds(int kb, int nc, int slices)
{
    HalfLds l = {};
    l.img = 0;
    l.hneg = kb * slices * 4096;                    // 32 kb rows of 64 halves per slice
    l.w = l.hneg + 32 * kb * 4;
    l.waug = l.w + 32 * kb * 4;
    l.mu = l.waug + 64 * kb * 4;
    l.moved = l.mu + 64 * nc * 4;
    l.misc = l.moved + kAssignWaves * kWaveMoved * 8;
    l.open = l.misc + 128;
    l.total = l.misc + 256;
    return l;
}

// Constants of a dictionary in scaled and centred units.
struct HalfConsts {
    float scale, inv;                               // 2^s, 2^-s
    float h, rho, acc;                              // h but for its term in ||X||, max ||C_k - C^_k|| / w_k, A
    float cmax;                                     // max ||C||
    float hx;                                       // what a unit of ||X|| adds to h, and to what the index bits do to a key (decide_half)
};

__device__ __forceinline__ float uniform(float v) { return __uint_as_float(__builtin_amdgcn_readfirstlane(__float_as_uint(v))); }

// Constants the compiler does not see through: with a literal -1 it splits the mixed-precision fma below into a conversion
// and a subtraction, and a median with a literal infinity becomes a maximum, before which it quiets NaNs one by one.
__device__ __forceinline__ float opaque(float v)
{
    int b = (int)__float_as_uint(v);
    asm("" : "+s"(b));
    return __uint_as_float((unsigned)b);
}

// Rounds four scaled, centred coordinates to fp16; adds their squares and the squares of what the rounding left out.
__device__ __forceinline__ halfx4 half4(const float4 &v, float &sq, float &dsq)
{
    const halfx2 a = __builtin_convertvector((floatv2){v.x, v.y}, halfx2);
    const halfx2 b = __builtin_convertvector((floatv2){v.z, v.w}, halfx2);
    const float m1 = opaque(-1.f);                   // one mixed-precision fma each: the remainder of a rounding is exact
    const float dx = fmaf((float)a.x, m1, v.x), dy = fmaf((float)a.y, m1, v.y);
    const float dz = fmaf((float)b.x, m1, v.z), dw = fmaf((float)b.y, m1, v.w);
    sq = fmaf(v.x, v.x, sq);
    sq = fmaf(v.y, v.y, sq);
    sq = fmaf(v.z, v.z, sq);
    sq = fmaf(v.w, v.w, sq);
    dsq = fmaf(dx, dx, dsq);
    dsq = fmaf(dy, dy, dsq);
    dsq = fmaf(dz, dz, dsq);
    dsq = fmaf(dw, dw, dsq);
    return (halfx4){a.x, a.y, b.x, b.y};
}

__device__ __forceinline__ float4 scaled(const float4 &v, float scale, const float4 &negmu)
{
    return make_float4(fmaf(v.x, scale, negmu.x), fmaf(v.y, scale, negmu.y), fmaf(v.z, scale, negmu.z), fmaf(v.w, scale, negmu.w));
}

// The exponent of half_shift for a largest ||c||^2/2.
__device__ __forceinline__ int half_exponent(float h)
{
    if (!(h > 0.f) || !(h < __builtin_inff())) return 0;
    int e;
    (void)frexpf(sqrtf(2.f * h), &e);
    const int s = 7 - e;
    return s < -100 ? -100 : s > 100 ? 100 : s;
}

// w_k of a codeword from its squares: its norm, with a floor for one near mu, so that rho stays that of ordinary rounding.
__device__ __forceinline__ float half_floor(float sq, float cmax) { return fmaxf(sqrtf(sq) * 1.001f, cmax * 0.00390625f); }

// Its share of rho: the measured rounding, and that of the scaled and centred fp32 values themselves (2^-24 of them).  The sums
// of squares are chains of at most 4 NC terms per lane and a few additions: relative error below 2^-10 for any D allowed.
__device__ __forceinline__ float half_rho(float dsq, float wk, float cmax)
{
    return cmax > 0.f ? (sqrtf(dsq) * 1.001f + wk * 1.2e-7f) / wk : 0.f;
}

// A: two units more than the MFMAs, for the norms and for the index bits in a score (decide_half).  A unit is what one of them
// may lose of the largest magnitude it adds.
constexpr float kHalfAccUnit = 17.f * 1.1920929e-7f;
__device__ __forceinline__ float half_acc(int NC) { return (float)(4 * NC + 3) * kHalfAccUnit; }

// h of a dictionary without its term in ||X||, from the largest ||C||^2 and a bound of the largest ||C||.
__device__ __forceinline__ float half_loss(float acc, float hm, float cmax) { return acc * (0.501f * hm + 6.2e-5f * cmax + 3.8e-9f); }

__device__ __forceinline__ float half_loss_x(float acc, float cmax) { return acc * 6.2e-5f + 2.1e-6f * cmax; }

// w_k rounded up to fp16: to nearest of 1.002 w and a spacing of the subnormal numbers.
__device__ __forceinline__ _Float16 half_up(float wk) { return (_Float16)(wk * 1.002f + 6e-8f); }

// e of a vector, rounded up to fp16 (to nearest of 1.002 e), and not below its smallest normal number.
__device__ __forceinline__ float half_bound(float x2, float dsq, float xn, const HalfConsts &c)
{
    const float dx = sqrtf(dsq) * 1.001f + xn * 1.2e-7f;
    const float e = fmaxf((dx * (1.f + c.rho) + xn * (c.rho + c.acc * (1.f + c.rho))) * 1.002f, 6.2e-5f);
    return (float)(_Float16)e;
}

// Power of two that brings the largest codeword norm into [2^6, 2^7): rows up to 1000 times that norm stay in fp16's
// range, and coordinates down to 2^-20 of it are normal numbers.  Every wave computes the same value; all its lanes take part.
__device__ __forceinline__ int half_shift(const float *__restrict__ hneg, int K)
{
    float h = 0.f;
    for (int k = lane_id(); k < K; k += kWave) h = fmaxf(h, -hneg[k]);
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) h = fmaxf(h, __shfl_xor(h, o, kWave));
    return half_exponent(h);
}

// Byte offset of the 16 bytes that lane (g, r) reads for k-step t (16 dims) of row block b: dims 16 t + 4 g .. + 3 and
// 16 t + 8 + 4 g .. + 3 of codeword 32 b + r.  The slot of a row is permuted within its kilobyte by (t, g), so that the
// stores of one row, which come from the lanes of a half wave, spread over the banks.
__device__ __forceinline__ int half_slot(int t, int g, int r) { return (32 * g + (r ^ ((t & 3) | (g << 2)))) * 16; }

// Sums NV values (a power of two, at most W) over groups of W lanes: NV - 1 exchanges for all of them, each halving the values
// a lane carries.  Lane i of the group ends with the total of value i (NV < W: the lanes that agree with it in their lowest
// bits too).
template <int NV, int W>
__device__ __forceinline__ float group_sums(float (&v)[NV])
{
    const int lane = lane_id();
#pragma unroll
    for (int o = NV / 2; o > 0; o >>= 1) {
#pragma unroll
        for (int i = 0; i < o; ++i) {
            float lo = v[i], hi = v[i + o];
            asm("" : "+v"(lo), "+v"(hi));                           // two values, not one array indexed by the lane
            const bool up = (lane & o) != 0;
            v[i] = (up ? hi : lo) + __shfl_xor(up ? lo : hi, o, kWave);
        }
    }
    float s = v[0];
#pragma unroll
    for (int o = NV; o < W; o <<= 1) s += __shfl_xor(s, o, kWave);
    return s;
}

// Constants of a dictionary from its codewords' sums: every thread brings the squares (sq) of a scaled, centred codeword and
// those of its rounding (dsq), or zeros; `holder` threads, one per row below 32 KB, write the row's entries.  Needs all
// threads of the block.
template <int KB>
__device__ __forceinline__ HalfConsts half_constants(
    char *lds, const HalfLds L, float sq, float dsq, int row, bool holder, int K, int NC, float scale, float inv)
{
    float *red = reinterpret_cast<float *>(lds + L.misc);
    const int wave = threadIdx.x >> 6;
    HalfConsts c;
    float hm = sq;
#pragma unroll
    for (int o = 1; o < kWave; o <<= 1) hm = fmaxf(hm, __shfl_xor(hm, o, kWave));
    if (lane_id() == 0) red[wave] = hm;
    __syncthreads();
#pragma unroll
    for (int i = 0; i < kAssignWaves; ++i) hm = fmaxf(hm, red[i]);
    c.cmax = sqrtf(hm) * 1.001f;
    const float wk = half_floor(sq, c.cmax);
    float rho = half_rho(dsq, wk, c.cmax);
    if (holder) {
        const bool real = row < K;
        const halfx2 up = {half_up(wk), (_Float16)0.f};
        reinterpret_cast<float *>(lds + L.hneg)[row] = real ? -0.5f * sq : -1e38f;   // finite: index bits in an infinity would be a NaN
        reinterpret_cast<float *>(lds + L.w)[row] = (float)up.x;
        unsigned *aug = reinterpret_cast<unsigned *>(lds + L.waug) + 64 * (row >> 5) + (row & 31);
        aug[0] = real ? __builtin_bit_cast(unsigned, up) : 0u;      // the operand of lane (0, r); lane (1, r) has zeros
        aug[32] = 0u;
    }
#pragma unroll
    for (int o = 1; o < kWave; o <<= 1) rho = fmaxf(rho, __shfl_xor(rho, o, kWave));
    if (lane_id() == 0) red[kAssignWaves + wave] = rho;
    __syncthreads();
#pragma unroll
    for (int i = 0; i < kAssignWaves; ++i) rho = fmaxf(rho, red[kAssignWaves + i]);
    __syncthreads();                                                // red is used again
    c.acc = half_acc(NC);
    // the same in every lane: scalar registers
    c.scale = uniform(scale);
    c.inv = uniform(inv);
    c.h = uniform(half_loss(c.acc, hm, c.cmax));
    c.rho = uniform(rho);
    c.cmax = uniform(c.cmax);
    c.hx = uniform(half_loss_x(c.acc, c.cmax));
    return c;
}

// Fills LDS with the dictionary (first D coordinates of rows of stride ld, zero beyond) and its constants.  A half wave
// takes a row: its loads are contiguous and its sums stay in the half wave.
template <int KB>
__device__ __forceinline__ HalfConsts stage_half(
    char *lds, const HalfLds L, const float *__restrict__ Cm, const float *__restrict__ hneg, int K, int D, int ld, int NC)
{
    constexpr int RP = 2 * KB;                                      // rows per half wave (512 threads)
    const int l32 = threadIdx.x & 31, hw = threadIdx.x >> 5;
    float *lds_mu = reinterpret_cast<float *>(lds + L.mu);
    float scale = 1.f, inv = 1.f;
    float sums[2 * RP];                                             // per row: squares, squares of the rounding
#pragma unroll
    for (int i = 0; i < 2 * RP; ++i) sums[i] = 0.f;
    for (int p0 = 0; p0 < 16 * NC; p0 += 32) {                      // all lanes stay: half_shift exchanges between them
        const int p = p0 + l32;
        float4 v[RP];
#pragma unroll
        for (int i = 0; i < RP; ++i) v[i] = load_row_piece(Cm, hw + 16 * i, 4 * p, K, D, ld);
        float4 mu = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
        for (int i = 0; i < kMuRows; ++i) {
            const float4 w = load_row_piece(Cm, (int)((unsigned)(i * K) / kMuRows), 4 * p, K, D, ld);
            mu.x += w.x;
            mu.y += w.y;
            mu.z += w.z;
            mu.w += w.w;
        }
        if (p0 == 0) {                                              // the loads above are on their way meanwhile
            const int s = half_shift(hneg, K);
            scale = ldexpf(1.f, s);
            inv = ldexpf(1.f, -s);
        }
        const float f = -scale / kMuRows;
        const float4 neg = make_float4(mu.x * f, mu.y * f, mu.z * f, mu.w * f);
        if (p >= 16 * NC) break;
        if (hw == 0) reinterpret_cast<float4 *>(lds_mu)[p] = neg;
        const int t = p >> 2, g = p & 1, hi = (p >> 1) & 1;
#pragma unroll
        for (int i = 0; i < RP; ++i) {
            const int row = hw + 16 * i;
            float4 w = scaled(v[i], scale, neg);
            if (row >= K) w = make_float4(0.f, 0.f, 0.f, 0.f);
            const halfx4 q = half4(w, sums[2 * i], sums[2 * i + 1]);
            *reinterpret_cast<halfx4 *>(lds + ((t * KB + (row >> 5)) * 1024 + half_slot(t, g, row & 31) + 8 * hi)) = q;
        }
    }
    // lane i: value i of its half wave, i.e. of row hw + 16 (i / 2) its squares (i even) or those of its rounding (i odd)
    const float mine = group_sums<2 * RP, 32>(sums);
    const float other = __shfl_xor(mine, 1, kWave);
    const int row = hw + 16 * ((l32 & (2 * RP - 1)) >> 1);
    const bool odd = (l32 & 1) != 0;
    return half_constants<KB>(lds, L, odd ? other : mine, odd ? mine : other, row, l32 < 2 * RP && !odd, K, NC, scale, inv);
}

// STEPS 16-dim steps of a tile's contraction.  base: LDS of the first step's operands (half_slot), of which all STEPS are there; live:
// steps that count (wave-uniform; the others are not contracted).  vec(t): the vectors' operand of step t; then(t)
// follows step t's MFMAs, and comes for the steps that do not count too.
// The dictionary's operands are read kAhead MFMAs ahead, in an order that the scheduler may not change: left to itself, with
// registers scarce, it reads each one right before its MFMA and waits out the latency of LDS 64 times a tile (pruned assignments of
// a training at N = 1M, D = 128, K = 256: 88 -> 82 us; 6 or 8 ahead are no faster).
constexpr int kAhead = 4;
template <int KB, int STEPS, typename Vec, typename Then>
__device__ __forceinline__ void contract_half(floatx16 (&acc)[KB], const char *base, int h, int r, int live, Vec vec, Then then)
{
    constexpr int n = STEPS * KB, P = kAhead < n ? kAhead : n;
    const char *slot[4];
#pragma unroll
    for (int t = 0; t < 4; ++t) slot[t] = base + half_slot(t, h, r);
    halfx8 a[P];
#pragma unroll
    for (int i = 0; i < P; ++i) a[i] = *reinterpret_cast<const halfx8 *>(slot[(i / KB) & 3] + i * 1024);
#pragma unroll
    for (int t = 0; t < STEPS; ++t) {
        if (t < live) {
            const halfx8 w = vec(t);
#pragma unroll
            for (int b = 0; b < KB; ++b) {
                const int i = t * KB + b;
                acc[b] = __builtin_amdgcn_mfma_f32_32x32x16_f16(a[i % P], w, acc[b], 0, 0, 0);
                if (i + P < n) a[i % P] = *reinterpret_cast<const halfx8 *>(slot[((i + P) / KB) & 3] + (i + P) * 1024);
                __builtin_amdgcn_sched_barrier(0x6);                // arithmetic may pass, MFMAs and memory not
            }
        }
        then(t);
    }
}

// One 64-dim chunk of a 32-vector tile: x as load_x_chunk leaves it (lane (g, r): dims 8 s + 4 g .. + 3 of row r for
// s = 0..7), so k-step t takes x[2t] and x[2t + 1].  steps: k-steps of the chunk that hold coordinates (PREFIX).
template <int KB, bool PREFIX, bool AMAX>
__device__ __forceinline__ void mfma_chunk_half(
    floatx16 (&acc)[KB], const float4 (&x)[8], const char *__restrict__ img, const float *__restrict__ negmu, int q, int lane,
    float scale, float &xsq, float &dsq, float &amax, int steps)
{
    constexpr int GB = KB < 4 ? KB : 4;              // codeword blocks whose operands are in registers at once
    const int g = lane >> 5, r = lane & 31;
    const float4 *mu4 = reinterpret_cast<const float4 *>(negmu) + 16 * q + g;
    const char *base = img + (size_t)q * 4 * KB * 1024;
#pragma unroll
    for (int t = 0; t < 4; ++t) {
        if (PREFIX && t >= steps) break;
        const float4 u = x[2 * t], v = x[2 * t + 1];
        if (AMAX) {
            amax = fmaxf(fmaxf(amax, fabsf(u.x)), fabsf(u.y));
            amax = fmaxf(fmaxf(amax, fabsf(u.z)), fabsf(u.w));
            amax = fmaxf(fmaxf(amax, fabsf(v.x)), fabsf(v.y));
            amax = fmaxf(fmaxf(amax, fabsf(v.z)), fabsf(v.w));
        }
        const char *at = base + half_slot(t, g, r);
        const halfx4 lo = half4(scaled(u, scale, mu4[4 * t]), xsq, dsq);
        const halfx4 hi = half4(scaled(v, scale, mu4[4 * t + 2]), xsq, dsq);
        const halfx8 w = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
#pragma unroll
        for (int b0 = 0; b0 < KB; b0 += GB) {
            halfx8 a[GB];
#pragma unroll
            for (int b = 0; b < GB; ++b) a[b] = *reinterpret_cast<const halfx8 *>(at + (t * KB + b0 + b) * 1024);
#pragma unroll
            for (int b = 0; b < GB; ++b) acc[b0 + b] = __builtin_amdgcn_mfma_f32_32x32x16_f16(a[b], w, acc[b0 + b], 0, 0, 0);
        }
    }
}

// A value of lane l and of lane l ^ 32: the low half's and the high half's.
__device__ __forceinline__ uint2 both_halves(unsigned v)
{
    const auto s = __builtin_amdgcn_permlane32_swap(v, v, false, false);
    return make_uint2(s[0], s[1]);
}
__device__ __forceinline__ int min_both(int v)
{
    const uint2 s = both_halves((unsigned)v);
    return min((int)s.x, (int)s.y);
}

// The largest of a lane's sixteen scores of a block, two a step (see block_key).
__device__ __forceinline__ float block_max(const floatx16 &a)
{
    float m = a[0];
#pragma unroll
    for (int v = 1; v < 15; v += 2) m = __builtin_elementwise_maximum(__builtin_elementwise_maximum(m, a[v]), a[v + 1]);
    return __builtin_elementwise_maximum(m, a[15]);
}

// The largest of a lane's sixteen scores of a block with its last four bits replaced by its index (2^-19 of it): two a step
// (v_maximum3; fmaxf would quiet NaNs one by one first).
__device__ __forceinline__ float block_key(const floatx16 &a)
{
    float m = -__builtin_inff();
#pragma unroll
    for (int v = 0; v < 16; v += 2) {
        const float x = __uint_as_float((__float_as_uint(a[v]) & ~15u) | (unsigned)v);
        const float y = __uint_as_float((__float_as_uint(a[v + 1]) & ~15u) | (unsigned)(v + 1));
        m = __builtin_elementwise_maximum(__builtin_elementwise_maximum(m, x), y);
    }
    return m;
}

// The best of a vector's scores on keys (mx) and its codeword, the same in both lanes that share the vector.
template <int KB>
__device__ __forceinline__ int best_half(const floatx16 (&acc)[KB], int h, int K, float &mx)
{
    mx = -__builtin_inff();
    int blk = 0;
#pragma unroll
    for (int b = 0; b < KB; ++b) {
        const float k = block_key(acc[b]);
        blk = k > mx ? b : blk;
        mx = __builtin_elementwise_maximum(mx, k);
    }
    const int v = (int)(__float_as_uint(mx) & 15u);
    const uint2 s = both_halves(__float_as_uint(mx)), k = both_halves((unsigned)(32 * blk + 8 * (v >> 2) + 4 * h + (v & 3)));
    const float lo = __uint_as_float(s.x), hi = __uint_as_float(s.y);
    mx = __builtin_elementwise_maximum(lo, hi);
    const int code = (int)(lo >= hi ? k.x : k.y);
    return code < K ? code : 0;                                     // beyond K only with non-finite input
}

// What a score may be off: h, what the index bits did to the best key, and what the subtraction of the threshold may lose of the larger
// of it and a score that is near it.
__device__ __forceinline__ float margin_half(const HalfConsts &c, float mx, float xn, float e)
{
    return fmaf(c.hx, xn, fmaf(4.3e-6f, fabsf(mx), fmaf(4.4e-6f * e, c.cmax, c.h))) + 1e-9f;
}

// Takes thr from every score, on the matrix cores: one more product of at most 4 terms, thr in three fp16 pieces of 11 bits (the
// remainders are exact, what they leave of thr is below 2^-33 of it and 2^-35).  |thr| < kHalfMaxThr.
constexpr float kHalfMaxThr = 6e7f;                 // 1024 times fp16's range, and some
template <int KB>
__device__ __forceinline__ void subtract_half(floatx16 (&acc)[KB], float thr, int h)
{
    const halfx4 one = h == 0 ? (halfx4){(_Float16)1024.f, (_Float16)1.f, (_Float16)0.0009765625f, (_Float16)0.f}
                              : (halfx4){(_Float16)0.f, (_Float16)0.f, (_Float16)0.f, (_Float16)0.f};
    const _Float16 a = (_Float16)(thr * -0.0009765625f);
    const float r = fmaf((float)a, -1024.f, -thr);
    const _Float16 b = (_Float16)r;
    const halfx4 w = {a, b, (_Float16)((r - (float)b) * 1024.f), (_Float16)0.f};
#pragma unroll
    for (int i = 0; i < KB; ++i) acc[i] = __builtin_amdgcn_mfma_f32_32x32x8f16(one, w, acc[i], 0, 0, 0);
}

// Scores that are not negative, as bitmap words of the lane's half of the codewords: the sign bits shifted into a word, an
// instruction per score.
template <int KB>
__device__ __forceinline__ void not_negative(uint32_t (&mk)[4], const floatx16 (&acc)[KB])
{
    mk[0] = mk[1] = mk[2] = mk[3] = 0u;
#pragma unroll
    for (int i = 0; i < (KB + 1) / 2; ++i) {
        uint32_t below = 0u;
#pragma unroll
        for (int v = KB == 1 ? 15 : 31; v >= 0; --v)
            below = __builtin_amdgcn_alignbit(below, __float_as_uint(acc[2 * i + (v >> 4)][v & 15]), 31);   // (below << 1) | sign
        mk[i] = KB == 1 ? ~below & 0xffffu : ~below;
    }
}

// Codewords whose score reaches thr, as bitmap words of the lane's half of them, without compare-and-select chains: the sign of
// score - threshold is shifted into a word (v_alignbit), two instructions per score.
template <int KB>
__device__ __forceinline__ void reaching(uint32_t (&mk)[4], const floatx16 (&acc)[KB], float thr)
{
    mk[0] = mk[1] = mk[2] = mk[3] = 0u;
#pragma unroll
    for (int b = 0; b < KB; ++b) {
        uint32_t below = 0u;
#pragma unroll
        for (int i = 15; i >= 0; --i)
            below = __builtin_amdgcn_alignbit(below, __float_as_uint(acc[b][i] - thr), 31);   // (below << 1) | sign
        mk[b >> 1] |= (~below & 0xffffu) << ((b & 1) * 16);
    }
}

// What a block has still to decide: the items are in global memory, these in LDS.
struct HalfOpen {
    unsigned items, many, hard;                     // items; one of them has many candidates; items left to fp64
};

// What a wave has to report (in LDS), and its block has still to decide.
struct HalfWave {
    HalfItem *items;                                // the block's
    HalfOpen *open;
    unsigned long long *moved;                      // [kWaveMoved]
    int nmoved;                                     // wave-uniform
};

// A barrier of the block comes between this and the first use of what it sets.
__device__ __forceinline__ HalfWave half_wave(char *lds, const HalfLds &L, HalfItem *items)
{
    HalfWave w;
    w.items = items;
    w.open = reinterpret_cast<HalfOpen *>(lds + L.open);
    w.moved = reinterpret_cast<unsigned long long *>(lds + L.moved) + (threadIdx.x >> 6) * kWaveMoved;
    w.nmoved = 0;
    if (threadIdx.x == 0) *w.open = HalfOpen{0u, 0u, 0u};
    return w;
}

// LDS of one wave: what its lanes wrote is there for all of them (LDS operations of a wave stay in order; this keeps the
// compiler from moving them).
__device__ __forceinline__ void wave_lds_fence()
{
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

// Hands the wave's moved vectors to the list in global memory: one counter add.
__device__ __forceinline__ void flush_moved(HalfWave &w, unsigned long long *__restrict__ list, unsigned *__restrict__ count)
{
    wave_lds_fence();
    unsigned base = 0;
    if (lane_id() == 0) base = atomicAdd(count, (unsigned)w.nmoved);
    base = __shfl(base, 0, kWave);
    for (int i = lane_id(); i < w.nmoved; i += kWave) list[base + i] = w.moved[i];
    w.nmoved = 0;
    wave_lds_fence();
}

// Lanes with `yes` report that vector n went from one codeword to another.
__device__ __forceinline__ void push_moved(HalfWave &w, bool yes, unsigned n, unsigned from, unsigned to,
                                           unsigned long long *__restrict__ list, unsigned *__restrict__ count)
{
    if (w.nmoved > kWaveMoved - kWave) flush_moved(w, list, count);
    const unsigned long long who = __ballot(yes);
    if (yes) {
        const int at = w.nmoved + __popcll(who & ((1ull << lane_id()) - 1ull));
        w.moved[at] = (unsigned long long)n | ((unsigned long long)from << 32) | ((unsigned long long)to << 40);
    }
    w.nmoved += __popcll(who);
}

// Narrows the candidates of up to 32 undecided vectors by scores from the fp32 matrix cores, whose bound is 2^-22 D of the
// magnitudes involved: data that lie far from their mean compared with what tells them apart (groups of clusters a long way from
// each other, codewords of very different norms, vectors beyond fp16's range) leave the fp16 scores tens of candidates a vector,
// and the direct form would pay for each of them.  Returns whether half of the candidates or more are left out.
// Bound: eps (max||c||^2/2 + ||x|| max||c||) is twice the rounding error of a score, D + 2 roundings of 2^-23 of the partial sums.
// Both operands come from memory, through caches that the other waves share.  Assignment of 200k vectors, D = 128, K = 256, us
// without / with: two groups 30 standard deviations apart 681 / 266, one codeword 100 times as long as the others 1010 / 660,
// codewords 10^-4 of the vectors 3178 / 253; where the fp32 bound says no more than the fp16 one (lognormal norms) 978 / 1014.
// A call, not inlined: few launches come here, and its registers would cost the others 5 to 10 % (N = 1M, D = 128, K = 256).
template <int KB, int PRUNE>
__device__ __attribute__((noinline)) bool rescore_items(
    HalfItem *items, int count, const float *__restrict__ xp, const float *__restrict__ Cm, const float *__restrict__ hneg,
    int D, int ld, int K, float slack_rel)
{
    const int lane = lane_id(), h = lane >> 5, r = lane & 31;
    HalfItem *it = items + (r < count ? r : 0);
    const float *xrow = xp + (size_t)it->n * ld;
    float hmax = 0.f;
    for (int k = lane; k < K; k += kWave) hmax = fmaxf(hmax, -hneg[k]);
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) hmax = fmaxf(hmax, __shfl_xor(hmax, o, kWave));
    floatx16 acc[KB];
    init_acc<KB>(acc, hneg, h);
    float x2 = 0.f;
#pragma unroll 1
    for (int c0 = 0; c0 < D; c0 += 8) {                             // rows of both operands straight from memory: the caches hold C
        const int col = c0 + 4 * h;
        const float4 x = col < D ? *reinterpret_cast<const float4 *>(xrow + col) : make_float4(0.f, 0.f, 0.f, 0.f);
        float4 a[KB];
#pragma unroll
        for (int b = 0; b < KB; ++b) a[b] = load_row_piece(Cm, 32 * b + r, col, K, D, ld);
        x2 = fmaf(x.x, x.x, x2);
        x2 = fmaf(x.y, x.y, x2);
        x2 = fmaf(x.z, x.z, x2);
        x2 = fmaf(x.w, x.w, x2);
#pragma unroll
        for (int b = 0; b < KB; ++b) {
            acc[b] = __builtin_amdgcn_mfma_f32_32x32x2f32(a[b].x, x.x, acc[b], 0, 0, 0);
            acc[b] = __builtin_amdgcn_mfma_f32_32x32x2f32(a[b].y, x.y, acc[b], 0, 0, 0);
            acc[b] = __builtin_amdgcn_mfma_f32_32x32x2f32(a[b].z, x.z, acc[b], 0, 0, 0);
            acc[b] = __builtin_amdgcn_mfma_f32_32x32x2f32(a[b].w, x.w, acc[b], 0, 0, 0);
        }
    }
    x2 += __shfl_xor(x2, 32, kWave);
    float mx = -__builtin_inff();
#pragma unroll
    for (int b = 0; b < KB; ++b)
#pragma unroll
        for (int v = 0; v < 16; ++v) mx = fmaxf(mx, acc[b][v]);
    mx = fmaxf(mx, __shfl_xor(mx, 32, kWave));
    const float eps = 2.02f * (float)(((D + kChunkD - 1) & ~(kChunkD - 1)) + 2) * 1.1920929e-7f;
    const float margin = eps * (hmax + sqrtf(x2) * sqrtf(2.f * hmax) * 1.000001f);
    const float thr = mx - margin;
    uint32_t mk[4];
    reaching<KB>(mk, acc, thr);
    const bool usable = fabsf(thr) < 1e37f;                         // else the sums may have left fp32's range
    uint32_t kept = 0u;                                             // codewords these scores keep and the fp16 scores did not
    int change = 0;
    if (r < count && usable) {
        uint4 *words = reinterpret_cast<uint4 *>(it->mask[h]);
        const uint4 was = *words;
        kept = (mk[0] & ~was.x) | (mk[1] & ~was.y) | (mk[2] & ~was.z) | (mk[3] & ~was.w);
        const uint4 now = make_uint4(was.x & mk[0], was.y & mk[1], was.z & mk[2], was.w & mk[3]);
        change = __popc(was.x) + __popc(was.y) + __popc(was.z) + __popc(was.w)
               - 2 * (__popc(now.x) + __popc(now.y) + __popc(now.z) + __popc(now.w));
        *words = now;
    }
    if (PRUNE) {
        // the codewords left out here have a true score <= out + margin / 2 (the evaluation of this line: see decide_half); those
        // that only the fp16 scores left out keep the bound those gave
        float out = -__builtin_inff();
#pragma unroll
        for (int b = 0; b < KB; ++b)
#pragma unroll
            for (int v = 0; v < 16; ++v) out = fmaxf(out, acc[b][v] < thr ? acc[b][v] : out);
        out = fmaxf(out, __shfl_xor(out, 32, kWave));
        kept |= (uint32_t)__shfl_xor((int)kept, 32, kWave);
        if (r < count && h == 0 && usable) {
            const float slack = slack_rel * (x2 + 2.f * fabsf(mx) + 2.f * fabsf(thr));
            const float l = sqrtf(fmaxf(0.f, (x2 - 2.f * (out + 0.5001f * margin)) - slack)) * 0.99999f;
            it->lrest = kept ? fminf(it->lrest, l) : l;
        }
    }
    __threadfence_block();
#pragma unroll
    for (int o = 1; o < kWave; o <<= 1) change += __shfl_xor(change, o, kWave);
    return change >= 0;
}

// Decides the block's items among their candidates; all its waves take part, eight lanes to an item, so that a block with few tiles
// (short lists, whose vectors are mostly undecided) is done after one round of gathers.
//
// First in fp32, direct form (after rescore_items where one has many candidates): the lanes share a row (contiguous pieces),
// two candidates at a time.  A sum of n non-negative terms accumulated in fp32 is within eta = (n + 6) 2^-24 of itself relatively,
// so where the best two are further apart than that, the smaller one is the nearest codeword.  What is left (exact and nearly exact
// ties) is decided in fp64: direct-form squared distances summed in ascending dimension order, smallest wins, exact ties go to the
// lowest index; kRefineLanes lanes share an item there and a lane takes one candidate at a time.
// PRUNE: the vector's bounds become these distances (the lower one limited by the bound on the codewords left out).
// Measured at N = 1M, D = 128, K = 256 with a fifth of the vectors undecided: 15 us of the kernel, 55 us with fp64 alone.
template <int KB, int PRUNE>
__device__ __forceinline__ void decide_items(
    HalfWave &w, const float *__restrict__ xp, const float *__restrict__ Cm, const float *__restrict__ hneg, int D, int ld, int K,
    int M, int m, uint8_t *__restrict__ codes, const PruneArgs &pa,
    unsigned long long *__restrict__ moved_list, unsigned *__restrict__ moved_count)
{
    __syncthreads();                                                // the items were written by all waves
    const int nitems = (int)w.open->items;
    if (!nitems) return;
    const int lane = lane_id(), wave = threadIdx.x >> 6;
    const int d4 = D >> 2;
    const bool want_moved = moved_list != nullptr;
    if (w.open->many) {
        for (int i0 = 32 * wave; i0 < nitems; i0 += 32 * kAssignWaves) {
            const HalfItem *it = w.items + min(i0 + (lane & 31), nitems - 1);
            const uint4 q = *reinterpret_cast<const uint4 *>(it->mask[lane >> 5]);
            const int most = max(max(__popc(q.x), __popc(q.y)), max(__popc(q.z), __popc(q.w)));
            if (!__ballot(most >= rescore_from(KB, D))) continue;
            if (!rescore_items<KB, PRUNE>(w.items + i0, min(32, nitems - i0), xp, Cm, hneg, D, ld, K, pa.slack)) break;
        }
        __syncthreads();
    }
    {
        const int sub = lane & 7, first = lane & 56;
        const int d4up = (D + 3) >> 2;
        const float eta = (float)(4 * ((d4up + 7) >> 3) + 6) * 6.1e-8f;
        for (int i0 = 8 * wave; i0 < nitems; i0 += 8 * kAssignWaves) {
            const bool live = i0 + (lane >> 3) < nitems;
            HalfItem *it = w.items + (live ? i0 + (lane >> 3) : 0);
            const unsigned n = it->n, old = it->old;
            const uint32_t word = it->mask[sub >> 2][sub & 3];
            const float lrest = it->lrest;                          // read before the branch: behind it, it costs a latency of its own
            uint32_t bits = live ? word : 0u;
            const float4 *x = reinterpret_cast<const float4 *>(xp + (size_t)n * ld);
            float best = __builtin_inff(), second = __builtin_inff();
            int kbest = 0;
            // next candidate of the lane's item, -1 when there is none; the same for its eight lanes
            auto next = [&]() {
                const unsigned have = (unsigned)(__ballot(bits != 0u) >> first) & 255u;
                const int src = have ? __ffs(have) - 1 : 0;
                const int p = __ffs(bits) - 1;
                const int k = __shfl(64 * (sub & 3) + 8 * (p >> 2) + 4 * (sub >> 2) + (p & 3), first + src, kWave);
                if (sub == src) bits &= bits - 1u;
                return have ? k : -1;
            };
            for (int round = 1; __ballot(bits != 0u); ++round) {
                const int k0 = next(), k1 = next();
                const float4 *c0 = reinterpret_cast<const float4 *>(Cm + (size_t)(k0 < 0 ? 0 : k0) * ld);
                const float4 *c1 = reinterpret_cast<const float4 *>(Cm + (size_t)(k1 < 0 ? 0 : k1) * ld);
                float s0 = 0.f, s1 = 0.f;
                auto term = [](float s, const float4 &u, const float4 &v) {
                    const float a = u.x - v.x, b = u.y - v.y, c = u.z - v.z, d = u.w - v.w;
                    return fmaf(d, d, fmaf(c, c, fmaf(b, b, fmaf(a, a, s))));
                };
                int d = sub;
                for (; d + 24 < d4; d += 32) {
                    float4 u[4], v[4], w[4];
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        u[i] = x[d + 8 * i];
                        v[i] = c0[d + 8 * i];
                        w[i] = c1[d + 8 * i];
                    }
                    __builtin_amdgcn_sched_barrier(0);              // twelve loads in flight: k_encode_rest takes twice as long with two
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        s0 = term(s0, u[i], v[i]);
                        s1 = term(s1, u[i], w[i]);
                    }
                }
                for (; d < d4; d += 8) {
                    const float4 u = x[d], v = c0[d], w = c1[d];
                    __builtin_amdgcn_sched_barrier(0);
                    s0 = term(s0, u, v);
                    s1 = term(s1, u, w);
                }
                if ((D & 3) && sub == (d4 & 7)) {                   // D need not be a multiple of 4
                    for (int d = 4 * d4; d < D; ++d) {
                        const float u = reinterpret_cast<const float *>(x)[d];
                        const float a = u - reinterpret_cast<const float *>(c0)[d], b = u - reinterpret_cast<const float *>(c1)[d];
                        s0 = fmaf(a, a, s0);
                        s1 = fmaf(b, b, s1);
                    }
                }
#pragma unroll
                for (int o = 1; o < 8; o <<= 1) {
                    s0 += __shfl_xor(s0, o, kWave);
                    s1 += __shfl_xor(s1, o, kWave);
                }
                if (k0 >= 0) {
                    second = s0 < best ? best : fminf(second, s0);
                    if (s0 < best) { best = s0; kbest = k0; }
                }
                if (k1 >= 0) {
                    second = s1 < best ? best : fminf(second, s1);
                    if (s1 < best) { best = s1; kbest = k1; }
                }
                // many candidates, and the two best of the first four cannot be told apart: codewords that are equal (a dictionary
                // of zeros, or one that counts in two dimensions only), left to fp64
                if (round == 2) {
                    int left = __popc(bits);
#pragma unroll
                    for (int o = 1; o < 8; o <<= 1) left += __shfl_xor(left, o, kWave);
                    if (left > 4 && !(best * (1.f + eta) < second * (1.f - eta))) bits = 0u;
                }
            }
            // (the second condition keeps underflow out: a sum this large has no denormal part that counts)
            const bool sure = best * (1.f + eta) < second * (1.f - eta) && second > 1e-25f;
            const bool lead = live && sub == 0;
            if (lead) it->pad = sure ? 0u : 1u;
            if (lead && !sure) atomicAdd(&w.open->hard, 1u);
            if (lead && sure) {
                codes[(size_t)n * M + m] = (uint8_t)kbest;
                if (PRUNE) {
                    pa.bu[n] = sqrtf(best * (1.f + eta)) * 1.000001f;
                    pa.bl[n] = fminf(sqrtf(second * (1.f - eta)) * 0.999999f, lrest);
                }
            }
            if (want_moved) push_moved(w, lead && sure && old != (unsigned)kbest, n, old, (unsigned)kbest, moved_list, moved_count);
        }
    }
    __syncthreads();
    if (!w.open->hard) return;
    const int sub = lane & (kRefineLanes - 1);
    constexpr int per = kWave / kRefineLanes;
    for (int i0 = per * wave; i0 < nitems; i0 += per * kAssignWaves) {
        const int e = i0 + lane / kRefineLanes;
        const HalfItem it = w.items[min(e, nitems - 1)];
        const bool live = e < nitems && it.pad;
        if (!__ballot(live)) continue;
        int total = 0;
#pragma unroll
        for (int i = 0; i < 8; ++i) total += __popc(it.mask[i >> 2][i & 3]);
        if (!live) total = 0;
        const float4 *x = reinterpret_cast<const float4 *>(xp + (size_t)it.n * ld);
        double best = __builtin_inf(), second = __builtin_inf();
        int kbest = 0x7fffffff;
        for (int j0 = sub; j0 < total; j0 += kRefineLanes) {
            int j = j0, k = 0;                                      // codeword of the j-th set bit
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                uint32_t bits = it.mask[i >> 2][i & 3];
                const int c = __popc(bits);
                if (j >= 0 && j < c) {
                    for (int q = 0; q < j; ++q) bits &= bits - 1;
                    const int p = __ffs(bits) - 1;
                    k = 64 * (i & 3) + 8 * (p >> 2) + 4 * (i >> 2) + (p & 3);
                    j = -1;
                } else if (j >= 0) {
                    j -= c;
                }
            }
            const float4 *c4 = reinterpret_cast<const float4 *>(Cm + (size_t)k * ld);
            double s = 0.0;
#pragma unroll 4
            for (int d = 0; d < d4; ++d) {                          // four rounds of loads in flight, additions in order
                const float4 a = x[d], b = c4[d];
                const double t0 = (double)a.x - (double)b.x, t1 = (double)a.y - (double)b.y;
                const double t2 = (double)a.z - (double)b.z, t3 = (double)a.w - (double)b.w;
                s += t0 * t0;
                s += t1 * t1;
                s += t2 * t2;
                s += t3 * t3;
            }
            for (int d = 4 * d4; d < D; ++d) {
                const double t = (double)reinterpret_cast<const float *>(x)[d] - (double)reinterpret_cast<const float *>(c4)[d];
                s += t * t;
            }
            if (s < best || (s == best && k < kbest)) { second = best; best = s; kbest = k; }
            else if (s < second) second = s;
        }
#pragma unroll
        for (int o = kRefineLanes / 2; o > 0; o >>= 1) {
            const double ob = __shfl_xor(best, o, kWave), os = __shfl_xor(second, o, kWave);
            const int ok = __shfl_xor(kbest, o, kWave);
            second = fmin(fmax(best, ob), fmin(second, os));
            if (ob < best || (ob == best && ok < kbest)) { best = ob; kbest = ok; }
        }
        const bool lead = live && sub == 0;
        if (lead) {
            codes[(size_t)it.n * M + m] = (uint8_t)kbest;
            if (PRUNE) {
                pa.bu[it.n] = (float)sqrt(best) * 1.000001f;
                pa.bl[it.n] = fminf((float)sqrt(second) * 0.999999f, it.lrest);
            }
        }
        if (want_moved) push_moved(w, lead && it.old != (unsigned)kbest, it.n, it.old, (unsigned)kbest, moved_list, moved_count);
    }
}

// Last step of a tile's contraction: the product's extra dimension.  Returns e, from the vector's norms.
template <int KB>
__device__ __forceinline__ float mfma_bound_half(
    floatx16 (&acc)[KB], const unsigned *__restrict__ waug, float x2, float dsq, float xn, const HalfConsts &c, int lane)
{
    const float e = half_bound(x2, dsq, xn, c);
    const halfx4 w = {(_Float16)e, (_Float16)0.f, (_Float16)0.f, (_Float16)0.f};
#pragma unroll
    for (int b = 0; b < KB; ++b) {
        const halfx2 u = __builtin_bit_cast(halfx2, waug[64 * b + lane]);
        const halfx4 a = {u.x, u.y, (_Float16)0.f, (_Float16)0.f};
        acc[b] = __builtin_amdgcn_mfma_f32_32x32x8f16(a, w, acc[b], 0, 0, 0);
    }
    return e;
}

// Decision for the wave's 32 vectors from their upper scores U_k.  old: the code the vector has now.
//
// The best score is found on keys that carry their index, because its w decides its lower bound (the largest w of its sixteen
// neighbours instead leaves 2.5 times as many vectors undecided).  The threshold is then taken from the scores by the matrix cores,
// so that the candidates are sign bits: one and a half instructions per score for the best, one for the bitmap and, where bounds are
// kept, half of one for the largest score left out (negative floats are smaller as integers the nearer they are to zero, and smaller
// than any that is not negative).  The second best on keys took one and a half more, and tiles with an undecided vector (nearly all)
// another two for the bitmap.
template <int KB, int PRUNE>
__device__ __forceinline__ void decide_half(
    floatx16 (&acc)[KB], float x2, float xn, float e, const HalfConsts &c, const float *__restrict__ lds_w, int lane,
    int n, int N, int D, int K, int M, int m, unsigned old, uint8_t *__restrict__ codes, const PruneArgs &pa, HalfWave &w,
    unsigned long long *__restrict__ moved_list, unsigned *__restrict__ moved_count)
{
    const int h = lane >> 5;
    float mx;
    const int code = best_half<KB>(acc, h, K, mx);
    const float hh = margin_half(c, mx, xn, e);
    const float low = mx - 2.f * e * lds_w[code] - hh;   // lower bound of the best one's true score
    const float thr = low - hh;                                     // candidates: U_k + h >= low
    const bool big = !(x2 < kHalfMaxNorm * kHalfMaxNorm && fabsf(thr) < kHalfMaxThr);   // may not fit fp16
    subtract_half<KB>(acc, thr, h);
    uint32_t mk[4];
    not_negative<KB>(mk, acc);
    float m2 = 0.f;                                                 // largest U_k below the threshold
    bool rest = false;                                              // there is one
    if (PRUNE) {
        int s = 0x7fffffff;
#pragma unroll
        for (int b = 0; b < KB; ++b)
#pragma unroll
            for (int v = 0; v < 16; v += 2) s = min(min(s, __float_as_int(acc[b][v])), __float_as_int(acc[b][v + 1]));
        s = min_both(s);
        rest = s < 0;
        m2 = thr + __int_as_float(s);
    }
    // a single candidate is the best one
    const uint2 count = both_halves((unsigned)(__popc(mk[0]) + __popc(mk[1]) + __popc(mk[2]) + __popc(mk[3])));
    const bool single = count.x + count.y == 1u;
    const bool amb = K > 1 && n < N && (big || !single);
    const bool mine = h == 0 && n < N;
    float lrest = __builtin_inff();                                 // lower bound on the distance to what is left out
    if (PRUNE) {
        // d^2 = ||X||^2 - 2 score.  slack covers the fp32 evaluation: x2 is a chain of D/2 fused multiply-adds per lane
        // (relative error <= (D/2 + 1) 2^-24, all terms positive), the rest a handful of roundings; pa.slack = (D/2 + 16) 2^-23.
        const float slack = pa.slack * (x2 + 2.f * fabsf(mx) + 2.f * fabsf(m2));
        const float out = m2 + fmaf(2.2e-6f, fabsf(m2), hh);        // the subtraction again, of a score far below the threshold
        if (rest && !big) lrest = sqrtf(fmaxf(0.f, (x2 - 2.f * out) - slack)) * 0.99999f * c.inv;
        if (mine && !amb) {
            // (a single codeword has no other one to be nearer than: settled for good)
            pa.bu[n] = K > 1 ? sqrtf(fmaxf(0.f, (x2 - 2.f * low) + slack)) * 1.00001f * c.inv : 0.f;
            pa.bl[n] = K > 1 ? lrest : __builtin_inff();
        }
    }
    if (mine && !amb) codes[(size_t)n * M + m] = (uint8_t)code;
    if (moved_list) push_moved(w, mine && !amb && old != (unsigned)code, (unsigned)n, old, (unsigned)code, moved_list, moved_count);
    const uint32_t who = (uint32_t)__ballot(amb && h == 0);
    if (!who) return;
    unsigned at = 0;
    if (lane == 0) at = atomicAdd(&w.open->items, (unsigned)__popc(who));
    at = __builtin_amdgcn_readfirstlane(at);
    constexpr int NW = (KB + 1) / 2;
    if (big) {
#pragma unroll
        for (int i = 0; i < NW; ++i) {
            uint32_t all = 0u;
#pragma unroll 1
            for (int p = 0; p < 32; ++p) all |= (64 * i + 8 * (p >> 2) + 4 * h + (p & 3) < K) ? 1u << p : 0u;
            mk[i] = all;
        }
    }
    if (amb) {
        HalfItem *it = w.items + at + __popc(who & ((1u << (lane & 31)) - 1u));
        if (h == 0) {
            it->n = (uint32_t)n;
            it->old = old;
            it->lrest = lrest;
        }
        *reinterpret_cast<uint4 *>(it->mask[h]) = make_uint4(mk[0], mk[1], mk[2], mk[3]);
    }
    const int most = max(max(__popc(mk[0]), __popc(mk[1])), max(__popc(mk[2]), __popc(mk[3])));
    if (amb && most >= rescore_from(KB, D)) w.open->many = 1u;
}

// End of a block: what its waves have left, with one atomic each: moved vectors, vectors decided again, max |x'|.
template <int PRUNE>
__device__ __forceinline__ void half_finish(
    char *lds, const HalfLds L, const HalfWave &w, float amax, unsigned *__restrict__ refine_count,
    unsigned long long *__restrict__ moved_list, unsigned *__restrict__ moved_count, unsigned long long *__restrict__ work)
{
    const int lane = lane_id(), wave = threadIdx.x >> 6;
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) amax = fmaxf(amax, __shfl_xor(amax, o, kWave));
    unsigned *tail = reinterpret_cast<unsigned *>(lds + L.misc);   // [8] moved, [8], [8] max, [1] base
    if (lane == 0) {
        tail[wave] = (unsigned)w.nmoved;
        tail[16 + wave] = __float_as_uint(amax);
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        unsigned nm = 0u, mxb = 0u;
        const unsigned nr = w.open->items;
        for (int i = 0; i < kAssignWaves; ++i) {
            nm += tail[i];
            mxb = max(mxb, tail[16 + i]);
        }
        if (nm) tail[24] = atomicAdd(moved_count, nm);
        if (nr) {
            atomicAdd(refine_count, nr);
            atomicAdd(work + 2, (unsigned long long)nr);
        }
        if (PRUNE != 2) atomicMax(refine_count + 1, mxb);           // of listed vectors nobody asks: it is known from the first pass
    }
    __syncthreads();
    if (w.nmoved) {
        unsigned at = tail[24];
        for (int i = 0; i < wave; ++i) at += tail[i];
        for (int i = lane; i < w.nmoved; i += kWave) moved_list[at + i] = w.moved[i];
    }
}

// Assignment with the whole dictionary resident in LDS as fp16 (half_lds within a workgroup's LDS: K <= 32 up to D = 2240, 64 up to 1152,
// 128 up to 576, 256 up to 256).  A wave owns tiles of 32 vectors, streams them from HBM into operand
// registers 64 dims at a time with the next chunk in flight, and keeps all 32 KB scores of a vector in accumulators.
template <int KB, int PRUNE, bool PREFIX>
__global__ __launch_bounds__(kAssignThreads) void k_assign_half(
    const float *__restrict__ xp, const float *__restrict__ Cm, const float *__restrict__ hneg,
    int N, int D, int ld, int K, int M, int m, int NC,
    uint8_t *__restrict__ codes, unsigned *__restrict__ refine_count, PruneArgs pa,
    unsigned long long *__restrict__ moved_list, unsigned *__restrict__ moved_count, unsigned long long *__restrict__ work,
    HalfItem *__restrict__ items, int ls)
{
    extern __shared__ float4 smem4[];
    char *lds = reinterpret_cast<char *>(smem4);
    const HalfLds L = half_lds(KB, NC, NC);
    const int lane = lane_id();
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);      // scalar, and the tile order with it: 469 -> 461 us, N = 8M, D = 32
    const int h = lane >> 5;
    const int r = lane & 31;
    const float *lds_h = reinterpret_cast<const float *>(lds + L.hneg);
    const float *lds_mu = reinterpret_cast<const float *>(lds + L.mu);
    const bool want_moved = moved_list != nullptr;

    // rows of this launch: all N vectors, or the listed ones (PRUNE 2; all in order when nearly all are listed)
    const int listed = PRUNE == 2 ? (int)*pa.active_count : N;
    const bool gather = PRUNE == 2 && listed < N - (N >> 5);
    const int rows = gather ? listed : N;
    const int ntiles = (int)(((unsigned)rows + kTileVec - 1) / kTileVec);
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        work[0] += 1ull;                                            // launches on one stream follow one another
        work[1] += (unsigned long long)listed;
    }
    if ((int)blockIdx.x >= ntiles) return;                      // no tile for any wave of this block

    if (PRUNE == 2) ls = -1;                                    // listed vectors lie anywhere
    const int t0 = half_tile(blockIdx.x, wave, gridDim.x, ls);
    HalfWave w = half_wave(lds, L, items + (size_t)half_share(ntiles, gridDim.x, ls) * kTileVec * blockIdx.x);
    const int my_tiles = half_tiles_of(blockIdx.x, wave, ntiles, gridDim.x, ls);
    const int64_t G = (int64_t)my_tiles * NC;                       // (tile, chunk) steps of this wave

    // vector behind column r of a tile; N (= "none") for the columns of the ragged tail
    auto vec_of = [&](int tile) -> int {
        const unsigned i = (unsigned)tile * kTileVec + r;
        if (i >= (unsigned)rows) return N;
        return gather ? (int)pa.active[i] : (int)i;
    };
    auto row_ptr = [&](int n) {
        if (n >= N) n = gather ? (int)pa.active[rows - 1] : N - 1;   // tail columns re-read the last row
        return xp + (size_t)n * ld;
    };

    float amax = 0.f;
    const int steps_last = PREFIX ? (D - kChunkD * (NC - 1) + kHalfStep - 1) / kHalfStep : 4;
    auto steps_of = [&](int qq) { return (PREFIX && qq == NC - 1) ? steps_last : 4; };
    int slot = wave, n = N;
    unsigned old = 0u;
    float4 xa[8], xb[8];
    if (G > 0) {                                                    // the first chunk travels while the dictionary is staged
        n = vec_of(t0);
        if (want_moved && n < N) old = codes[(size_t)n * M + m];
        load_x_chunk<PREFIX>(xa, row_ptr(n), 0, h, D, 2 * steps_of(0));
    }
    const HalfConsts c = stage_half<KB>(lds, L, Cm, hneg, K, D, ld, NC);
    if (G > 0) {
        floatx16 acc[KB];
        float xsq = 0.f, dsq = 0.f;
        int q = 0;
        init_acc<KB>(acc, lds_h, h);
        // one step: contract x (chunk q of the tile) while the next step's chunk travels into xn
        auto step = [&](float4 (&x)[8], float4 (&xn)[8], bool more) {
            int n_n = n;
            unsigned old_n = old;
            int q_n = q + 1;
            if (q_n == NC) {
                q_n = 0;
                slot += kAssignWaves;
                if (more) {
                    n_n = vec_of(half_tile(blockIdx.x, slot, gridDim.x, ls));
                    if (want_moved) old_n = n_n < N ? codes[(size_t)n_n * M + m] : 0u;
                }
            }
            if (more) load_x_chunk<PREFIX>(xn, row_ptr(n_n), q_n, h, D, 2 * steps_of(q_n));
            mfma_chunk_half<KB, PREFIX, PRUNE != 2>(acc, x, lds + L.img, lds_mu, q, lane, c.scale, xsq, dsq, amax, steps_of(q));
            if (q == NC - 1) {
                const float x2 = xsq + __shfl_xor(xsq, 32, kWave), norm = sqrtf(x2) * 1.001f;
                const float e = mfma_bound_half<KB>(acc, reinterpret_cast<const unsigned *>(lds + L.waug), x2,
                                                    dsq + __shfl_xor(dsq, 32, kWave), norm, c, lane);
                decide_half<KB, PRUNE>(acc, x2, norm, e, c, reinterpret_cast<const float *>(lds + L.w), lane, n, N, D, K, M, m, old, codes, pa, w, moved_list, moved_count);
                init_acc<KB>(acc, lds_h, h);                        // here and not where the next tile begins: dead until now
                xsq = 0.f;
                dsq = 0.f;
            }
            n = n_n;
            old = old_n;
            q = q_n;
        };
        for (int64_t g = 0; g < G; g += 2) {
            step(xa, xb, g + 1 < G);
            if (g + 1 >= G) break;
            step(xb, xa, g + 2 < G);
        }
    }
    decide_items<KB, PRUNE>(w, xp, Cm, hneg, D, ld, K, M, m, codes, pa, moved_list, moved_count);

    half_finish<PRUNE>(lds, L, w, amax, refine_count, moved_list, moved_count, work);
}

// The fp16 dictionary for k_assign_half_chunked, slice by slice in the order its LDS holds them, with the sums its
// constants come from.  A wave per row of the padded dictionary.
__global__ __launch_bounds__(256) void k_half_image(
    const float *__restrict__ Cm, const float *__restrict__ hneg, int K, int D, int ld, int kb, int NC,
    char *__restrict__ img, float *__restrict__ sums, float *__restrict__ negmu)
{
    const int lane = lane_id();
    const int row = blockIdx.x * 4 + (threadIdx.x >> 6);
    const float scale = ldexpf(1.f, half_shift(hneg, K));
    float sq = 0.f, dsq = 0.f;
    for (int p = lane; p < 16 * NC; p += kWave) {
        const float4 v = load_row_piece(Cm, row, 4 * p, K, D, ld);
        float4 mu = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
        for (int i = 0; i < kMuRows; ++i) {
            const float4 w = load_row_piece(Cm, (int)((unsigned)(i * K) / kMuRows), 4 * p, K, D, ld);
            mu.x += w.x;
            mu.y += w.y;
            mu.z += w.z;
            mu.w += w.w;
        }
        const float f = -scale / kMuRows;
        const float4 neg = make_float4(mu.x * f, mu.y * f, mu.z * f, mu.w * f);
        if (row == 0) reinterpret_cast<float4 *>(negmu)[p] = neg;
        float4 w = scaled(v, scale, neg);
        if (row >= K) w = make_float4(0.f, 0.f, 0.f, 0.f);
        const halfx4 q = half4(w, sq, dsq);
        const int t = p >> 2, g = p & 1, hi = (p >> 1) & 1;
        *reinterpret_cast<halfx4 *>(img + (size_t)(t * kb + (row >> 5)) * 1024 + half_slot(t, g, row & 31) + 8 * hi) = q;
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        sq += __shfl_xor(sq, o, kWave);
        dsq += __shfl_xor(dsq, o, kWave);
    }
    if (lane == 0) {
        sums[2 * row] = sq;
        sums[2 * row + 1] = dsq;
    }
}

// One 64-dim slice of k_assign_half_chunked: contracts x (the slice's chunk in registers) with the dictionary slice in `cur`
// and brings in what the next one needs: k-step t refills x[2t], x[2t + 1] from xnext as soon as it has converted them, and
// fetches a piece of the next dictionary slice at its start and stores it to `nxt` behind its MFMAs.
// EXACT: D is a multiple of 64.  Otherwise the refill clamps its addresses into the row and what lies past D is multiplied by
// zero at use (mu and the dictionary are zero there).
template <int KB, bool AMAX, bool EXACT>
__device__ __forceinline__ void mfma_slice_half_refill(
    floatx16 (&acc)[KB], float4 (&x)[8], const char *__restrict__ cur, char *__restrict__ nxt, const char *__restrict__ src,
    const float *__restrict__ xnext, const float *__restrict__ negmu, int q, int qn, int D, int lane, float scale,
    float &xsq, float &dsq, float &amax)
{
    constexpr int GB = KB < 4 ? KB : 4;
    constexpr int PIECES = KB * 256;                                // uint4 of a slice
    const int g = lane >> 5, r = lane & 31;
    const float4 *mu4 = reinterpret_cast<const float4 *>(negmu) + 16 * q + g;
    const float4 *xn4 = reinterpret_cast<const float4 *>(xnext + (EXACT ? kChunkD * qn + 4 * g : 0));
#pragma unroll
    for (int t = 0; t < 4; ++t) {
        const int at = t * kAssignThreads + (int)threadIdx.x;
        uint4 piece = make_uint4(0u, 0u, 0u, 0u);
        if ((t + 1) * kAssignThreads <= PIECES || (t * kAssignThreads < PIECES && at < PIECES)) piece = reinterpret_cast<const uint4 *>(src)[at];
        const float4 u = x[2 * t], v = x[2 * t + 1];
        float su = scale, sv = scale;
        if (EXACT) {
            x[2 * t] = xn4[4 * t];
            x[2 * t + 1] = xn4[4 * t + 2];
        } else {
            const int col = kChunkD * q + 16 * t + 4 * g, coln = kChunkD * qn + 16 * t + 4 * g;
            su = col < D ? scale : 0.f;
            sv = col + 8 < D ? scale : 0.f;
            x[2 * t] = *reinterpret_cast<const float4 *>(xnext + min(coln, last_piece(D)));
            x[2 * t + 1] = *reinterpret_cast<const float4 *>(xnext + min(coln + 8, last_piece(D)));
        }
        if (AMAX) {
            amax = fmaxf(fmaxf(amax, fabsf(u.x)), fabsf(u.y));
            amax = fmaxf(fmaxf(amax, fabsf(u.z)), fabsf(u.w));
            amax = fmaxf(fmaxf(amax, fabsf(v.x)), fabsf(v.y));
            amax = fmaxf(fmaxf(amax, fabsf(v.z)), fabsf(v.w));
        }
        const char *base = cur + half_slot(t, g, r);
        const halfx4 lo = half4(scaled(u, su, mu4[4 * t]), xsq, dsq);
        const halfx4 hi = half4(scaled(v, sv, mu4[4 * t + 2]), xsq, dsq);
        const halfx8 w = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
#pragma unroll
        for (int b0 = 0; b0 < KB; b0 += GB) {
            halfx8 a[GB];
#pragma unroll
            for (int b = 0; b < GB; ++b) a[b] = *reinterpret_cast<const halfx8 *>(base + (t * KB + b0 + b) * 1024);
#pragma unroll
            for (int b = 0; b < GB; ++b) acc[b0 + b] = __builtin_amdgcn_mfma_f32_32x32x16_f16(a[b], w, acc[b0 + b], 0, 0, 0);
        }
        // the store (and the wait for its load) stays behind the step's MFMAs
        __builtin_amdgcn_sched_barrier(0x10f);
        if ((t + 1) * kAssignThreads <= PIECES || (t * kAssignThreads < PIECES && at < PIECES)) reinterpret_cast<uint4 *>(nxt)[at] = piece;
    }
}

// The same assignment for dictionaries that do not fit LDS even as fp16: a block walks the D axis in 64-dim slices for every
// tile of 8 x 32 vectors, the accumulators persisting across slices.  Two LDS buffers hold the slice in use and the one
// being brought in from k_half_image's array, one barrier per slice; the refills run under the MFMAs, across tiles too.
template <int KB, int PRUNE, bool EXACT>
__global__ __launch_bounds__(kAssignThreads) void k_assign_half_chunked(
    const float *__restrict__ xp, const float *__restrict__ Cm, const float *__restrict__ hneg,
    const char *__restrict__ img, const float *__restrict__ sums, const float *__restrict__ negmu,
    int N, int D, int ld, int K, int M, int m, int NC,
    uint8_t *__restrict__ codes, unsigned *__restrict__ refine_count, PruneArgs pa,
    unsigned long long *__restrict__ moved_list, unsigned *__restrict__ moved_count, unsigned long long *__restrict__ work,
    HalfItem *__restrict__ items)
{
    extern __shared__ float4 smem4[];
    char *lds = reinterpret_cast<char *>(smem4);
    const HalfLds L = half_lds(KB, NC, 2);
    constexpr int SLICE = KB * 4096;
    const int lane = lane_id();
    const int wave = threadIdx.x >> 6;
    const int h = lane >> 5, r = lane & 31;
    const float *lds_h = reinterpret_cast<const float *>(lds + L.hneg);
    float *lds_mu = reinterpret_cast<float *>(lds + L.mu);

    const int listed = PRUNE == 2 ? (int)*pa.active_count : N;
    const bool gather = PRUNE == 2 && listed < N - (N >> 5);
    const int rows = gather ? listed : N;
    const int nbt = (int)(((unsigned)rows + kTileVec * kAssignWaves - 1) / (kTileVec * kAssignWaves));   // block tiles
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        work[0] += 1ull;                                            // launches on one stream follow one another
        work[1] += (unsigned long long)listed;
    }
    if ((int)blockIdx.x >= nbt) return;

    // vector this lane's column of block tile bt stands for; N (= "none") in the ragged tail
    auto vec_of = [&](int bt) -> int {
        const unsigned i = ((unsigned)bt * kAssignWaves + wave) * kTileVec + r;
        if (i >= (unsigned)rows) return N;
        return gather ? (int)pa.active[i] : (int)i;
    };
    auto row_ptr = [&](int n) {
        if (n >= N) n = gather ? (int)pa.active[rows - 1] : N - 1;  // tail columns re-read the last row
        return xp + (size_t)n * ld;
    };
    HalfWave w = half_wave(lds, L, items + (size_t)((nbt + gridDim.x - 1) / gridDim.x) * kTileVec * kAssignWaves * blockIdx.x);
    int n = vec_of(blockIdx.x);
    const float *xrow = row_ptr(n);
    unsigned old = moved_list && n < N ? codes[(size_t)n * M + m] : 0u;
    float4 x[8];
#pragma unroll
    for (int s = 0; s < 8; ++s) x[s] = *reinterpret_cast<const float4 *>(xrow + min(8 * s + 4 * h, last_piece(D)));

    // slice 0 (the same for every tile), mu and the constants
    for (int e = threadIdx.x; e < SLICE / 16; e += kAssignThreads)
        reinterpret_cast<uint4 *>(lds)[e] = reinterpret_cast<const uint4 *>(img)[e];
    for (int d = threadIdx.x; d < kChunkD * NC; d += kAssignThreads) lds_mu[d] = negmu[d];
    const int s = half_shift(hneg, K);
    const bool holder = (int)threadIdx.x < 32 * KB;
    const HalfConsts c = half_constants<KB>(lds, L, holder ? sums[2 * threadIdx.x] : 0.f, holder ? sums[2 * threadIdx.x + 1] : 0.f,
                                            threadIdx.x, holder, K, NC, ldexpf(1.f, s), ldexpf(1.f, -s));

    floatx16 acc[KB];
    float amax = 0.f;
    int par = 0;
    for (int bt = blockIdx.x; bt < nbt; bt += gridDim.x) {
        int n_n = n;
        const float *xrow_n = xrow;                                 // the last tile refills with itself: unused
        unsigned old_n = old;
        if (bt + (int)gridDim.x < nbt) {
            n_n = vec_of(bt + gridDim.x);
            xrow_n = row_ptr(n_n);
            if (moved_list) old_n = n_n < N ? codes[(size_t)n_n * M + m] : 0u;
        }
        float xsq = 0.f, dsq = 0.f;
        init_acc<KB>(acc, lds_h, h);
#pragma unroll 1
        for (int q = 0; q < NC; ++q) {
            const bool last = q + 1 == NC;
            const int qn = last ? 0 : q + 1;
            mfma_slice_half_refill<KB, PRUNE != 2, EXACT>(acc, x, lds + par * SLICE, lds + (par ^ 1) * SLICE, img + (size_t)qn * SLICE,
                                                   last ? xrow_n : xrow, lds_mu, q, qn, D, lane, c.scale, xsq, dsq, amax);
            __syncthreads();                                        // slice q consumed by all, slice qn complete
            par ^= 1;
        }
        const float x2 = xsq + __shfl_xor(xsq, 32, kWave), norm = sqrtf(x2) * 1.001f;
        const float e = mfma_bound_half<KB>(acc, reinterpret_cast<const unsigned *>(lds + L.waug), x2, dsq + __shfl_xor(dsq, 32, kWave),
                                            norm, c, lane);
        decide_half<KB, PRUNE>(acc, x2, norm, e, c, reinterpret_cast<const float *>(lds + L.w), lane, n, N, D, K, M, m, old, codes, pa, w, moved_list, moved_count);
        n = n_n;
        xrow = xrow_n;
        old = old_n;
    }
    decide_items<KB, PRUNE>(w, xp, Cm, hneg, D, ld, K, M, m, codes, pa, moved_list, moved_count);
    half_finish<PRUNE>(lds, L, w, amax, refine_count, moved_list, moved_count, work);
}

}  // namespace hclae
