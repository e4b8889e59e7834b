// Angular LSH: h(x) = argmax([xR; -xR]) for every query and round
// (Reformer, Sec. 2 "Locality sensitive hashing"; one R per round as in
// eq. union-pairs).
//
// Design (gfx950):
//  * The projections xR are a dense [rows x 64] * [64 x n_b/2] contraction per
//    round, run on the matrix cores with 16-bit operands and fp32
//    accumulation.  For bf16 input, q and each round of R are scaled by
//    powers of two (which leaves every argmax unchanged) and R is split into
//    binary16 planes R = R_hi + R_mid + res, |R_hi - R| <= 2^-12 |R|;
//    the scaled bf16 q is exact in binary16.  For fp32 input, q and R are
//    split into bf16 planes instead.  16-bit products are exact in fp32, so
//    a screened projection differs from the exact one by a bounded amount
//    (residual, fp32 accumulation, and the index bits packed into the low
//    mantissa).
//  * R streams through LDS by direct global-to-LDS copies, up to 256 columns
//    (128 in the screen, 64 with both planes of bf16 input) per stage, while
//    each wave's products for the next tile are interleaved with the vector
//    epilogue of the current one (one in-order instruction stream keeps both
//    the matrix core and the vector ALUs busy).
//  * Each lane keeps the two largest |projection| keys it has seen; the
//    index inside a 32-column tile rides in the low bits of the key, so an
//    and-or per projection and a max3, a med3 and a max per two suffice, and
//    the tile of the best key is noted once per tile.  A row's ids for all
//    rounds are written together at the end.
//  * If the gap between the best and second-best key cannot rule out an
//    exchange under the error bound, the row-round is appended to a list for
//    the next pass.  Large bf16 calls are screened over the hi plane alone and
//    their open row-rounds recomputed over both; small bf16 calls take both
//    planes at once, fp32 calls both planes of q and R.  What these leave open a
//    last kernel decides in fp64 (same products and summation order as a plain
//    loop), so the ids always equal the exact argmax.
#include "common.h"
#include "launch.h"

#include <type_traits>

namespace lsh {
namespace {

typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));

constexpr int kRB = 2;  // 32-row blocks per wave: each staged R tile feeds 2 * 8 MFMAs

// x * 2^e for |e| up to 254, in two exact steps.
__device__ __forceinline__ double ldexp2(double x, int e) {
    const int a = e / 2;
    return x * __builtin_bit_cast(double, (uint64_t)(1023 + a) << 52) *
           __builtin_bit_cast(double, (uint64_t)(1023 + e - a) << 52);
}

// Nearest binary16 of x (|x| < 2^15 here), or 0 below fp16's normal range:
// the planes hold no subnormal, whatever the matrix cores do with them.
__device__ __forceinline__ uint32_t f16_normal_bits(double x) {
    const _Float16 h = fabs(x) < 0x1p-14 ? (_Float16)0.f : (_Float16)(float)x;
    return (uint32_t)__builtin_bit_cast(uint16_t, h);
}

// R's planes and norms: two 16-bit planes hi/mid and R itself,
// [round][half_pad][64] (column contiguous, zero padded); three 2-norms of
// every column, [3][rounds][half_pad]: |R_c|, |R_c - hi_c|,
// |R_c - hi_c - mid_c|, and the largest of each, [3][rounds].
//  * F16 (bf16 input): binary16 planes of R_c * 2^sr, sr (in r_exp) bringing
//    the round's largest |R| into [2^14, 2^15), 0 when the round is zero or
//    not finite (a positive scale of a whole round leaves every argmax
//    unchanged); the norms are of the scaled column.
//  * bf16 planes (fp32 input): R = hi + mid + res with each step exact.
// The norms are formed in fp64 from exact residuals.  A block takes 64
// columns of a round, wave w the t's 4 w .. 4 w + 3 of them, and for F16
// looks the whole round (at most 128 KB, in the L2 after the first block)
// over for its largest |R| by itself, so that the scale needs no launch of
// its own.  A round of one block also needs none for the norms' maxima (up to
// 128 buckets: one launch instead of three, 12 -> 5 us); longer ones take
// prep_r_max_kernel.  The first block of a round clears its list counters.
constexpr int kPrepThreads = 1024;
constexpr int kPrepCols = 64;

template <bool F16>
__global__ __launch_bounds__(kPrepThreads) void prep_r_kernel(
    const float* __restrict__ R, int half, int half_pad, int* __restrict__ r_exp, uint16_t* __restrict__ r_hi,
    uint16_t* __restrict__ r_mid, float* __restrict__ r_t, float* __restrict__ col_norm, float* __restrict__ norm_max,
    int* __restrict__ seg_counts, int n_segs, int* __restrict__ counts) {
    constexpr int T = kHeadDim * kPrepCols / kPrepThreads;  // t's per thread
    static_assert(T == 4 && kPrepCols == 64, "a wave per four t's");
    constexpr int kWaves = kPrepThreads / 64;
    __shared__ double sums[3][kPrepThreads];
    __shared__ float red[kWaves];
    const int r = blockIdx.y, n_r = gridDim.y, tid = threadIdx.x, lane = tid & 63;
    const int sp = __builtin_amdgcn_readfirstlane(tid >> 6);
    if (blockIdx.x == 0) {
        if (tid < n_segs) seg_counts[(size_t)r * n_segs + tid] = 0;
        if (tid == 0) counts[r] = 0;
    }
    const int c = blockIdx.x * kPrepCols + lane;
    const bool live = c < half_pad;
    const float* Rr = R + (size_t)r * kHeadDim * half;
    float x[T];
#pragma unroll
    for (int j = 0; j < T; ++j) x[j] = Rr[(size_t)(sp * T + j) * half + min(c, half - 1)];
    int sr = 0;
    if constexpr (F16) {
        const int n = kHeadDim * half;
        float m = 0.f;
#pragma unroll 8
        for (int i = tid; i < n; i += kPrepThreads) m = fmaxf(m, fabsf(Rr[i]));
        m = wave_max(m);
        if (lane == 0) red[sp] = m;
        __syncthreads();
#pragma unroll
        for (int i = 0; i < kWaves; ++i) m = fmaxf(m, red[i]);
        // m in [2^e, 2^(e+1)) (frexp: m = f 2^k with f in [0.5, 1), e = k - 1)
        int k = 0;
        (void)frexpf(m, &k);
        sr = (m > 0.f && m <= 3.4e38f) ? 14 - (k - 1) : 0;
        if (blockIdx.x == 0 && tid == 0) r_exp[r] = sr;
    }
    double s0 = 0., s1 = 0., s2 = 0.;
    uint32_t hi[T / 2], mid[T / 2];
#pragma unroll
    for (int j = 0; j < T; ++j) {
        if (c >= half) x[j] = 0.f;
        const double xs = F16 ? ldexp2((double)x[j], sr) : (double)x[j];
        uint32_t hb, mb;
        double res, res2;
        if constexpr (F16) {
            hb = f16_normal_bits(xs);
            res = xs - (double)f16_bits_to_f32(hb);  // exact in fp64
            mb = f16_normal_bits(res);
            res2 = res - (double)f16_bits_to_f32(mb);  // exact
        } else {
            hb = f32_to_bf16_bits(x[j]);
            const float rs = x[j] - bf16_bits_to_f32(hb);  // exact (Sterbenz)
            mb = f32_to_bf16_bits(rs);
            res = (double)rs;
            res2 = (double)(rs - bf16_bits_to_f32(mb));  // exact
        }
        s0 += xs * xs;
        s1 += res * res;
        s2 += res2 * res2;
        hi[j / 2] = j & 1 ? hi[j / 2] | (hb << 16) : hb;
        mid[j / 2] = j & 1 ? mid[j / 2] | (mb << 16) : mb;
    }
    if (live) {
        const size_t o = ((size_t)r * half_pad + c) * kHeadDim + sp * T;
        *reinterpret_cast<f32x4*>(r_t + o) = f32x4{x[0], x[1], x[2], x[3]};
        *reinterpret_cast<uint2*>(r_hi + o) = make_uint2(hi[0], hi[1]);
        *reinterpret_cast<uint2*>(r_mid + o) = make_uint2(mid[0], mid[1]);
    }
    sums[0][tid] = s0;
    sums[1][tid] = s1;
    sums[2][tid] = s2;
    __syncthreads();
    if (sp < 3) {  // wave w: norm w of the block's columns
        double t = 0.;
#pragma unroll
        for (int k = 0; k < kWaves; ++k) t += sums[sp][64 * k + lane];
        // rounded up to fp32 (the bounds that use them are upper bounds)
        const float n = live ? (float)sqrt(t) * (1.f + 0x1p-22f) : 0.f;
        if (live) col_norm[((size_t)sp * n_r + r) * half_pad + c] = n;
        if (gridDim.x == 1) {
            const float mw = wave_max(n);
            if (lane == 0) norm_max[(size_t)sp * n_r + r] = mw;
        }
    }
}

// Largest of each column norm per round (block (round, which)), for rounds
// of more than one prep block.
__global__ __launch_bounds__(512) void prep_r_max_kernel(const float* __restrict__ col_norm, int n_r, int half_pad,
                                                         float* __restrict__ norm_max) {
    __shared__ float red[8];
    const int r = blockIdx.x, which = blockIdx.y, tid = threadIdx.x;
    const float* cn = col_norm + ((size_t)which * n_r + r) * half_pad;
    float mx = wave_max(tid < half_pad ? cn[tid] : 0.f);  // half_pad <= 512
    if ((tid & 63) == 0) red[tid >> 6] = mx;
    __syncthreads();
    if (tid < 8) {
        mx = group8_max(red[tid]);
        if (tid == 0) norm_max[which * n_r + r] = mx;
    }
}

template <bool F32>
__device__ __forceinline__ float q_value(const void* q, int64_t row, int k) {
    if constexpr (F32) {
        return static_cast<const float*>(q)[row * kHeadDim + k];
    } else {
        return bf16_bits_to_f32(static_cast<const uint16_t*>(q)[row * kHeadDim + k]);
    }
}

// Exact argmax of [xR; -xR] for the listed row-rounds of one round.  A block
// keeps the round's R in registers and takes the list in groups of 16
// entries, in two passes:
//  1. fp32 projections of every column on the matrix cores
//     (v_mfma_f32_16x16x4_f32: 16 columns x 16 entries).  Wave w owns columns
//     32 w .. 32 w + 31 as two tiles; k-step s of lane group g is t = 16 g + s,
//     so a lane holds 16 consecutive values of its entry's q row and, per
//     tile, 16 consecutive values of its column (r_t: R with its columns
//     contiguous), loaded once per block, all in flight together.  The fp32
//     value is within
//       eps = (64 * 2^-23 + 64 * 2^-24) * 1.05 * |q| * max_c |R_c|
//     of the exact one (64 additions to within an ulp, products to within
//     half), in any order, so only a column whose fp32 magnitude is within
//     2 eps of the entry's largest can hold the exact argmax;
//  2. for those candidates, the projection as the oracle forms it: the
//     left-to-right sum over t of the exact products q_t * R_tc in fp64, one
//     lane per (entry, candidate), eight candidate lanes per entry.  Ties go
//     to the first index of [xR; -xR].
// An entry with more than eight candidates, or whose |q| max_c |R_c| leaves
// the range in which eps bounds fp32's error (q = 0 and non-finite rows among
// them), takes the plain fp64 pass over every column, one wave per entry.
// Bound by latency: launch, a chain of dependent loads (count, list, q; R
// beside them; the candidates' columns) and the instruction fetch of code
// that each block runs once, so loops stay rolled where that costs little.
// Measured against the earlier form (lane = entry, R by scalar loads one t
// after another, 64 entries a block): 32 -> 6.2 us at L = 1K fp32, 23 -> 9.4
// at 4 x 8 x 4K with 64 buckets, 39 -> 29 at 16 x 64K with 8 rounds of 1024.
// Sixteen waves of two tiles hold R in registers without a spill (109 of 128);
// eight of four tiles, two blocks to a CU, kept 36 to 100 bytes a lane in scratch.
// Whole hash, us: 27.5 -> 25.0 at 4 x 8 x 4K with 64 buckets, 31.0 -> 28.6 at
// 2 x 4 x 6001 fp32, 69.9 -> 66.3 at 2 x 8 x 16K, 72.4 -> 68.3 at 2 x 8 x 12K with
// one R per head.
// Long lists are dealt out over all blocks.  With each round's list left to its
// own blocks, one round of equal columns took the hash of 16 x 64K (8 rounds)
// 63 ms against 16.6 now and 17 in the form of 256 blocks a round, and a head of
// zero rows among 8 of 12K, one R each, 1.53 ms against 0.44 and 1.29.
constexpr int kRefineThreads = 1024;
constexpr int kRefineWaves = kRefineThreads / 64;
constexpr int kRefineGroup = 16;     // entries per pass: a matrix tile's columns
constexpr int kRefineCand = 8;       // candidate lanes per entry
constexpr int kRefineTiles = 2;      // 16-column tiles per wave in pass 1
constexpr int kRefineOwn = 2;        // groups of its own round's list that a block takes before other rounds'
static_assert(kRefineWaves * kRefineTiles * 16 >= 512, "pass 1 covers n_b / 2 <= 512 columns");

__device__ __forceinline__ void better(double v, int i, double& bv, int& bi) {
    if (v > bv || (v == bv && i < bi)) {
        bv = v;
        bi = i;
    }
}

struct RefineShared {
    float qs[kRefineGroup][kHeadDim + 4];  // the group's q rows
    float qn[kRefineGroup];                // and their norms
    float mx[kRefineWaves][kRefineGroup];  // per wave: largest |fp32 projection| of each entry
    int cnt[kRefineGroup];                 // candidates found per entry
    int cand[kRefineGroup][kRefineCand];   // their columns
};

template <bool F32>
__global__ __launch_bounds__(kRefineThreads, 4) void hash_refine_kernel(
    const void* __restrict__ q, const float* __restrict__ r_t, int half, int half_pad, int n_r, int64_t list_stride,
    const int* __restrict__ lists, const int* __restrict__ counts, const float* __restrict__ col_norm_max,
    const int* __restrict__ r_exp, int32_t* __restrict__ buckets_) {
    __shared__ __attribute__((aligned(16))) RefineShared S;
    const int lane = lane_id(), e16 = lane & 15, g16 = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int c0 = wave * kRefineTiles * 16;  // this wave's columns in pass 1
    const bool has_cols = c0 < half;          // uniform per wave
    // A round's own blocks (those of its blockIdx.y) take kRefineOwn groups each
    // of its list, which is all of an ordinary one; the rest of a long list is
    // dealt out over the whole grid, so that one round's, or one head's, does
    // not wait for its own few blocks.  Lane l looks at the round k0 + l places
    // after the block's own.
    const int rounds = gridDim.y, own = kRefineOwn * gridDim.x;
    for (int k0 = 0; k0 < rounds; k0 += 64) {
    const int k_l = k0 + lane, r_l = (int)blockIdx.y + k_l;
    const int n_l = k_l < rounds ? counts[r_l < rounds ? r_l : r_l - rounds] : 0;
    uint64_t todo = __ballot((n_l + kRefineGroup - 1) / kRefineGroup >
                             (k_l == 0 ? 0 : own + k_l * (int)gridDim.x) + (int)blockIdx.x);
    for (; todo; todo &= todo - 1) {  // uniform per block
    const int kk = __ffsll((unsigned long long)todo) - 1;
    const int n = __builtin_amdgcn_readlane(n_l, kk);
    const int groups = (n + kRefineGroup - 1) / kRefineGroup;
    int r = (int)blockIdx.y + k0 + kk;  // round of the R sets: r % n_r of its rows
    r = r < rounds ? r : r - rounds;
    int32_t* buckets = buckets_ + r % n_r;
    const int* list = lists + list_stride * r;
    const float* Rt = r_t + (size_t)r * half_pad * kHeadDim;  // [column][t], zero columns up to half_pad
    // max_c |R_c| of the round as given (the planes' norms are of R * 2^r_exp)
    const float cn = r_exp ? ldexpf(col_norm_max[r], -r_exp[r]) : col_norm_max[r];
    f32x4 rc[kRefineTiles][4];                // column c0 + 16 tile + e16 (clamped), t = 16 g16 ..
    if (has_cols) {
        int col = c0 + e16;
        asm("" : "+v"(col));  // formed here: the addresses, kept over the loops, were spilled
#pragma unroll
        for (int tile = 0; tile < kRefineTiles; ++tile) {
            const uint32_t src = (uint32_t)min(col + 16 * tile, half - 1) * kHeadDim + 16 * g16;
#pragma unroll
            for (int k = 0; k < 4; ++k) rc[tile][k] = *reinterpret_cast<const f32x4*>(Rt + src + 4 * k);
        }
    }

    for (int g = (k0 + kk == 0 ? 0 : own + (k0 + kk) * (int)gridDim.x) + blockIdx.x; g < groups;
         g += g < own ? gridDim.x : gridDim.x * rounds) {
        if (threadIdx.x < kRefineGroup) S.cnt[threadIdx.x] = 0;
        // pass 1: the waves with columns (wave 0 always has some, and also
        // keeps the q rows for pass 2)
        f32x4 p[kRefineTiles] = {};
        if (has_cols) {
            const int64_t row = list[min(g * kRefineGroup + e16, n - 1)];
            f32x4 qv[4];
            if constexpr (F32) {
                const f32x4* src = reinterpret_cast<const f32x4*>(static_cast<const float*>(q) + row * kHeadDim + 16 * g16);
#pragma unroll
                for (int k = 0; k < 4; ++k) qv[k] = src[k];
            } else {
                const u32x4* src = reinterpret_cast<const u32x4*>(static_cast<const uint16_t*>(q) + row * kHeadDim + 16 * g16);
#pragma unroll
                for (int k = 0; k < 2; ++k) {
                    const u32x4 x = src[k];
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        qv[2 * k + e / 2][2 * (e & 1)] = __uint_as_float(x[e] << 16);
                        qv[2 * k + e / 2][2 * (e & 1) + 1] = __uint_as_float(x[e] & 0xFFFF0000u);
                    }
                }
            }
            if (wave == 0) {
                float ss = 0.f;
#pragma unroll
                for (int k = 0; k < 4; ++k) {
#pragma unroll
                    for (int e = 0; e < 4; ++e) ss = fmaf(qv[k][e], qv[k][e], ss);
                    *reinterpret_cast<f32x4*>(&S.qs[e16][16 * g16 + 4 * k]) = qv[k];
                }
                ss = sum_xor32(sum_xor16(ss));
                if (g16 == 0) S.qn[e16] = sqrtf(ss);
            }
            // p[tile][j]: |projection| of column c0 + 16 tile + 4 g16 + j for entry e16
#pragma unroll
            for (int s = 0; s < 16; ++s)
#pragma unroll
                for (int tile = 0; tile < kRefineTiles; ++tile)
                    p[tile] = __builtin_amdgcn_mfma_f32_16x16x4f32(rc[tile][s >> 2][s & 3], qv[s >> 2][s & 3], p[tile],
                                                                   0, 0, 0);
            float m = 0.f;
#pragma unroll
            for (int tile = 0; tile < kRefineTiles; ++tile)
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const float a = fabsf(p[tile][j]);
                    // a column past the round: below any cut
                    p[tile][j] = c0 + 16 * tile + 4 * g16 + j < half ? a : -1.f;
                    m = fmaxf(m, p[tile][j]);
                }
            m = max_xor32(max_xor16(m));
            if (g16 == 0) S.mx[wave][e16] = m;
        } else if (lane < kRefineGroup) {
            S.mx[wave][lane] = 0.f;
        }
        __syncthreads();
        if (has_cols) {
            float mx = S.mx[0][e16];
#pragma unroll
            for (int w = 1; w < kRefineWaves; ++w) mx = fmaxf(mx, S.mx[w][e16]);
            // |q| max |R_c| bounds every partial sum: above fp32's range a sum
            // may overflow, and far below it products (or q's squares, and with
            // them |q|) lose bits that eps does not count.  Such an entry gets
            // no candidates, whatever its projections came to (an infinity is
            // not below any cut).
            const float qn = S.qn[e16], size = qn * cn;
            const float eps = (float)(64 * (0x1p-23 + 0x1p-24) * 1.05) * size;
            const bool bounded = qn > 0x1p-64f && size > 0x1p-80f && size < 0x1p120f;
            const float cut = fmaxf(mx - 2.f * eps, 0.f);
            uint32_t mine = 0;  // bit 4 tile + j: a candidate
#pragma unroll
            for (int tile = 0; tile < kRefineTiles; ++tile)
#pragma unroll
                for (int j = 0; j < 4; ++j) mine |= (uint32_t)(bounded && p[tile][j] >= cut) << (4 * tile + j);
            while (mine) {
                const int jj = __ffs((int)mine) - 1;
                mine &= mine - 1;
                const int k = atomicAdd(&S.cnt[e16], 1);
                if (k < kRefineCand) S.cand[e16][k] = c0 + 16 * (jj >> 2) + 4 * g16 + (jj & 3);
            }
        }
        __syncthreads();

        // pass 2: lane = (entry i, candidate k), eight entries per wave
        if (wave < kRefineGroup * kRefineCand / 64) {
            const int i = wave * (64 / kRefineCand) + lane / kRefineCand;
            const int k = lane % kRefineCand;
            const int ci = S.cnt[i];
            double bv = -__builtin_inf();
            int bi = 0x7FFFFFFF;
            const int ei = g * kRefineGroup + i;
            const int row = list[min(ei, n - 1)];  // loaded beside the columns
            if (k < ci && ci <= kRefineCand) {
                const int cc = S.cand[i][k];
                const f32x4* col = reinterpret_cast<const f32x4*>(Rt + (size_t)cc * kHeadDim);
                // q_t * R_tc is exact in fp64 (at most 48 significant bits), so
                // whether the compiler fuses the multiply into the add or not,
                // the sum rounds exactly as the plain loop does.
                double acc = 0.0;
#pragma unroll 1
                for (int u0 = 0; u0 < 16; u0 += 4) {
                    f32x4 xr[4];
#pragma unroll
                    for (int u = 0; u < 4; ++u) xr[u] = col[u0 + u];
#pragma unroll
                    for (int u = 0; u < 4; ++u) {
                        const f32x4 xq = *reinterpret_cast<const f32x4*>(&S.qs[i][4 * (u0 + u)]);
#pragma unroll
                        for (int e = 0; e < 4; ++e) acc = __dadd_rn(acc, __dmul_rn((double)xq[e], (double)xr[u][e]));
                    }
                }
                better(acc, cc, bv, bi);
                better(-acc, half + cc, bv, bi);
            }
#pragma unroll
            for (int o = 1; o < kRefineCand; o <<= 1) {
                const double ov = __shfl_xor(bv, o);
                const int oi = __shfl_xor(bi, o);
                better(ov, oi, bv, bi);
            }
            if (k == 0 && ei < n && ci >= 1 && ci <= kRefineCand) buckets[(int64_t)row * n_r] = bi;
        }

        // entries left to fp64: every column, one wave each
        for (int i = wave; i < kRefineGroup; i += kRefineWaves) {
            const int ei = g * kRefineGroup + i;
            const int ci = S.cnt[i];
            if (ei >= n || (ci >= 1 && ci <= kRefineCand)) continue;  // uniform per wave
            double bv = -__builtin_inf();
            int bi = 0x7FFFFFFF;
#pragma unroll 1
            for (int c = lane; c < half; c += 64) {
                double acc = 0.0;
#pragma unroll 4
                for (int u = 0; u < 16; ++u) {
                    const f32x4 xq = *reinterpret_cast<const f32x4*>(&S.qs[i][4 * u]);
                    const f32x4 xr = reinterpret_cast<const f32x4*>(Rt + (size_t)c * kHeadDim)[u];
#pragma unroll
                    for (int e = 0; e < 4; ++e) acc = __dadd_rn(acc, __dmul_rn((double)xq[e], (double)xr[e]));
                }
                better(acc, c, bv, bi);
                better(-acc, half + c, bv, bi);
            }
#pragma unroll 1
            for (int o = 32; o >= 1; o >>= 1) {
                const double ov = __shfl_xor(bv, o);
                const int oi = __shfl_xor(bi, o);
                better(ov, oi, bv, bi);
            }
            if (lane == 0) buckets[(int64_t)list[ei] * n_r] = bi;
        }
        __syncthreads();  // the group's LDS is reused by the next one
    }
    }
    }
}

// R streams through LDS in stages of ST tiles (32 ST columns) of one round,
// NP planes, double-buffered: 2 x NP x 32 ST x 128 B, at most 128 KB (two
// planes with ST = 8; see launch_pass).  ST is the round's tile count rounded
// up to a power of two, capped by the pass, so small rounds compute no idle
// tiles and large ones few barriers.  A stage is copied straight from
// global memory into LDS (buffer loads to LDS, no registers in between)
// while the previous one is consumed, so there is one barrier per stage.  A
// 16-byte piece p of column c sits at slot p ^ stage_swz(c) of the column's
// 128 bytes: the 16 columns read together by one operand load then hit
// distinct banks.
template <int NP, int ST>
struct Stage {
    static constexpr int kCols = 32 * ST;
    static constexpr size_t kBytes = 2ull * NP * kCols * 128;  // both buffers
    static __device__ __forceinline__ uint32_t offset(int buf, int plane, int col) {
        return (uint32_t)(((buf * NP + plane) * kCols + col) * 128);
    }
};

__device__ __forceinline__ int stage_swz(int c) { return (c ^ (c >> 3)) & 7; }

// LDS past the stage buffers: each wave's winners [64 rows][rounds] as
// 16-bit ids.  The stage area is at least as large as the screen's final
// list gathering needs, [rounds][64 WAVES] rows and two counters per round.
__host__ __device__ constexpr size_t hash_win_offset(size_t stage_bytes, int waves, int rounds) {
    const size_t lists = (size_t)rounds * (64 * waves + 2) * 4;
    return ((stage_bytes > lists ? stage_bytes : lists) + 15) / 16 * 16;
}

// The screen's open row-rounds go to kSegs segments per round (workgroup b
// appends to segment b % kSegs), so each list counter sees few atomics.
constexpr int kSegs = 64;

// The screen: waves per SIMD it is built for (three workgroups of four waves
// on a CU, registers and LDS permitting), and its largest stage.
constexpr int kScreenOcc = 3;
constexpr int kScreenMaxTiles = 4;

// Passes of the main kernel.
enum : int {
    kScreen = 0,  // bf16 input: R's hi plane only, every row and round
    kExact = 1,   // both planes (three products for fp32 input), every row and round
    kListed = 2,  // bf16 input: both planes, the rows the screen left open in one round
};

struct Tile {
    f32x16 acc[kRB];
};

// Keys order projections by |projection| truncated to a few bits less than
// fp32's 24 (non-negative floats order like their bit patterns), with an
// index in the bits the truncation frees:
//  * fp32 input: the bit pattern rotated left by one (sign in bit 0,
//    |projection| in bits 5..31, the register j of the tile in bits 1..4):
//    one rotate and one and-or per projection, and the key also carries the
//    winner's sign.  The winner's tile is noted after every tile.
//  * bf16 input: |projection| in bits 6..30 and 16 (t % 4) + j in bits
//    0..5 (tile t of the round), one and-or; the winner's group of four
//    tiles is noted after every fourth tile, and its sign is recomputed once
//    per row and round.
// Keys of tiles past the round are masked to their index, near zero.
template <bool F32, int ST>
constexpr int kKeyTiles = F32 ? 1 : (ST < 4 ? ST : 4);  // tiles sharing one index field

template <bool F32>
__device__ __forceinline__ uint32_t proj_key(float x, int idx, bool live) {
    const uint32_t u = __float_as_uint(x);
    if constexpr (F32) {
        return (__builtin_amdgcn_alignbit(u, u, 31) & (live ? 0xFFFFFFE1u : 0u)) | ((uint32_t)idx << 1);
    } else {
        return (u & (live ? 0x7FFFFFC0u : 0u)) | (uint32_t)idx;
    }
}
template <bool F32>
__device__ __forceinline__ uint32_t key_index(uint32_t key) {
    return F32 ? (key >> 1) & 15u : key & 63u;
}
template <bool F32>
__device__ __forceinline__ float key_magnitude(uint32_t key) {
    return __uint_as_float(F32 ? (key >> 1) & 0x7FFFFFF0u : key & 0x7FFFFFC0u);
}

// Running best b and second best sc (b >= sc) after two more keys: the
// largest of {b, k1, k2} is the new best, the middle one is the largest of
// the rest of those three, and sc joins the rest.  One max3, one med3 and
// one max per two projections.
// (max3 as inline assembly: left to itself the compiler shares max(b, k1)
// with the median and spends a fourth instruction.)
__device__ __forceinline__ void key_update2(uint32_t k1, uint32_t k2, uint32_t& b, uint32_t& sc) {
    const uint32_t mid = max(min(b, k1), min(max(b, k1), k2));  // median of three
    uint32_t top;
    asm("v_max3_u32 %0, %1, %2, %3" : "=v"(top) : "v"(b), "v"(k1), "v"(k2));
    b = top;
    sc = max(sc, mid);
}

// Lane offsets of the NP-plane operand pieces of tiles 0 and 1 inside a
// stage buffer: piece i is k-step i / NP of plane i % NP.  Column 32 t + n
// of tile t sits at 4096 t + 128 n with its pieces in swizzled slots, and
// stage_swz(32 t + n) = stage_swz(n) ^ 4 (t % 2): even tiles share tile 0's
// slot pattern, odd ones tile 1's.
template <int NP, int ST>
__device__ __forceinline__ void piece_offsets(uint32_t (&off)[2][8], int n, int h) {
#pragma unroll
    for (int par = 0; par < 2; ++par)
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const int s = NP == 2 ? i >> 1 : i;
            const int plane = NP == 2 ? (i & 1) : 0;
            off[par][i] = (uint32_t)(plane * Stage<NP, ST>::kCols * 128 + (32 * par + n) * 128 +
                                     (((4 * h + s) ^ stage_swz(32 * par + n)) << 4));
        }
}

// Products of 16-bit operand words: bf16 planes for fp32 input, binary16
// planes (of scaled q and R) for bf16 input.
template <bool F32>
__device__ __forceinline__ f32x16 mfma_op(u32x4 a, u32x4 b, f32x16 c) {
    if constexpr (F32)
        return mfma32x32x16(as_bf16x8(a), as_bf16x8(b), c);
    else
        return mfma32x32x16(as_f16x8(a), as_f16x8(b), c);
}

// One step of the tile pipeline, in eight slices.  Slice i issues (MF) the
// products of the tile held in `op` into `nxt` for operand piece i (both
// planes; for fp32 input the hi plane also meets q's second plane) or, with
// one plane, for piece i / 2 on even slices; refills that piece with the same
// piece of tile TP (PREF) of the stage at `sb`; and runs one eighth of the
// epilogue of the previous tile `cur`, tile TC of the stage (EPI).  A wave
// issues in order, so this interleaving is what lets the vector ALUs work
// while the matrix core runs; the scheduling barriers keep the compiler from
// regrouping the slices.  Tile numbers are compile-time constants, so the
// operand addresses are a lane offset plus an immediate and the key indices
// are inline constants.
template <bool F32, int NP, int G, bool MF, int TP, int TC>
__device__ __forceinline__ void tile_step(Tile& nxt, u32x4 (&op)[8], const char* __restrict__ sb,
                                          const uint32_t (&poff)[2][8], const u32x4 (&qa)[kRB][4],
                                          const u32x4 (&qm)[kRB][4], const Tile& cur, bool live,
                                          uint32_t (&best)[kRB], uint32_t (&second)[kRB]) {
    static_assert(kRB == 2, "slices written for two row blocks");
    constexpr bool PREF = TP >= 0, EPI = TC >= 0;
    constexpr int idx0 = EPI ? 16 * (TC % G) : 0;
    uint32_t b[kRB] = {best[0], best[1]}, sc[kRB] = {second[0], second[1]};
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        __builtin_amdgcn_sched_barrier(0);
        if (MF && (NP == 2 || (i & 1) == 0)) {
            const int pi = NP == 2 ? i : i >> 1;  // operand piece
            const int s = i >> 1;  // k-step
            const bool hi_plane = NP == 1 || (i & 1) == 0;
#pragma unroll
            for (int rb = 0; rb < kRB; ++rb)
                nxt.acc[rb] = mfma_op<F32>(op[pi], qa[rb][s], pi == 0 ? f32x16{} : nxt.acc[rb]);
            if constexpr (F32) {
                if (hi_plane) {
#pragma unroll
                    for (int rb = 0; rb < kRB; ++rb) nxt.acc[rb] = mfma_op<F32>(op[pi], qm[rb][s], nxt.acc[rb]);
                }
            }
            if constexpr (PREF)
                op[pi] = *reinterpret_cast<const u32x4*>(sb + poff[TP & 1][pi] + (TP & ~1) * 4096);
        }
        __builtin_amdgcn_sched_barrier(0);
        if constexpr (EPI) {
#pragma unroll
            for (int rb = 0; rb < kRB; ++rb)
                key_update2(proj_key<F32>(cur.acc[rb][2 * i], idx0 + 2 * i, live),
                            proj_key<F32>(cur.acc[rb][2 * i + 1], idx0 + 2 * i + 1, live), b[rb], sc[rb]);
        }
    }
    __builtin_amdgcn_sched_barrier(0);
    if constexpr (EPI) {
#pragma unroll
        for (int rb = 0; rb < kRB; ++rb) {
            best[rb] = b[rb];
            second[rb] = sc[rb];
        }
    }
}

// Source offsets of 1 KB runs of 8 columns (c0 .. c0+7, c0 a multiple of
// 8, stage-local): lane = 8 cl + slot fetches the piece that belongs at LDS
// slot `slot` of column c0 + cl, piece slot ^ stage_swz(c0 + cl).  As
// stage_swz(c0 + cl) = cl ^ (c0 / 8 % 8), the lane's byte offset in the run
// is run_lane_offset(lane) ^ (16 * (c0 / 8 % 8)): one xor per run.
__device__ __forceinline__ uint32_t run_lane_offset(int lane) {
    const int cl = lane >> 3, slot = lane & 7;
    return (uint32_t)(cl * 128 + ((slot ^ cl) << 4));
}

// Raw buffer over one R plane (word 3 of the descriptor: raw, untyped
// 32-bit data as on other CDNA parts); loads past num_records return 0.
constexpr int kRawBufferWord3 = 0x00020000;

__device__ __forceinline__ __amdgpu_buffer_rsrc_t plane_buffer(const uint16_t* plane, uint32_t bytes) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t*>(plane), 0, (int)bytes, kRawBufferWord3);
}

// One run straight into LDS: a buffer load with the run's column in the
// scalar offset and the lane's piece in the vector offset (no 64-bit vector
// addresses to keep).
__device__ __forceinline__ void copy_run(__amdgpu_buffer_rsrc_t plane, int64_t col0, uint32_t lane_off, int c0,
                                         char* lds_dst) {
    __builtin_amdgcn_raw_ptr_buffer_load_lds(plane, (__attribute__((address_space(3))) void*)lds_dst, 16,
                                             lane_off ^ (uint32_t)(((c0 >> 3) & 7) << 4), (uint32_t)(col0 * 128),
                                             0, 0);
}

// Copy global stage g (round g / spr, columns (g % spr) * 32 ST ...) of NP
// planes into buffer buf.  Each wave moves whole 1 KB runs of 8 columns of
// one plane; a run past the round copies the round's first columns instead
// (any valid address: never read).
template <int WAVES, int NP, int ST>
__device__ __forceinline__ void load_stage(char* smem, int buf, int g, int spr, int half_pad,
                                           __amdgpu_buffer_rsrc_t r_hi, __amdgpu_buffer_rsrc_t r_mid, int wave,
                                           uint32_t lane_off) {
    constexpr int kCols = Stage<NP, ST>::kCols;
    constexpr int kRuns = NP * kCols / 8;  // 1 KB runs per stage
    const int r = g / spr, st = g % spr;
#pragma unroll
    for (int i = 0; i < (kRuns + WAVES - 1) / WAVES; ++i) {
        const int run = wave + i * WAVES;  // uniform per wave
        if (kRuns % WAVES == 0 || run < kRuns) {
            const int plane = run / (kCols / 8);
            const int c0 = (run % (kCols / 8)) * 8;
            const int gc0 = st * kCols + c0;
            copy_run(plane ? r_mid : r_hi, (int64_t)r * half_pad + (gc0 < half_pad ? gc0 : 0), lane_off, c0,
                     smem + Stage<NP, ST>::offset(buf, plane, c0));
        }
    }
}

// This lane half's 32 k-values of q . R_col for one binary16 plane: 16 pair
// products in four short chains (fp32 sums of exact products).
__device__ __forceinline__ float dot_planes(const u32x4 (&qa4)[4], const u32x4 (&rv)[4]) {
    typedef _Float16 f16x2 __attribute__((ext_vector_type(2)));
    float part[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int s4 = 0; s4 < 4; ++s4) {
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const uint32_t qw = qa4[s4][e], rw = rv[s4][e];
            part[e] = __builtin_amdgcn_fdot2(__builtin_bit_cast(f16x2, qw), __builtin_bit_cast(f16x2, rw), part[e],
                                             false);
        }
    }
    return (part[0] + part[1]) + (part[2] + part[3]);
}

// The tile pipeline of one stage of ST tiles: step T issues tile T's
// products (into ta for even T, tb for odd), prefetches tile T + 1's
// operands and runs the epilogue of tile T - 1; a last step runs tile
// ST - 1's epilogue alone.  ge(t) is called after tile t's epilogue.
template <bool F32, int NP, int ST, int T, class GE>
__device__ __forceinline__ void stage_pipe(Tile& ta, Tile& tb, u32x4 (&op)[8], const char* __restrict__ sb,
                                           const uint32_t (&poff)[2][8], const u32x4 (&qa)[kRB][4],
                                           const u32x4 (&qm)[kRB][4], int nt, uint32_t (&best)[kRB],
                                           uint32_t (&second)[kRB], GE& ge) {
    if constexpr (T < ST) {
        Tile& nxt = T % 2 == 0 ? ta : tb;
        Tile& cur = T % 2 == 0 ? tb : ta;
        tile_step<F32, NP, kKeyTiles<F32, ST>, true, (T + 1 < ST ? T + 1 : -1), T - 1>(
            nxt, op, sb, poff, qa, qm, cur, T - 1 < nt, best, second);
        if constexpr (T >= 1) ge(T - 1);
        stage_pipe<F32, NP, ST, T + 1>(ta, tb, op, sb, poff, qa, qm, nt, best, second, ge);
    } else {
        Tile& cur = (ST - 1) % 2 == 0 ? ta : tb;
        tile_step<F32, NP, kKeyTiles<F32, ST>, false, -1, ST - 1>(cur, op, sb, poff, qa, qm, cur, ST - 1 < nt, best,
                                                                  second);
        ge(ST - 1);
    }
}

// Winner of a row-round as kept in LDS until the row's ids are written:
// the bucket id, or kUnsettled when a later pass must decide.
constexpr uint16_t kUnsettled = 0xFFFFu;

// The main kernel, one of three passes (MODE).  A wave owns 64 rows (two
// 32-row blocks) and sweeps every staged tile once for them.
//  * R comes in sets of n_r rounds: one set for all rows, or one per head
//    (Slices).  The rows form slices that share a set; blocks are numbered
//    slice after slice, so no block's rows span two sets.  Rounds count
//    through the sets: round r of set s is s * n_r + r in the planes, norms,
//    lists and counts.
//  * kScreen and kExact take 64 * WAVES rows of one slice and all rounds of
//    its set; kListed takes, for round blockIdx.z, the rows the screen left
//    open in that round (its segments one after another), in chunks of
//    64 * WAVES, workgroup blockIdx.x taking every gridDim.x-th chunk.
//  * Every screened projection is within
//        eps = |q| * (res_max[r] + err_acc * max_c |R_c|)
//    of the exact one (res_max: largest 2-norm of R's columns less the
//    planes used, none for fp32 input, whose planes' residual is inside
//    err_acc), and a key's magnitude is low by at most err_pack of it.  For
//    bf16 input the best key's column w is then recomputed, by the screen
//    over the hi plane (within |q| (|R_w - hi_w| + err_acc max_c |R_c|)),
//    by the listed pass over both planes (within eps2, from res_max2 and
//    err_acc2), and the row-round is settled when that value's magnitude
//    less its bound exceeds the second key plus eps; for fp32 input when the
//    best and second keys are more than 2 eps apart.
//    A settled id goes to buckets.  Otherwise the row is appended to the round's list: the
//    screen's lists are segmented, [round][kSegs][seg_cap] with counts
//    [round][kSegs]; the exact passes' are [round][rows] with one count per
//    round (few rows reach them).
struct Slices {
    int64_t rows;     // rows of a slice
    int blocks;       // blocks of a slice
    int sets;         // slices s, s + sets, ... share set s
    int heads, head0; // slice s starts at row ((s / sets) heads + head0 + s % sets) rows
    int64_t set_rows; // rows of a set, over all its slices (the stride of the exact passes' lists)
};

template <bool F32, int MODE, int WAVES, int ST>
__global__ __launch_bounds__(WAVES * 64, (MODE == kScreen ? kScreenOcc : 1)) void hash_kernel(
    const void* __restrict__ q, Slices sl, int n_r, int half, int half_pad,
    const uint16_t* __restrict__ r_hi_, const uint16_t* __restrict__ r_mid_,
    const float* __restrict__ col_norm_max_, const float* __restrict__ res_max_, float err_acc,
    const float* __restrict__ res_max2_, float err_acc2, float err_pack, const float* __restrict__ col_res_,
    int32_t* __restrict__ buckets, const int* __restrict__ list_in,
    const int* __restrict__ count_in, int* __restrict__ list_out_, int* __restrict__ count_out_,
    int64_t seg_cap) {
    static_assert(!F32 || MODE == kExact, "fp32 input takes the exact pass only");
    constexpr int NP = MODE == kScreen ? 1 : 2;
    constexpr int kWaveRows = 64;
    extern __shared__ __attribute__((aligned(16))) char smem[];

    const int tid = threadIdx.x;
    const int lane = tid & 63, h = lane >> 5, n = lane & 31;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const uint32_t run_off = run_lane_offset(lane);
    // the slice of this block (kListed: unused) and its rows
    const int slice = MODE == kListed ? 0 : (int)blockIdx.x / sl.blocks;
    const int64_t slice_row = ((int64_t)(slice / sl.sets) * sl.heads + sl.head0 + slice % sl.sets) * sl.rows;
    const int slice_block = MODE == kListed ? (int)blockIdx.x : (int)blockIdx.x % sl.blocks;
    // this block's rounds of R: those of its set, or (kListed) the one round
    // of blockIdx.z; everything per round is addressed from the first of them
    const int64_t rr0 = MODE == kListed ? (int)blockIdx.z : slice % sl.sets * n_r;
    const uint16_t *r_hi = r_hi_ + rr0 * half_pad * kHeadDim, *r_mid = r_mid_ + rr0 * half_pad * kHeadDim;
    const float *col_norm_max = col_norm_max_ + rr0, *res_max = F32 ? nullptr : res_max_ + rr0;
    const float *res_max2 = F32 ? nullptr : res_max2_ + rr0;
    const float* col_res = MODE == kScreen ? col_res_ + rr0 * half_pad : nullptr;
    int* list_out = list_out_ + rr0 * (MODE == kScreen ? kSegs * seg_cap : sl.set_rows);
    int* count_out = count_out_ + rr0 * (MODE == kScreen ? kSegs : 1);
    const int nrb = MODE == kListed ? 1 : n_r;  // rounds of this block
    int32_t* bucket_cols = MODE == kListed ? buckets + (int)blockIdx.z % n_r : buckets;
    const uint32_t plane_bytes = (uint32_t)((size_t)nrb * half_pad * kHeadDim * 2);
    const __amdgpu_buffer_rsrc_t rs_hi = plane_buffer(r_hi, plane_bytes), rs_mid = plane_buffer(r_mid, plane_bytes);
    using SG = Stage<NP, ST>;
    const int tpr = half_pad / 32;            // tiles per round
    const int spr = (tpr + ST - 1) / ST;      // stages per round
    // kListed: the round's open rows, segment after segment; lane s holds
    // the end of segment s in that sequence (kSegs is the wave width)
    int64_t listed = 0;
    int seg_end = 0;
    if constexpr (MODE == kListed) {
        static_assert(kSegs == 64, "one segment per lane");
        int incl = count_in[rr0 * kSegs + lane];
        for (int o = 1; o < 64; o <<= 1) {
            const int y = __shfl_up(incl, o);
            if (lane >= o) incl += y;
        }
        seg_end = incl;
        listed = __shfl(incl, 63);
    }
    // kListed: the workgroups take the round's chunks of 64 * WAVES rows in
    // turn; the other passes take one chunk each.
    for (int64_t chunk = slice_block;; chunk += gridDim.x) {
    if (MODE == kListed && chunk * (WAVES * kWaveRows) >= listed) break;  // uniform per block
    const int64_t slot0 = chunk * (WAVES * kWaveRows) + wave * kWaveRows;
    // the row of lane n of row block rb (lane half h keeps row block h's
    // results at the end)
    auto row_of = [&](int rb, bool& valid) -> int64_t {
        const int64_t k = slot0 + rb * 32 + n;
        if constexpr (MODE == kListed) {
            valid = k < listed;
            // segment of entry k: the first s with seg_end[s] > k (binary
            // search over the lanes; every lane takes part in the shuffles)
            const int kk = (int)min(k, max(listed - 1, (int64_t)0));
            int sg = 0;
#pragma unroll
            for (int step = 32; step >= 1; step >>= 1)
                if (__shfl(seg_end, sg + step - 1) <= kk) sg += step;
            sg = min(sg, 63);
            const int before = __shfl(seg_end, max(sg - 1, 0));
            const int64_t at = (rr0 * kSegs + sg) * seg_cap + (kk - (sg > 0 ? before : 0));
            return valid ? list_in[at] : 0;
        } else {
            valid = k < sl.rows;
            return slice_row + (valid ? k : 0);
        }
    };
    // this wave's winners: [row in wave][round of the block]
    uint16_t* win = reinterpret_cast<uint16_t*>(smem + hash_win_offset(SG::kBytes, WAVES, nrb)) +
                    (size_t)wave * kWaveRows * nrb;

    load_stage<WAVES, NP, ST>(smem, 0, 0, spr, half_pad, rs_hi, rs_mid, wave, run_off);

    // Queries as the B operand: lane holds row (n) and k = 32h + 8s + e, s = 0..3.
    u32x4 qa[kRB][4];
    u32x4 qm[kRB][4];  // fp32 input: second bf16 plane of q
    float qn[kRB];
#pragma unroll
    for (int rb = 0; rb < kRB; ++rb) {
        bool valid;
        const int64_t row = row_of(rb, valid);
        float ss = 0.f;
        if constexpr (F32) {
            const float* src = static_cast<const float*>(q) + row * kHeadDim + 32 * h;
#pragma unroll
            for (int s4 = 0; s4 < 4; ++s4) {
                f32x4 x0 = valid ? *reinterpret_cast<const f32x4*>(src + 8 * s4) : f32x4{0, 0, 0, 0};
                f32x4 x1 = valid ? *reinterpret_cast<const f32x4*>(src + 8 * s4 + 4) : f32x4{0, 0, 0, 0};
                float xs[8] = {x0[0], x0[1], x0[2], x0[3], x1[0], x1[1], x1[2], x1[3]};
                u32x4 hi, mid;
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const uint32_t h0 = f32_to_bf16_bits(xs[2 * e]), h1 = f32_to_bf16_bits(xs[2 * e + 1]);
                    const uint32_t m0 = f32_to_bf16_bits(xs[2 * e] - bf16_bits_to_f32(h0));
                    const uint32_t m1 = f32_to_bf16_bits(xs[2 * e + 1] - bf16_bits_to_f32(h1));
                    hi[e] = h0 | (h1 << 16);
                    mid[e] = m0 | (m1 << 16);
                    ss = fmaf(xs[2 * e], xs[2 * e], ss);
                    ss = fmaf(xs[2 * e + 1], xs[2 * e + 1], ss);
                }
                qa[rb][s4] = hi;
                qm[rb][s4] = mid;
            }
        } else {
            // The row times 2^sq, with its largest |q_t| brought into
            // [2^14, 2^15): exact in fp32, and in binary16 for every value
            // from fp16's smallest normal 2^-14 up (bf16 has 8 significant
            // bits); smaller values are dropped, |delta q| <= 8 * 2^-14.
            const uint16_t* src = static_cast<const uint16_t*>(q) + row * kHeadDim + 32 * h;
            u32x4 raw[4];
            float mx = 0.f;
#pragma unroll
            for (int s4 = 0; s4 < 4; ++s4) {
                raw[s4] = valid ? *reinterpret_cast<const u32x4*>(src + 8 * s4) : u32x4{0, 0, 0, 0};
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    mx = fmaxf(mx, fmaxf(fabsf(__uint_as_float(raw[s4][e] << 16)),
                                         fabsf(__uint_as_float(raw[s4][e] & 0xFFFF0000u))));
            }
            mx = max_xor32(mx);
            int k = 0;
            (void)frexpf(mx, &k);
            const int sq = (mx > 0.f && mx <= 3.4e38f) ? 14 - (k - 1) : 0;
            const float f1 = __uint_as_float((uint32_t)(127 + sq / 2) << 23);
            const float f2 = __uint_as_float((uint32_t)(127 + sq - sq / 2) << 23);
            auto to_f16 = [&](float x) {
                const float xs = x * f1 * f2;
                ss = fmaf(xs, xs, ss);
                return fabsf(xs) < 0x1p-14f ? 0.f : xs;
            };
#pragma unroll
            for (int s4 = 0; s4 < 4; ++s4) {
                u32x4 w;
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    w[e] = pack_f16x2(to_f16(__uint_as_float(raw[s4][e] << 16)),
                                      to_f16(__uint_as_float(raw[s4][e] & 0xFFFF0000u)));
                qa[rb][s4] = w;
                qm[rb][s4] = u32x4{0, 0, 0, 0};
            }
        }
        ss = sum_xor32(ss);
        qn[rb] = sqrtf(ss);
    }
    __builtin_amdgcn_s_waitcnt(0);
    __syncthreads();

    uint32_t poff[2][8];
    piece_offsets<NP, ST>(poff, n, h);
    constexpr int G = kKeyTiles<F32, ST>;
    // best and second key, the best key before the current group of G
    // tiles, and the group the best key came from
    uint32_t best[kRB], second[kRB], grp_start[kRB];
    int best_grp[kRB];
    const int g_end = nrb * spr;
    for (int g = 0; g < g_end; ++g) {
        const int r = g / spr, st = g % spr, buf = g & 1;
        if (st == 0) {
#pragma unroll
            for (int rb = 0; rb < kRB; ++rb) {
                best[rb] = second[rb] = grp_start[rb] = 0u;
                best_grp[rb] = 0;
            }
        }
        // the next stage lands in the other buffer while this one computes
        if (g + 1 < g_end)
            load_stage<WAVES, NP, ST>(smem, buf ^ 1, g + 1, spr, half_pad, rs_hi, rs_mid, wave, run_off);
        const char* sb = smem + SG::offset(buf, 0, 0);
        const int nt = min(ST, tpr - st * ST);
        const int t0 = st * ST;
        // after the epilogue of stage tile tc: note the group if it ends there
        // (stages start on group boundaries: G divides ST)
        auto group_end = [&](int tc) {
            if ((tc + 1) % G == 0) {
#pragma unroll
                for (int rb = 0; rb < kRB; ++rb) {
                    best_grp[rb] = best[rb] != grp_start[rb] ? (t0 + tc) / G : best_grp[rb];
                    grp_start[rb] = best[rb];
                }
            }
        };
        // Every stage runs all ST tiles; tiles past the round (a last,
        // partial stage) compute on stale LDS and their keys are masked to
        // (near) zero, so they can only win when every key is tiny, and such
        // a row is left to the exact passes.
        {
            Tile ta, tb;
            u32x4 op[8];
#pragma unroll
            for (int i = 0; i < 4 * NP; ++i) op[i] = *reinterpret_cast<const u32x4*>(sb + poff[0][i]);
            stage_pipe<F32, NP, ST, 0>(ta, tb, op, sb, poff, qa, qm, nt, best, second, group_end);
        }

        if (st == spr - 1) {
            // Round epilogue: merge the two lane halves (different columns of
            // the same row) and decide; lane half h keeps row block h's result.
            const float cn = col_norm_max[r];
            const float res = F32 ? 0.f : res_max[r];
            uint32_t bk[kRB], sk[kRB];
            int col[kRB];
#pragma unroll
            for (int rb = 0; rb < kRB; ++rb) {
                const uint32_t bb = best[rb], ss2 = second[rb];
                const uint32_t bp = xor32(bb), sp = xor32(ss2);
                const int tp = (int)xor32((uint32_t)best_grp[rb]);
                const bool mine = bb > bp || (bb == bp && h == 0);
                bk[rb] = mine ? bb : bp;
                sk[rb] = max(min(bb, bp), max(ss2, sp));
                const int hw = mine ? h : (h ^ 1);
                const int gw = mine ? best_grp[rb] : tp;
                const uint32_t idx = key_index<F32>(bk[rb]), j = idx & 15u;
                const int tw = gw * G + (int)(idx >> 4);  // tile of the round
                col[rb] = tw * 32 + 8 * (int)(j >> 2) + 4 * hw + (int)(j & 3u);
            }
            if constexpr (F32) {
                // Every screened key is within eps of its exact |projection|;
                // an exchange of winners needs a gap <= 2 eps.  When the gap is
                // larger the winner's magnitude exceeds eps, so the screened
                // sign (bit 0 of the key) is the exact one.
#pragma unroll
                for (int rb = 0; rb < kRB; ++rb) {
                    const float b1 = key_magnitude<F32>(bk[rb]), s1 = key_magnitude<F32>(sk[rb]);
                    const float thr = 2.04f * (qn[rb] * (res + err_acc * cn) + err_pack * b1);
                    const bool flag = !(b1 - s1 > thr) || col[rb] >= half;
                    const int id = (bk[rb] & 1u) ? half + col[rb] : col[rb];
                    if (rb == h) win[(rb * 32 + n) * nrb + r] = flag ? kUnsettled : (uint16_t)id;
                }
            } else {
                // x = q_row . R_col of the best key's column (fp32 sums of
                // the exact products; each lane half adds its 32 k-values).
                // Every other column's exact |projection| is at most the
                // second key (raised by the truncated bits) plus the pass's
                // eps, so the winner is certain when |x| less x's own error
                // bound exceeds that, and its sign is x's.  A flagged winner
                // may sit past the round; any valid column stands in.
                //  * The screen takes x over the hi plane alone: within
                //    eps_w = |q| (|R_w - hi_w| + err_acc max_c |R_c|) for the
                //    winner's column w.  Rows it leaves open go to the listed
                //    pass, which costs less than the mid plane's loads here.
                //  * The listed pass takes x over both planes, within eps2.
                // The pieces come from global memory (the planes are small
                // and stay in the caches).
                constexpr bool kHiOnly = MODE == kScreen;
                u32x4 hv[kRB][4], mv[kRB][4];
                // Lane half h keeps only row block h's decision, so it needs
                // only that winner's residual: one gather (a 4-byte gather
                // costs the address unit as much as a 16-byte one), issued
                // first, with the planes' (left to itself the compiler issues
                // it after the first block's products and waits on it).
                float res_own = 0.f;
                if constexpr (kHiOnly)
                    res_own = col_res[(size_t)r * half_pad + min(h ? col[1] : col[0], half_pad - 1)];
#pragma unroll
                for (int rb = 0; rb < kRB; ++rb) {
                    const int cc = min(col[rb], half_pad - 1);
                    const size_t o = ((size_t)r * half_pad + cc) * kHeadDim + 32 * h;
                    const u32x4* ph = reinterpret_cast<const u32x4*>(r_hi + o);
                    const u32x4* pm = reinterpret_cast<const u32x4*>(r_mid + o);
#pragma unroll
                    for (int s4 = 0; s4 < 4; ++s4) {
                        hv[rb][s4] = ph[s4];
                        if constexpr (!kHiOnly) mv[rb][s4] = pm[s4];
                    }
                }
                if constexpr (kHiOnly) asm volatile("" : "+v"(res_own));
#pragma unroll
                for (int rb = 0; rb < kRB; ++rb) {
                    float half_x = dot_planes(qa[rb], hv[rb]);
                    if constexpr (!kHiOnly) half_x += dot_planes(qa[rb], mv[rb]);
                    const float x = sum_xor32(half_x);
                    const float s1 = key_magnitude<F32>(sk[rb]);
                    const float eps = 1.02f * qn[rb] * (res + err_acc * cn);
                    const float eps_x = kHiOnly ? 1.02f * qn[rb] * (res_own + err_acc * cn)  // kept for rb == h
                                                : 1.02f * qn[rb] * (res_max2[r] + err_acc2 * cn);
                    const bool flag = !(fabsf(x) - eps_x > s1 * (1.f + 2.f * err_pack) + eps) || col[rb] >= half;
                    const int id = x < 0.f ? half + col[rb] : col[rb];
                    if (rb == h) win[(rb * 32 + n) * nrb + r] = flag ? kUnsettled : (uint16_t)id;
                }
            }
        }
        // the next stage has landed and every wave is done with this buffer
        __builtin_amdgcn_s_waitcnt(0);
        __syncthreads();
    }

    // Write each row's ids and queue the row-rounds left open.
    bool valid;
    const int64_t row = row_of(h, valid);
    const uint16_t* w = win + (h * 32 + n) * nrb;
    if constexpr (MODE == kScreen) {
        // Gather the block's open rows per round in LDS (the stage buffers
        // are free now), then reserve room in this block's segment with one
        // atomic per round and copy them out.
        int* lq = reinterpret_cast<int*>(smem);            // [nrb][WAVES * 64]
        int* lcnt = lq + nrb * WAVES * kWaveRows;          // [nrb]
        int* lbase = lcnt + nrb;                           // [nrb]
        if (tid < nrb) lcnt[tid] = 0;
        __syncthreads();
        for (int rr = 0; rr < nrb; ++rr) {
            const uint16_t id = w[rr];
            const bool queue = valid && id == kUnsettled;
            if (valid) bucket_cols[row * n_r + rr] = id == kUnsettled ? 0 : (int32_t)id;
            const uint64_t qmask = __ballot(queue);
            if (qmask) {
                const int leader = __ffsll((unsigned long long)qmask) - 1;
                int lslot = 0;
                if (lane == leader) lslot = atomicAdd(&lcnt[rr], __popcll(qmask));
                lslot = __shfl(lslot, leader);
                if (queue) lq[rr * WAVES * kWaveRows + lslot + __popcll(qmask & ((1ull << lane) - 1ull))] = (int)row;
            }
        }
        __syncthreads();
        // blocks of a set go round its segments
        const int64_t seg = ((int64_t)(slice / sl.sets) * sl.blocks + slice_block) % kSegs;
        if (tid < nrb) lbase[tid] = lcnt[tid] > 0 ? atomicAdd(&count_out[(int64_t)tid * kSegs + seg], lcnt[tid]) : 0;
        __syncthreads();
        for (int rr = 0; rr < nrb; ++rr) {
            int* dst = list_out + ((int64_t)rr * kSegs + seg) * seg_cap + lbase[rr];
            for (int i = tid; i < lcnt[rr]; i += WAVES * 64) dst[i] = lq[rr * WAVES * kWaveRows + i];
        }
    } else {
        for (int rr = 0; rr < nrb; ++rr) {
            const uint16_t id = w[rr];
            const bool queue = valid && id == kUnsettled;
            if (valid) bucket_cols[row * n_r + rr] = id == kUnsettled ? 0 : (int32_t)id;
            // wave-aggregated append to this round's list
            const uint64_t qmask = __ballot(queue);
            if (qmask) {
                int* list = list_out + sl.set_rows * rr;
                const int leader = __ffsll((unsigned long long)qmask) - 1;
                int lslot = 0;
                if (lane == leader) lslot = atomicAdd(&count_out[rr], __popcll(qmask));
                lslot = __shfl(lslot, leader);
                if (queue) list[lslot + __popcll(qmask & ((1ull << lane) - 1ull))] = (int)row;
            }
        }
    }
    if (MODE != kListed) break;
    __syncthreads();  // the next chunk restages R over the buffers just read
    }
}

struct HashWs {
    uint16_t* r_hi;
    uint16_t* r_mid;
    float* r_t;       // R as given, [n_r][half_pad][64] (columns contiguous, zero padded)
    float* col_norm;  // [3][n_r][half_pad]: |R_c|, |R_c - hi_c|, |R_c - hi_c - mid_c|
    float* norm_max;  // [3][n_r]: the largest of each
    int* r_exp;       // [n_r]: binary16 planes hold R * 2^r_exp (bf16 input)
    int* count;       // [n_r][kSegs] rows left open by the screen, then [n_r] by the exact passes
    int* list1;       // [n_r][kSegs][seg_cap]
    int* list2;       // [n_r][rows]
    int64_t seg_cap;
    size_t bytes;
};

constexpr int kHashWaves = 4;
constexpr int64_t kRowsPerBlock = kHashWaves * 64;

// n_rounds: the rounds of all sets; rows, blocks: those of one set.
HashWs carve(void* base, int64_t rows, int64_t blocks, int n_rounds, int half_pad) {
    const size_t per = (size_t)n_rounds * half_pad * kHeadDim;
    char* p = static_cast<char*>(base);
    HashWs w{};
    w.seg_cap = (blocks + kSegs - 1) / kSegs * kRowsPerBlock;
    size_t off = 0;
    w.r_hi = reinterpret_cast<uint16_t*>(p + off);
    off += align256(per * 2);
    w.r_mid = reinterpret_cast<uint16_t*>(p + off);
    off += align256(per * 2);
    w.r_t = reinterpret_cast<float*>(p + off);
    off += align256(per * 4);
    w.col_norm = reinterpret_cast<float*>(p + off);
    off += align256((size_t)3 * n_rounds * half_pad * 4);
    w.norm_max = reinterpret_cast<float*>(p + off);
    off += align256((size_t)3 * n_rounds * 4);
    w.r_exp = reinterpret_cast<int*>(p + off);
    off += align256((size_t)n_rounds * 4);
    w.count = reinterpret_cast<int*>(p + off);
    off += align256((size_t)n_rounds * (kSegs + 1) * 4);
    w.list1 = reinterpret_cast<int*>(p + off);
    off += align256((size_t)n_rounds * kSegs * w.seg_cap * 4);
    w.list2 = reinterpret_cast<int*>(p + off);
    off += align256((size_t)n_rounds * rows * 4);
    w.bytes = off;
    return w;
}

// Arguments of one pass of hash_kernel.
struct PassArgs {
    const void* q;
    Slices slices;
    int n_r, half, half_pad;
    const uint16_t *r_hi, *r_mid;
    const float *cn_max, *res;
    float err_acc;
    const float* res2;
    float err_acc2, err_pack;
    const float* col_res;
    int32_t* buckets;
    const int *list_in, *count_in;
    int *list_out, *count_out;
    int64_t seg_cap;
};

template <bool F32, int MODE, int WAVES, int ST>
void launch_pass_st(const PassArgs& a, dim3 grid, int rounds, hipStream_t stream) {
    constexpr int NP = MODE == kScreen ? 1 : 2;
    const size_t lds = hash_win_offset(Stage<NP, ST>::kBytes, WAVES, rounds) + (size_t)WAVES * 64 * rounds * 2;
    auto* k = &hash_kernel<F32, MODE, WAVES, ST>;
    (void)hipFuncSetAttribute(reinterpret_cast<const void*>(k), hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    k<<<grid, WAVES * 64, lds, stream>>>(a.q, a.slices, a.n_r, a.half, a.half_pad, a.r_hi, a.r_mid, a.cn_max, a.res,
                                         a.err_acc, a.res2, a.err_acc2, a.err_pack, a.col_res, a.buckets, a.list_in,
                                         a.count_in, a.list_out, a.count_out, a.seg_cap);
}

// Tiles per stage: the round's tile count rounded up to a power of two, at
// most kScreenMaxTiles for the screen (one plane), 8 for the fp32 pass (two
// planes) and 2 for bf16 input's two planes (240 registers, two waves a
// SIMD; four tiles take 337, one wave a SIMD, and were slower).
template <bool F32, int MODE, int WAVES>
void launch_pass(const PassArgs& a, dim3 grid, int rounds, hipStream_t stream) {
    constexpr int kMax = MODE == kScreen ? kScreenMaxTiles : (F32 ? 8 : 2);
    const int tpr = a.half_pad / 32;
    if (tpr <= 1)
        launch_pass_st<F32, MODE, WAVES, 1>(a, grid, rounds, stream);
    else if (tpr <= 2 || kMax == 2)
        launch_pass_st<F32, MODE, WAVES, 2>(a, grid, rounds, stream);
    else if (tpr <= 4 || kMax == 4) {
        if constexpr (kMax >= 4) launch_pass_st<F32, MODE, WAVES, 4>(a, grid, rounds, stream);
    } else {
        if constexpr (kMax >= 8) launch_pass_st<F32, MODE, WAVES, 8>(a, grid, rounds, stream);
    }
}

}  // namespace

namespace {

// How a call's rows fall into slices and R sets.  With one R per head, the
// heads are hashed together, up to kMaxSetRounds rounds of R at a time (which
// bounds the planes' workspace at 256 MiB).
constexpr int kMaxSetRounds = 1024;

// bf16 calls of at most this many projections (rows x rounds x columns) take
// both planes of R at once: twice the products, but no pass over the rows a
// screen leaves open, which costs 10 us however few they are.  Whole hash,
// one pass against screen and listed pass: 30.4 / 38.3 us at 8 M projections,
// 39.2 / 43.3 at 32 M, 65.9 / 58.8 at 72 M, 78.7 / 70.2 at 128 M.  With one R
// per head the line lies lower for few columns and higher for more: 16 heads of
// 64 buckets 53 / 59 at 30 M and 72 / 67 at 39 M, 8 of 192 buckets 51 / 67 at
// 42 M and 122 / 104 at 150 M; for 8 of 1024 buckets, few rows each, the screen is
// the faster one at every size (129 / 111 at 10 M, 130 / 113 at 39 M).
constexpr int64_t kSmallProjections = (int64_t)40 << 20;

Slices slices_of(int64_t BH, int L, int heads, int n_rounds) {
    Slices s{};
    if (heads == 0) {  // one R
        s.rows = BH * L;
        s.heads = s.sets = 1;
        s.set_rows = s.rows;
    } else {
        s.rows = L;
        s.heads = heads;
        s.sets = std::min(heads, std::max(1, kMaxSetRounds / n_rounds));
        s.set_rows = BH / heads * L;
    }
    s.blocks = (int)((s.rows + kRowsPerBlock - 1) / kRowsPerBlock);
    return s;
}

HashWs carve(void* base, const Slices& s, int n_rounds, int half_pad) {
    return carve(base, s.set_rows, s.set_rows / s.rows * s.blocks, s.sets * n_rounds, half_pad);
}

template <bool F16>
void launch_prep(const float* R, int rounds, int half, int half_pad, const HashWs& w, hipStream_t stream) {
    const int blocks = (half_pad + kPrepCols - 1) / kPrepCols;
    prep_r_kernel<F16><<<dim3(blocks, rounds), kPrepThreads, 0, stream>>>(
        R, half, half_pad, w.r_exp, w.r_hi, w.r_mid, w.r_t, w.col_norm, w.norm_max, w.count, kSegs,
        w.count + (size_t)rounds * kSegs);
    if (blocks > 1) prep_r_max_kernel<<<dim3(rounds, 3), 512, 0, stream>>>(w.col_norm, rounds, half_pad, w.norm_max);
}

// Hash the slices of `sl` (all heads, or a group of them; `all` sizes the
// workspace) with their R sets.
hipError_t launch_hash_sets(const void* q, bool f32, const Slices& sl, const Slices& all, int n_rounds, int half,
                            int half_pad, const float* R, int32_t* buckets, void* workspace, hipStream_t stream) {
    const int rounds = sl.sets * n_rounds;
    HashWs w = carve(workspace, all, n_rounds, half_pad);
    R += (size_t)sl.head0 * n_rounds * kHeadDim * half;
    const float* cn_max = w.norm_max;                  // max |R_c|
    const float* res1_max = w.norm_max + rounds;       // max |R_c - hi_c|
    const float* res2_max = w.norm_max + 2 * rounds;   // max |R_c - hi_c - mid_c|
    int* count1 = w.count;                             // [rounds][kSegs]: left open by the screen
    int* count2 = w.count + (size_t)rounds * kSegs;    // [rounds]: left to the fp64 refinement
    if (f32)
        launch_prep<false>(R, rounds, half, half_pad, w, stream);
    else
        launch_prep<true>(R, rounds, half, half_pad, w, stream);

    // Error of a screened key against the exact |projection| p_c, beyond the
    // planes' residual q . (R_c - planes) <= |q| |R_c - planes|:
    //  * fp32 accumulation of the exact 16-bit products, <= one ulp of the
    //    partial sum (<= 2^-23 sum_t |q_t R_tc|) per addition;
    //  * for bf16 input, the scaled q's values below 2^-14 that binary16
    //    drops: |delta q| <= 8 * 2^-14 <= 2^-25 |q| (|q| >= 2^14 scaled);
    //  * for fp32 input, q's own residual after two bf16 planes and R's
    //    after two (<= 3.1 * 2^-16 sum_t |q_t R_tc| together);
    //  * the index bits written over the low mantissa, < 2^-19 |key| for
    //    fp32 input (4 bits), < 2^-17 |key| for bf16 input (6 bits).
    // sum_t |q_t R_tc| <= |q| |R_c| (Cauchy-Schwarz) <= |q| max_c |R_c|.
    const float err_pack = f32 ? (float)0x1p-19 : (float)0x1p-17;
    const float acc1 = (float)((kHeadDim * 0x1p-23 + 0x1p-25) * 1.01);
    const float acc2 = (float)((2 * kHeadDim * 0x1p-23 + 0x1p-25) * 1.01);
    const float acc_f32 = (float)((3.1 * 0x1p-16 + 3 * kHeadDim * 0x1p-23) * 1.01);

    constexpr int kWaves = kHashWaves;
    const int64_t n_slices = sl.set_rows / sl.rows * sl.sets;
    const unsigned grid = (unsigned)(n_slices * sl.blocks);
    // Refinement blocks: one per CU over all rounds.  A typical list holds 0.1% of
    // the rows (64 groups of 16 at 1M rows).
    const unsigned refine_blocks = (unsigned)std::max<int64_t>(
        1, std::min<int64_t>(std::max(1, 256 / rounds), (sl.set_rows + kRefineGroup - 1) / kRefineGroup));
    if (f32) {
        launch_pass<true, kExact, kWaves>(
            PassArgs{q, sl, n_rounds, half, half_pad, w.r_hi, w.r_mid, cn_max, nullptr, acc_f32, nullptr, 0.f,
                     err_pack, nullptr, buckets, nullptr, nullptr, w.list2, count2, 0},
            dim3(grid), n_rounds, stream);
        hash_refine_kernel<true><<<dim3(refine_blocks, rounds), kRefineThreads, 0, stream>>>(
            q, w.r_t, half, half_pad, n_rounds, sl.set_rows, w.list2, count2, cn_max, nullptr, buckets);
    } else if (sl.set_rows * sl.sets * n_rounds * half_pad <= kSmallProjections) {
        // both planes at once
        launch_pass<false, kExact, kWaves>(
            PassArgs{q, sl, n_rounds, half, half_pad, w.r_hi, w.r_mid, cn_max, res2_max, acc2, res2_max, acc2,
                     err_pack, nullptr, buckets, nullptr, nullptr, w.list2, count2, 0},
            dim3(grid), n_rounds, stream);
        hash_refine_kernel<false><<<dim3(refine_blocks, rounds), kRefineThreads, 0, stream>>>(
            q, w.r_t, half, half_pad, n_rounds, sl.set_rows, w.list2, count2, cn_max, w.r_exp, buckets);
    } else {
        // screen with R's hi plane; the rows it leaves open get both planes;
        // what those leave open gets the fp64 refinement
        launch_pass<false, kScreen, kWaves>(
            PassArgs{q, sl, n_rounds, half, half_pad, w.r_hi, w.r_mid, cn_max, res1_max, acc1, res2_max, acc2,
                     err_pack, w.col_norm + (size_t)rounds * half_pad, buckets, nullptr, nullptr, w.list1, count1,
                     w.seg_cap},
            dim3(grid), n_rounds, stream);
        // Four waves a workgroup.  Deciding from the hi plane alone, the
        // screen leaves about 1.5% of row-rounds open on Gaussian data:
        // 128 workgroups per round cover 128 * 256 open rows, 3.1% of 1M
        // rows; longer lists loop.
        constexpr int kListedWaves = 4;
        const int64_t listed_rows = kListedWaves * 64;
        const unsigned per_round = (unsigned)std::min<int64_t>(std::min(128, std::max(4, 1024 / rounds)),
                                                               (sl.set_rows + listed_rows - 1) / listed_rows);
        launch_pass<false, kListed, kListedWaves>(
            PassArgs{q, sl, n_rounds, half, half_pad, w.r_hi, w.r_mid, cn_max, res2_max, acc2, res2_max, acc2,
                     err_pack, nullptr, buckets, w.list1, count1, w.list2, count2, w.seg_cap},
            dim3(per_round, 1, rounds), 1, stream);
        hash_refine_kernel<false><<<dim3(refine_blocks, rounds), kRefineThreads, 0, stream>>>(
            q, w.r_t, half, half_pad, n_rounds, sl.set_rows, w.list2, count2, cn_max, w.r_exp, buckets);
    }
    return hipGetLastError();
}

}  // namespace

size_t hash_workspace_bytes(int64_t BH, int L, int heads, int n_rounds, int n_buckets) {
    const int half_pad = (n_buckets / 2 + 31) / 32 * 32;
    return carve(nullptr, slices_of(BH, L, heads, n_rounds), n_rounds, half_pad).bytes;
}

hipError_t launch_hash(const void* q, bool f32, int64_t BH, int L, int heads, int n_rounds, int n_buckets,
                       const float* R, int32_t* buckets, void* workspace, hipStream_t stream) {
    const int half = n_buckets / 2;
    const int half_pad = (half + 31) / 32 * 32;
    if (BH == 0 || L == 0) return hipSuccess;
    Slices sl = slices_of(BH, L, heads, n_rounds);
    if (sl.head0 + sl.sets < sl.heads) {  // groups of heads, one after another
        for (int h = 0; h < heads; h += sl.sets) {
            Slices part = sl;
            part.head0 = h;
            part.sets = std::min(sl.sets, heads - h);
            const hipError_t e = launch_hash_sets(q, f32, part, sl, n_rounds, half, half_pad, R, buckets, workspace, stream);
            if (e != hipSuccess) return e;
        }
        return hipSuccess;
    }
    return launch_hash_sets(q, f32, sl, sl, n_rounds, half, half_pad, R, buckets, workspace, stream);
}

}  // namespace lsh
