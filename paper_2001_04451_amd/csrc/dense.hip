// Full shared-QK attention, forward: the memory-efficient baseline of Sec. 2
// (every query's softmax over all keys, without materialising QK^T), which
// the LSH forward approximates and which the paper's speed-versus-length
// comparison (Sec. 5) sets it against.  Keys are k_j = q_j/|q_j|; the logit
// of query i and key j is scale*q_i.k_j, the self key j == i carries the
// App. A mask (its weight exp(-1e5) vanishes in fp32 whenever the query has
// another key; without one the output is v_i and the log-partition is
// scale*|q_i| - self_mask), and under causal masking no later key counts.
//
// gfx950 design.  A workgroup of four waves owns 64 QT consecutive queries of
// one (batch, head); each wave holds QT 16-query tiles as matrix-core B
// operands in registers for the whole kernel.  The workgroup walks the keys in
// blocks of 64: the next block's k and v rows and key scales are copied from
// global memory straight into the free half of a double-buffered LDS area
// (global_load_lds) while the current block is used, with one barrier per
// block.  Per 32 keys and query tile the scores come as S^T = K Q^T (two
// 16-key tiles, mfma_f32_16x16x32_bf16: lane l holds keys 4(l/16)..+3 of query
// l%16), the softmax weights are packed to bf16 in place, and the lane's eight
// weights are the B operand of O^T += V^T P^T on the same instruction, with
// V^T read through the LDS transpose read in the same key order.  One more
// product, with ones, gives the sums of the bf16 weights.  As in the chunked
// kernel, no running maximum is needed while the logit bound
// B_i = scale*log2(e)*|q_i| (Cauchy-Schwarz: every logit lies in [-B_i, B_i])
// of the workgroup's queries is at most 60, since exp2 then neither overflows
// nor underflows; workgroups with a larger bound keep the online maximum.
// Masks are applied only in blocks that hold one of the wave's own positions
// or the sequence end; under causal masking a wave stops after the block
// holding its last query.
//
// Bound by the matrix cores and the exponentials, which two waves a SIMD only
// partly overlap (1.09 PFLOP/s of useful products at 16 heads of 32K, causal).
// Against the earlier kernel (32 queries a wave, P V on 16x16x16 products at
// half the rate, both softmax forms in one loop with their addresses spilled,
// workgroups numbered query block by query block over the XCDs): 32 heads of
// 8K, causal, 576 -> 285 us.  Of that, the products and the split loops gave
// 576 -> 398 with QT = 2 (by XCD), QT = 4 -> 350, the order of the causal
// query blocks -> 285.
#include "attn_common.h"
#include "launch.h"

namespace lsh {
namespace {

constexpr int kDenseWaves = 4;
constexpr int kKeyBlock = 64;
constexpr float kDenseFastBound = 60.f;
constexpr int kSwz = 1;  // LDS row layout (attn_common.h): 16-row operand reads
constexpr bf16x8 kOnes8 = {(__bf16)1.0f, (__bf16)1.0f, (__bf16)1.0f, (__bf16)1.0f,
                           (__bf16)1.0f, (__bf16)1.0f, (__bf16)1.0f, (__bf16)1.0f};

struct DenseShared {
    char Ks[2][kKeyBlock * 128];  // k rows (the stored q), swizzled 16-byte pieces
    char Vs[2][kKeyBlock * 128];  // v rows, same layout
    float cf[2][kKeyBlock];       // scale*log2(e)/|q_j|, 0 for a zero row
};

template <bool B>
struct Tag {
    static constexpr bool value = B;
};

// Key scale of every row: scale*log2(e)/|q_j| (0 for a zero row, whose key is
// the zero vector).  Eight lanes per row, 16 bytes each.
__global__ __launch_bounds__(256) void dense_prep_kernel(const uint16_t* __restrict__ q,
                                                         float* __restrict__ cf, int64_t rows,
                                                         float scale_log2e) {
    const int64_t row = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) >> 3;
    const int part = threadIdx.x & 7;
    if (row >= rows) return;  // whole 8-lane groups leave
    const u32x4 x = *reinterpret_cast<const u32x4*>(q + row * kHeadDim + part * 8);
    float ss = 0.f;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const float a = __uint_as_float(x[e] << 16), b = __uint_as_float(x[e] & 0xFFFF0000u);
        ss = fmaf(a, a, fmaf(b, b, ss));
    }
    ss += __shfl_xor(ss, 1);
    ss += __shfl_xor(ss, 2);
    ss += __shfl_xor(ss, 4);
    if (part == 0) cf[row] = ss > 0.f ? scale_log2e / sqrtf(ss) : 0.f;
}

template <bool CAUSAL, int QT, int OCC>
__global__ __launch_bounds__(256, OCC) void dense_attn_fwd_kernel(
    const uint16_t* __restrict__ q, const uint16_t* __restrict__ v, const float* __restrict__ cf,
    uint16_t* __restrict__ out, float* __restrict__ lse, int64_t BH, int L, int sets, float scale_log2e, float self_mask) {
    constexpr int kWaveQueries = 16 * QT, kQueries = kDenseWaves * kWaveQueries;
    __shared__ __attribute__((aligned(16))) DenseShared S;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int n = lane & 15, g = lane >> 4;
    // Query block and slice of the workgroup (see launch_dense_fwd).
    const int n_qb = (L + kQueries - 1) / kQueries;
    const int xcd = (int)(blockIdx.x % kXcds);
    const int slices = (int)(BH / sets);  // of this XCD's set
    constexpr int kGroup = CAUSAL ? 8 : 1;
    const int64_t item = (int64_t)(blockIdx.x / kXcds) * (kXcds / sets) + xcd / sets;
    if (item >= (int64_t)slices * n_qb) return;
    const int group0 = (int)(item / ((int64_t)kGroup * n_qb)) * kGroup;
    const int group = min(kGroup, slices - group0);
    const int in_group = (int)(item - (int64_t)group0 * n_qb);
    const int64_t bh = (int64_t)(group0 + in_group % group) * sets + xcd % sets;
    const int qb = CAUSAL ? n_qb - 1 - in_group / group : in_group / group;  // longest first
    const int q0 = qb * kQueries;
    const int qw0 = q0 + kWaveQueries * wave;  // this wave's first query
    const uint16_t* qh = q + bh * L * kHeadDim;
    const uint16_t* vh = v + bh * L * kHeadDim;
    const float* cfh = cf + bh * L;

    const int n_blocks = (L + kKeyBlock - 1) / kKeyBlock;
    // blocks the workgroup walks, and the last one this wave needs
    const int wg_end = CAUSAL ? (min(q0 + kQueries, L) - 1) / kKeyBlock + 1 : n_blocks;
    const bool active = qw0 < L;
    const int wave_end = !active ? 0 : (CAUSAL ? (min(qw0 + kWaveQueries, L) - 1) / kKeyBlock + 1 : n_blocks);

    // Query operands: lane holds query qw0 + 16qt + n, dims 32ks + 8g .. +7.
    bf16x8 qop[QT][2];
    float bound[QT];
    bool small = true;
#pragma unroll
    for (int qt = 0; qt < QT; ++qt) {
        const int row = min(qw0 + 16 * qt + n, L - 1);
        float ss = 0.f;
#pragma unroll
        for (int ks = 0; ks < 2; ++ks) {
            const u32x4 x = *reinterpret_cast<const u32x4*>(qh + (int64_t)row * kHeadDim + 32 * ks + 8 * g);
            qop[qt][ks] = as_bf16x8(x);
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const float a = __uint_as_float(x[e] << 16), b = __uint_as_float(x[e] & 0xFFFF0000u);
                ss = fmaf(a, a, fmaf(b, b, ss));
            }
        }
        ss += __shfl_xor(ss, 16);
        ss += __shfl_xor(ss, 32);
        bound[qt] = scale_log2e * sqrtf(ss);
        small = small && bound[qt] <= kDenseFastBound;
    }

    // Stage key block kb into buffer b: wave w copies rows 16w .. 16w+15 of k
    // and of v (each lane the piece that belongs at its LDS slot), wave 0 the
    // 64 key scales.  Rows past L repeat row L-1 and are masked out.
    auto stage = [&](int kb, int b) {
#pragma unroll
        for (int k = 0; k < 2; ++k) {
            const int row = 16 * wave + 8 * k + (lane >> 3);
            const int key = min(kb * kKeyBlock + row, L - 1);
            const int64_t off = (int64_t)key * kHeadDim + swz<kSwz>(row, lane & 7) * 8;
            copy16_to_lds(qh + off, S.Ks[b] + (16 * wave + 8 * k) * 128);
            copy16_to_lds(vh + off, S.Vs[b] + (16 * wave + 8 * k) * 128);
        }
        if (wave == 0) copy4_to_lds(cfh + min(kb * kKeyBlock + lane, L - 1), &S.cf[b][0]);
    };

    float m[QT];  // running maxima (slow path)
    f32x4 oacc[QT][4];
    f32x4 osum[QT];  // sums of the bf16 weights (the same in every register and lane group)
#pragma unroll
    for (int qt = 0; qt < QT; ++qt) {
        m[qt] = -__builtin_inff();
        osum[qt] = f32x4{};
#pragma unroll
        for (int dt = 0; dt < 4; ++dt) oacc[qt][dt] = f32x4{};
    }

    // One key block for the wave's query tiles.  EDGE: the block holds one of
    // the wave's own positions or the sequence end, so keys are tested one by
    // one.  Two 16-key tiles at a time: the lane's four keys of each, side by
    // side, are the eight k-slots of one 16x16x32 product with V^T, whose
    // operand takes its rows in the same order.
    auto attend = [&](const char* Ks, const char* Vs, const float* cfb, int kb, auto fast_tag,
                      auto edge_tag) {
        constexpr bool FAST = decltype(fast_tag)::value;
        constexpr bool EDGE = decltype(edge_tag)::value;
#pragma unroll
        for (int kp = 0; kp < 2; ++kp) {
            bf16x8 k0[2], k1[2];
            f32x4 cfk[2];
#pragma unroll
            for (int t = 0; t < 2; ++t) {
                const int r0 = 32 * kp + 16 * t;
                k0[t] = as_bf16x8(lds_piece<kSwz>(Ks, r0 + n, g));
                k1[t] = as_bf16x8(lds_piece<kSwz>(Ks, r0 + n, 4 + g));
                cfk[t] = *reinterpret_cast<const f32x4*>(cfb + r0 + 4 * g);
            }
            bf16x8 pk[QT];
#pragma unroll
            for (int qt = 0; qt < QT; ++qt) {
                f32x4 acc[2];
#pragma unroll
                for (int t = 0; t < 2; ++t) {
                    acc[t] = mfma16x16x32(k0[t], qop[qt][0], f32x4{});
                    acc[t] = mfma16x16x32(k1[t], qop[qt][1], acc[t]);
                }
                const int query = qw0 + 16 * qt + n;
#pragma unroll
                for (int t = 0; t < 2; ++t)
#pragma unroll
                    for (int j = 0; j < 4; ++j) {
                        acc[t][j] *= cfk[t][j];
                        if constexpr (EDGE) {
                            const int key = kb * kKeyBlock + 32 * kp + 16 * t + 4 * g + j;
                            const bool ok = key < L && (CAUSAL ? key < query : key != query);
                            acc[t][j] = ok ? acc[t][j] : -__builtin_inff();
                        }
                    }
                float off = 0.f;
                if constexpr (!FAST) {  // online maximum over the four lane groups of a query
                    float mt = fmaxf(fmaxf(fmaxf(acc[0][0], acc[0][1]), fmaxf(acc[0][2], acc[0][3])),
                                     fmaxf(fmaxf(acc[1][0], acc[1][1]), fmaxf(acc[1][2], acc[1][3])));
                    mt = max_xor32(max_xor16(mt));
                    const float m_new = fmaxf(m[qt], mt);
                    off = m_new > -__builtin_inff() ? m_new : 0.f;
                    const float corr = __builtin_amdgcn_exp2f(m[qt] - off);
                    osum[qt] *= corr;
#pragma unroll
                    for (int dt = 0; dt < 4; ++dt) oacc[qt][dt] *= corr;
                    m[qt] = m_new;
                }
                u32x4 pw;
#pragma unroll
                for (int t = 0; t < 2; ++t)
#pragma unroll
                    for (int h2 = 0; h2 < 2; ++h2)
                        pw[2 * t + h2] = pack_bf16x2(__builtin_amdgcn_exp2f(acc[t][2 * h2] - off),
                                                     __builtin_amdgcn_exp2f(acc[t][2 * h2 + 1] - off));
                pk[qt] = as_bf16x8(pw);
                osum[qt] = mfma16x16x32(kOnes8, pk[qt], osum[qt]);
            }
#pragma unroll
            for (int dt = 0; dt < 4; ++dt) {
                const bf16x8 vt = cat4(vt_read(Vs + vt_offset<kSwz>(32 * kp, 16 * dt, lane)),
                                       vt_read(Vs + vt_offset<kSwz>(32 * kp + 16, 16 * dt, lane)));
#pragma unroll
                for (int qt = 0; qt < QT; ++qt) oacc[qt][dt] = mfma16x16x32(vt, pk[qt], oacc[qt][dt]);
            }
        }
    };

    stage(0, 0);
    __builtin_amdgcn_s_waitcnt(0);
    const bool fast = __syncthreads_and(small);
    // The walk over the key blocks, built for each of the two softmax forms
    // (the choice inside the loop kept both forms' addresses in registers and
    // spilled 82 of them).
    auto walk = [&](auto fast_tag) {
        for (int kb = 0; kb < wg_end; ++kb) {
            const int b = kb & 1;
            if (kb + 1 < wg_end) stage(kb + 1, b ^ 1);
            if (kb < wave_end) {
                const int k_lo = kb * kKeyBlock;
                if (k_lo + kKeyBlock > L || (k_lo + kKeyBlock > qw0 && k_lo < qw0 + kWaveQueries))
                    attend(S.Ks[b], S.Vs[b], S.cf[b], kb, fast_tag, Tag<true>{});
                else
                    attend(S.Ks[b], S.Vs[b], S.cf[b], kb, fast_tag, Tag<false>{});
            }
            __builtin_amdgcn_s_waitcnt(0);  // this wave's copies of block kb+1 have landed
            __syncthreads();                // ... and every wave is done with block kb
        }
    };
    if (fast)
        walk(Tag<true>{});
    else
        walk(Tag<false>{});
    if (!active) return;

    // Lane holds O^T[d = 16dt + 4g + e][query qw0 + 16qt + n].
#pragma unroll
    for (int qt = 0; qt < QT; ++qt) {
        const int query = qw0 + 16 * qt + n;
        const float l = osum[qt][0];
        if (query >= L) continue;
        uint16_t* orow = out + (bh * L + query) * kHeadDim;
        if (l > 0.f) {
            const float inv = __builtin_amdgcn_rcpf(l);
#pragma unroll
            for (int dt = 0; dt < 4; ++dt) {
                const uint2 w = make_uint2(pack_bf16x2(oacc[qt][dt][0] * inv, oacc[qt][dt][1] * inv),
                                           pack_bf16x2(oacc[qt][dt][2] * inv, oacc[qt][dt][3] * inv));
                *reinterpret_cast<uint2*>(orow + 16 * dt + 4 * g) = w;
            }
            if (lse && g == 0) lse[bh * L + query] = ((fast ? 0.f : m[qt]) + __log2f(l)) * kLn2;
        } else {
            // the query's only key is itself: output v_i
            const uint16_t* vrow = vh + (int64_t)query * kHeadDim;
#pragma unroll
            for (int dt = 0; dt < 4; ++dt)
                *reinterpret_cast<uint2*>(orow + 16 * dt + 4 * g) =
                    *reinterpret_cast<const uint2*>(vrow + 16 * dt + 4 * g);
            if (lse && g == 0) lse[bh * L + query] = bound[qt] * kLn2 - self_mask;
        }
    }
}

}  // namespace

size_t dense_workspace_bytes(int64_t BH, int L) { return align256((size_t)BH * L * sizeof(float)); }

hipError_t launch_dense_fwd(int64_t BH, int L, bool causal, float scale, float self_mask,
                            const void* q_, const void* v_, void* out_, float* lse, void* workspace,
                            hipStream_t stream) {
    if (BH == 0 || L == 0) return hipSuccess;
    const uint16_t* q = static_cast<const uint16_t*>(q_);
    const uint16_t* v = static_cast<const uint16_t*>(v_);
    uint16_t* out = static_cast<uint16_t*>(out_);
    float* cf = static_cast<float*>(workspace);
    const int64_t rows = BH * L;
    const float scale_log2e = scale * kLog2e;
    dense_prep_kernel<<<(unsigned)((rows * 8 + 255) / 256), 256, 0, stream>>>(q, cf, rows, scale_log2e);
    // Workgroups go to the XCDs in turn.  Each XCD takes whole slices, or where
    // BH is no multiple of the XCDs, kXcds / sets of them share one, so that
    // every XCD has the same work and its L2 few slices' keys.  Under causal
    // masking the query blocks of up to eight slices are interleaved, those
    // with the most keys first: the first workgroups of a CU and those that
    // follow them then add up alike (32 heads of 8K: 350 -> 285 us against
    // slice after slice, 64 of 4K: 209 -> 163).
    int sets = kXcds;
    while (BH % sets != 0) sets /= 2;
    auto go = [&](auto kernel, int queries) {
        const int64_t items = (int64_t)((L + queries - 1) / queries) * (BH / sets);
        const int per = kXcds / sets;
        kernel<<<(unsigned)((items + per - 1) / per * kXcds), 256, 0, stream>>>(q, v, cf, out, lse, BH, L, sets,
                                                                               scale_log2e, self_mask);
    };
    // 64 queries a wave read each key from LDS a quarter as often as 16 do, but
    // give a quarter of the workgroups, two to a CU.  Measured in us, 256 against
    // 64 queries a workgroup (128 lay between them or equal to one): causal, 1024
    // workgroups of 256, 163 / 203; 512, 100 / 106; 256, 173 / 114; without a
    // mask, 512, 142 / 203; 256, 175 / 204; 128, 95 / 68.
    const int64_t wide = (int64_t)((L + 255) / 256) * BH;
    if (wide >= (causal ? 512 : 256))
        causal ? go(dense_attn_fwd_kernel<true, 4, 2>, 256) : go(dense_attn_fwd_kernel<false, 4, 2>, 256);
    else
        causal ? go(dense_attn_fwd_kernel<true, 1, 3>, 64) : go(dense_attn_fwd_kernel<false, 1, 3>, 64);
    return hipGetLastError();
}

}  // namespace lsh
