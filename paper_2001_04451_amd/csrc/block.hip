// The reversible block around LSH attention (Reformer Sec. 3, "RevNets",
// "Reversible Transformer" and "Chunking"): the layer normalisations inside
// the residual branches and the block's dense products.  The attention
// itself is the library's LSH forward; the block's entry points (block_api.cpp)
// chain these kernels with it.
//
// LayerNorm: one wave per row, the row held in registers, mean and variance
// in fp32 by wave reductions, bf16 output (the products' operand precision).
//
// Products: C = A W^T with A the activations (rows of K bf16 values, or the
// attention's output in its [B, H, L, 64] layout) and W a weight matrix
// [N][K] in bf16, fp32 accumulation on the matrix cores
// (mfma_f32_16x16x32_bf16), W as the first operand (a lane ends up with four
// consecutive output columns of one row).  A workgroup of four waves computes
// a square tile of C of 256, 128 or 64 (by the tile count, launch_gemm); A
// and W pass through a ring of LDS stages of 64 k-values, copied there by
// buffer loads and counted by hand, and each wave holds the next stage's
// operands in registers by the time it needs them: one barrier a stage, no
// wait on an LDS read.  What bounded the earlier kernel (128 x 128, two
// buffers, operands read when needed; 650-750 TFLOP/s) was the copies: 64
// bytes a cycle into a CU are as long as the products of a 128 x 128 tile.  A
// 256 x 256 tile needs half of that; its single wave per SIMD then must not
// issue anything in a row, so every copy and operand read stands alone between
// two products.  16384 x 1024 x 4096 with residual: 173 -> 119 us (1.15
// PFLOP/s), 16384 x 4096 x 1024 to bf16: 183 -> 153 us, 65536 x 1024 x 1024
// with residual (0.67 GB): 320 -> 215 us; 4095 x 512 x 2048: 38 -> 17 us.
// Workgroups are numbered so that an XCD works on a block of row and column
// tiles at a time and reads their rows of A and W from
// memory once.  The epilogue adds the bias and either
//  * adds the product, times a sign, to an fp32 residual (the branch outputs:
//    y = x + F or x = y - F),
//  * applies ReLU and stores bf16 (the feed-forward's hidden layer), or
//  * stores bf16 q or v in the attention's [B, H, L, 64] layout.
#include "attn_common.h"
#include "launch.h"

#include <type_traits>

namespace lsh {
namespace {

// ---------------------------------------------------------------------------
// LayerNorm

constexpr int kLnMaxPairs = 32;  // rows of up to 64 x 2 x 32 = 4096 values

__device__ __forceinline__ float wave_sum(float x) {
    // butterfly: every lane ends with the same (commutative) sums
    for (int o = 32; o >= 1; o >>= 1) x += __shfl_xor(x, o);
    return x;
}

// PAIRS: value pairs per lane, rounded up to a power of two; loads past the
// row's own repeat its last pair, so that a row's loads are unconditional and
// all in flight together (under conditions each waited for the one before:
// the ten calls of a block forward and inverse at 65,536 x 1024 took 657 us,
// now 372).
template <int PAIRS>
__global__ __launch_bounds__(256) void layer_norm_kernel(const float* __restrict__ x, const float* __restrict__ g,
                                                         const float* __restrict__ b, uint32_t* __restrict__ out,
                                                         int64_t rows, int D, float eps) {
    const int lane = threadIdx.x & 63;
    const int64_t row = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
    if (row >= rows) return;  // uniform per wave
    const int P = D / 128;    // value pairs per lane
    const float2* xr = reinterpret_cast<const float2*>(x + row * D);
    const float2* g2 = reinterpret_cast<const float2*>(g);
    const float2* b2 = reinterpret_cast<const float2*>(b);
    float2 v[PAIRS];
    float s = 0.f;
#pragma unroll
    for (int i = 0; i < PAIRS; ++i) v[i] = xr[lane + 64 * min(i, P - 1)];
#pragma unroll
    for (int i = 0; i < PAIRS; ++i)
        if (i < P) s += v[i].x + v[i].y;
    const float mu = wave_sum(s) / (float)D;
    float ss = 0.f;
#pragma unroll
    for (int i = 0; i < PAIRS; ++i)
        if (i < P) {
            const float dx = v[i].x - mu, dy = v[i].y - mu;
            ss += dx * dx + dy * dy;
        }
    const float rstd = 1.0f / sqrtf(wave_sum(ss) / (float)D + eps);
    uint32_t* orow = out + row * (D / 2);
#pragma unroll
    for (int i = 0; i < PAIRS; ++i)
        if (i < P) {
            const int c = lane + 64 * i;
            const float2 gg = g2[c], bb = b2[c];
            orow[c] = pack_bf16x2((v[i].x - mu) * rstd * gg.x + bb.x, (v[i].y - mu) * rstd * gg.y + bb.y);
        }
}

// ---------------------------------------------------------------------------
// Products

enum : int { kInRows = 0, kInHeads = 1 };                    // A layout
enum : int { kOutResid = 0, kOutReluBf16 = 1, kOutHeads = 2 };  // epilogue

struct GemmArgs {
    const uint16_t* a;      // [M][K] rows, or [B][H][L][64] (kInHeads: K = 64 H, M = B L)
    const uint16_t* w;      // [N][K]
    int64_t M;
    int N, K;
    int L, H;               // kInHeads / kOutHeads: sequence length and heads
    const float* bias;      // [N] or null
    const float* resid;     // kOutResid: [M][N] fp32 or null (then 0)
    float sign;             // kOutResid: out = resid + sign (A W^T + bias)
    float* out_f32;         // kOutResid: [M][N]
    uint16_t* out_bf16;     // kOutReluBf16: [M][N]; kOutHeads: [B][H][L][64]
};

// Raw buffer descriptor (word 3: raw, untyped 32-bit data).
__device__ __forceinline__ u32x4 raw_buffer(const void* p, uint64_t bytes) {
    const uint64_t a = (uint64_t)p;
    return u32x4{(uint32_t)a, (uint32_t)(a >> 32), bytes >= 0xFFFFFFFFull ? 0xFFFFFFFFu : (uint32_t)bytes, 0x00020000u};
}

// 16 bytes per lane from the buffer at byte v_off + s_off straight to LDS at
// lds + 16 * lane.  Inline assembly, so that the compiler neither orders LDS
// reads behind it nor waits for it: the kernel counts its own loads.
__device__ __forceinline__ void buffer_to_lds(u32x4 buf, uint32_t v_off, uint32_t s_off, uint32_t lds) {
    asm volatile("s_mov_b32 m0, %3\n\ts_nop 0\n\tbuffer_load_dwordx4 %0, %1, %2 offen lds" ::"v"(v_off), "s"(buf),
                 "s"(s_off), "s"(lds)
                 : "memory", "m0");
}

// Shape of one product kernel: a workgroup of four waves computes a TM x TN
// tile of C, each wave a quarter of TM / 2 x TN / 2 as 16 x 16 products.  A and
// W pass through LDS in stages of KB k-values, STAGES of them in flight.
template <int TM_, int TN_, int KB_, int STAGES_>
struct GemmShape {
    static constexpr int TM = TM_, TN = TN_, KB = KB_, STAGES = STAGES_;
    static constexpr int kPieces = KB / 8;             // 16-byte pieces per row
    static constexpr int kRowBytes = 2 * KB;
    static constexpr int kRunRows = 64 / kPieces;      // rows one copy instruction fills
    static constexpr int kStageBytes = (TM + TN) * kRowBytes;
    static constexpr int kLoadsA = TM / kRunRows / 4, kLoadsW = TN / kRunRows / 4;  // per wave and stage
    static constexpr int kLoads = kLoadsA + kLoadsW;
    static constexpr int MI = TM / 32, NI = TN / 32;   // 16-row blocks per wave
    static constexpr int KS = KB / 32;                 // k-steps per stage
    static constexpr size_t kLds = (size_t)STAGES * kStageBytes;
    // Slot of piece p of a row.  The LDS serves a 16-byte read in groups of
    // sixteen lanes, 0-3, 12-15, 20-23 and 24-27 the first of them (inferred
    // from SQ_LDS_BANK_CONFLICT under several layouts); under these slots a
    // group's rows and pieces meet all 64 banks once: no conflicts counted.
    static_assert(KB == 64, "slots and head offsets of 64 k-values");
    static __device__ __forceinline__ int slot(int row, int p) { return p ^ (row & 7); }
};

// Until at most N of the wave's loads are in flight and its LDS reads are
// done (as the builtin, so that the compiler knows of the latter).
template <int N>
__device__ __forceinline__ void wait_loads() {
    static_assert(N < 64, "vmcnt has six bits");
    __builtin_amdgcn_s_waitcnt((N & 15) | ((N >> 4) << 14) | (7 << 4));
    asm volatile("" ::: "memory");
}

// acc += a b, in place in the accumulation registers.  Inline assembly ties
// the result to the accumulator's registers: with the builtin the allocator
// gives results other registers than their addends and moves them back (350
// moves beside the 128 products of two stages at 256 accumulators a lane).
__device__ __forceinline__ void mfma_into(f32x4& acc, bf16x8 a, bf16x8 b) {
    asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+a"(acc) : "v"(a), "v"(b));
}

// Workgroup barrier alone (no wait for copies in flight); no LDS access moves
// across it.
__device__ __forceinline__ void barrier() {
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
}

template <class S, int IN, int OUT>
__global__ __launch_bounds__(256, (S::kLds > 80 * 1024 ? 1 : 2)) void gemm_bf16_kernel(GemmArgs g) {
    extern __shared__ __attribute__((aligned(16))) char smem[];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);

    // Tile of this workgroup (workgroup b runs on XCD b % 8): the tiles in bands
    // of an eighth of the row tiles, a band four columns of tiles at a time, and
    // each XCD a run of an eighth of that walk, so that the tiles in flight on it
    // share rows of A and of W in its L2.  For any number of row tiles: with
    // plain numbering where they were no multiple of eight, 12,100 x 512 x 2048
    // took 40.7 us against 33.6, 9000 x 1024 x 4096 124 against 103, 33,000 x
    // 1024 x 2048 226 against 189; multiples of eight as before.
    const int nN = g.N / S::TN;
    const int nM = (int)((g.M + S::TM - 1) / S::TM);
    int tm, tn;
    {
        const int tiles = nM * nN, xcd = (int)(blockIdx.x % 8);
        const int i = xcd * (tiles / 8) + min(xcd, tiles % 8) + (int)(blockIdx.x / 8);  // place in the walk
        const int mx = (nM + 7) / 8, band = i / (mx * nN), j = i - band * mx * nN;
        const int rows = min(mx, nM - band * mx);
        const int cg = j / (4 * rows), k = j - cg * 4 * rows, gn = min(4, nN - 4 * cg);
        tm = band * mx + k / gn;
        tn = 4 * cg + k % gn;
    }
    const int64_t m0 = (int64_t)tm * S::TM;
    const int n0 = tn * S::TN;
    const int n_st = g.K / S::KB;

    // Copies: lane l of a copy fills slot l % kPieces of row l / kPieces of a
    // run of kRunRows rows.  Rows past M repeat the last row (not stored).
    const u32x4 buf_a = raw_buffer(g.a, (uint64_t)g.M * g.K * 2), buf_w = raw_buffer(g.w, (uint64_t)g.N * g.K * 2);
    uint32_t off[S::kLoads];
    const int lrow = lane / S::kPieces, lslot = lane % S::kPieces;
#pragma unroll
    for (int j = 0; j < S::kLoadsA; ++j) {
        const int r = (wave * S::kLoadsA + j) * S::kRunRows + lrow;
        const int64_t m = min(m0 + r, g.M - 1);
        const uint32_t piece = 16u * (uint32_t)S::slot(r, lslot);
        if constexpr (IN == kInRows)
            off[j] = (uint32_t)(m * g.K * 2) + piece;
        else
            off[j] = (uint32_t)((m / g.L * g.H * g.L + m % g.L) * 128) + piece;
    }
#pragma unroll
    for (int j = 0; j < S::kLoadsW; ++j) {
        const int r = (wave * S::kLoadsW + j) * S::kRunRows + lrow;
        off[S::kLoadsA + j] = (uint32_t)((int64_t)(n0 + r) * g.K * 2) + 16u * (uint32_t)S::slot(r, lslot);
    }
    const uint32_t lds0 = lds_addr(smem);
    // copy j of stage st (into ring slot `ring`)
    auto load = [&](int st, int ring, int j) {
        const bool is_a = j < S::kLoadsA;
        uint32_t k_off;  // bytes along k: a head is 64 k-values
        if (IN == kInHeads && is_a)
            k_off = (uint32_t)st * (uint32_t)g.L * 128u;
        else
            k_off = (uint32_t)st * S::kRowBytes;
        const uint32_t run = is_a ? wave * S::kLoadsA + j : S::TM / S::kRunRows + wave * S::kLoadsW + (j - S::kLoadsA);
        buffer_to_lds(is_a ? buf_a : buf_w, off[j], k_off, lds0 + ring * S::kStageBytes + run * 1024);
    };

    // Operands: lane l reads row 16 i + l % 16 of its wave's rows, piece
    // 4 ks + l / 16 of k-step ks (the slots repeat every 16 rows).
    const int wm = wave & 1, wn = wave >> 1;
    uint32_t op[S::KS];
#pragma unroll
    for (int ks = 0; ks < S::KS; ++ks)
        op[ks] = (lane & 15) * S::kRowBytes + 16 * S::slot(lane & 15, 4 * ks + (lane >> 4));
    // W's operands meet every group of a stage's products and are
    // double-buffered; A's meet one group each, and the next stage's replace
    // them in place right after it.
    struct FragsW {
        bf16x8 w[S::KS][S::NI];
    };
    bf16x8 fa[S::KS][S::MI];
    auto read_a = [&](int ring, int ks, int i) {
        fa[ks][i] = as_bf16x8(*reinterpret_cast<const u32x4*>(
            smem + ring * S::kStageBytes + op[ks] + (wm * S::TM / 2 + 16 * i) * S::kRowBytes));
    };
    auto read_w = [&](FragsW& f, int ring, int ks, int i) {
        f.w[ks][i] = as_bf16x8(*reinterpret_cast<const u32x4*>(
            smem + ring * S::kStageBytes + op[ks] + (S::TM + wn * S::TN / 2 + 16 * i) * S::kRowBytes));
    };

    f32x4 acc[S::NI][S::MI];
#pragma unroll
    for (int i = 0; i < S::NI; ++i)
#pragma unroll
        for (int j = 0; j < S::MI; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};

    // Stage st: its operands are in `cur` (read from LDS during stage st - 1)
    // and its ring slot is free once every wave has passed the barrier, so
    // stage st + STAGES is copied there; stage st + 1, which has landed by
    // then, is read into `nxt`; both are spread between the products.
    auto stage = [&](int st, int ring, FragsW& cur, FragsW& nxt, auto steady) {
        constexpr bool STEADY = decltype(steady)::value;  // more stages to copy: no branches
        if (STEADY || st + S::STAGES - 1 < n_st)
            wait_loads<(S::STAGES - 2) * S::kLoads>();
        else
            wait_loads<0>();
        barrier();
        const bool more = STEADY || st + S::STAGES < n_st, next = STEADY || st + 1 < n_st;
        const int ring1 = ring + 1 == S::STAGES ? 0 : ring + 1;
        constexpr int kGroups = S::KS * S::MI;               // groups of NI products
        constexpr int kReadsW = S::KS * S::NI;
        // one copy or read at a time between two products, so that its issue
        // hides behind the product before it
        constexpr int kProducts = kGroups * S::NI;
        // a ring of two waits for these copies at the stage's end: early
        constexpr int kCopyProducts = S::STAGES == 2 ? kProducts * 5 / 8 : kProducts;
#pragma unroll
        for (int gi = 0; gi < kGroups; ++gi) {
            const int ks = gi / S::MI, j = gi % S::MI;
#pragma unroll
            for (int i = 0; i < S::NI; ++i) {
                const int u = gi * S::NI + i;
                __builtin_amdgcn_sched_barrier(0);
                mfma_into(acc[i][j], cur.w[ks][i], fa[ks][j]);
                if (more) {
#pragma unroll
                    for (int l = u * S::kLoads / kCopyProducts; l < (u + 1) * S::kLoads / kCopyProducts; ++l)
                        if (l < S::kLoads) load(st + S::STAGES, ring, l);
                }
                if (next) {
#pragma unroll
                    for (int l = u * kReadsW / kProducts; l < (u + 1) * kReadsW / kProducts; ++l)
                        read_w(nxt, ring1, l / S::NI, l % S::NI);
                    if (i == S::NI / 2 && gi > 0) read_a(ring1, (gi - 1) / S::MI, (gi - 1) % S::MI);
                }
            }
        }
        __builtin_amdgcn_sched_barrier(0);
        if (next) read_a(ring1, S::KS - 1, S::MI - 1);
    };

#pragma unroll
    for (int st = 0; st < S::STAGES; ++st)
        if (st < n_st) {
#pragma unroll
            for (int l = 0; l < S::kLoads; ++l) load(st, st, l);
        }
    if (n_st >= S::STAGES)
        wait_loads<(S::STAGES - 1) * S::kLoads>();
    else
        wait_loads<0>();
    barrier();
    FragsW f0, f1;
#pragma unroll
    for (int ks = 0; ks < S::KS; ++ks) {
#pragma unroll
        for (int i = 0; i < S::NI; ++i) read_w(f0, 0, ks, i);
#pragma unroll
        for (int i = 0; i < S::MI; ++i) read_a(0, ks, i);
    }
    int ring = 0, st = 0;
    for (; st + 1 + S::STAGES < n_st; st += 2) {
        stage(st, ring, f0, f1, std::true_type{});
        ring = ring + 1 == S::STAGES ? 0 : ring + 1;
        stage(st + 1, ring, f1, f0, std::true_type{});
        ring = ring + 1 == S::STAGES ? 0 : ring + 1;
    }
    for (; st < n_st; st += 2) {
        stage(st, ring, f0, f1, std::false_type{});
        ring = ring + 1 == S::STAGES ? 0 : ring + 1;
        if (st + 1 < n_st) stage(st + 1, ring, f1, f0, std::false_type{});
        ring = ring + 1 == S::STAGES ? 0 : ring + 1;
    }

    // Wait for the last products' results: the compiler does not count the
    // products' latency in inline assembly.  The epilogue takes the accumulators
    // from assembly behind this wait, a row block at a time, so that neither a
    // read nor a spill of one can come before it.
    asm volatile("s_nop 15\n\ts_nop 15" ::: "memory");

    // Epilogue: acc[i][j] holds C[m][n .. n+3] with m = m0 + TM/2 wm + 16 j +
    // l%16 and n = n0 + TN/2 wn + 16 i + 4 (l/16).
#pragma unroll
    for (int j = 0; j < S::MI; ++j) {
#pragma unroll
        for (int i = 0; i < S::NI; ++i) asm volatile("" : "+a"(acc[i][j]));
        const int64_t m = m0 + S::TM / 2 * wm + 16 * j + (lane & 15);
        if (m >= g.M) continue;
        f32x4 r[S::NI];
        if constexpr (OUT == kOutResid) {  // a row's residual values, their loads in flight together
#pragma unroll
            for (int i = 0; i < S::NI; ++i)
                r[i] = g.resid ? *reinterpret_cast<const f32x4*>(g.resid + m * g.N + n0 + S::TN / 2 * wn + 16 * i + 4 * (lane >> 4))
                               : f32x4{0.f, 0.f, 0.f, 0.f};
        }
        int64_t head_row = 0;
        if constexpr (OUT == kOutHeads) head_row = m / g.L * g.H * g.L + m % g.L;
#pragma unroll
        for (int i = 0; i < S::NI; ++i) {
            const int n = n0 + S::TN / 2 * wn + 16 * i + 4 * (lane >> 4);
            f32x4 c = acc[i][j];
            if (g.bias) c += *reinterpret_cast<const f32x4*>(g.bias + n);
            if constexpr (OUT == kOutResid) {
#pragma unroll
                for (int e = 0; e < 4; ++e) r[i][e] = fmaf(g.sign, c[e], r[i][e]);
                *reinterpret_cast<f32x4*>(g.out_f32 + m * g.N + n) = r[i];
            } else if constexpr (OUT == kOutReluBf16) {
                const uint2 p = make_uint2(pack_bf16x2(fmaxf(c[0], 0.f), fmaxf(c[1], 0.f)),
                                           pack_bf16x2(fmaxf(c[2], 0.f), fmaxf(c[3], 0.f)));
                *reinterpret_cast<uint2*>(g.out_bf16 + m * g.N + n) = p;
            } else {
                const int h = n >> 6, e = n & 63;
                const uint2 p = make_uint2(pack_bf16x2(c[0], c[1]), pack_bf16x2(c[2], c[3]));
                *reinterpret_cast<uint2*>(g.out_bf16 + (head_row + (int64_t)h * g.L) * 64 + e) = p;
            }
        }
    }
}

template <class S, int IN, int OUT>
hipError_t launch_shape(const GemmArgs& g, hipStream_t stream) {
    const int64_t tiles = (int64_t)(g.N / S::TN) * ((g.M + S::TM - 1) / S::TM);
    auto* k = &gemm_bf16_kernel<S, IN, OUT>;
    (void)hipFuncSetAttribute(reinterpret_cast<const void*>(k), hipFuncAttributeMaxDynamicSharedMemorySize, (int)S::kLds);
    k<<<(unsigned)tiles, 256, S::kLds, stream>>>(g);
    return hipGetLastError();
}

template <int IN, int OUT>
hipError_t launch_gemm(const GemmArgs& g, hipStream_t stream) {
    if (g.M == 0) return hipSuccess;
    // Tiles of 256 x 256, one workgroup a CU, where they fill whole waves of the
    // chip's 256 CUs well enough.  Nothing overlaps a workgroup's first copies and
    // its epilogue, which weigh more the fewer stages there are, so the fill that
    // it takes falls with K.  us with tiles of 256 / 128 (share of the waves filled):
    //   K >= 1536: 3/4.  16384 x 1024 x 4096 119 / 132 (1), 12,100 x 1024 x 2048
    //   59 / 65 (0.75), 8192 x 1536 x 1536 53 / 56 (0.75); 9000 x 1024 x 1024
    //   42 / 41 (0.56).
    //   512 < K < 1536: 0.85.  16384 x 4096 x 1024 146 / 157 (1), 14,000 x 1024 x
    //   1024 45.1 / 45.4 (0.86); 20,000 x 2048 x 1024 104 / 94 (0.82), 26,000 x
    //   2048 x 1024 137 / 124 (0.80), 8192 x 3072 x 768 61 / 49 (0.75).
    //   K = 512: only full waves.  65,536 x 512 x 512 89 / 102 (1), but 33,000 x
    //   2048 x 512 124 / 102 (0.81), 57,000 x 1024 x 512 100 / 84 (0.87).
    //   K < 512: none.  65,536 x 256 x 256 36 / 31 (1), 65,536 x 1024 x 256 83 / 72.
    // Tiles of 128 from one per CU on: 15.3 us against 22.4 with 64 at 4095 x 2048
    // x 512 (512 tiles); below that the smaller tiles spread the work further: 17.1
    // against 28 at 4095 x 512 x 2048 (128 tiles), 41 against 46 at 3000 x 1024 x
    // 4096 (192).
    auto tiles = [&](int t) { return g.N % t ? 0 : (int64_t)(g.N / t) * ((g.M + t - 1) / t); };
    const int64_t t256 = tiles(256), waves = (t256 + 255) / 256;
    const int fill = g.K >= 1536 ? 192 : (g.K > 512 ? 218 : (g.K == 512 ? 252 : 257));  // tiles per wave
    if (t256 > 0 && t256 >= fill * waves) return launch_shape<GemmShape<256, 256, 64, 2>, IN, OUT>(g, stream);
    if (tiles(128) >= 256) return launch_shape<GemmShape<128, 128, 64, 2>, IN, OUT>(g, stream);
    return launch_shape<GemmShape<64, 64, 64, 4>, IN, OUT>(g, stream);
}

}  // namespace

hipError_t launch_layer_norm(const float* x, const float* g, const float* b, uint16_t* out, int64_t rows, int D,
                             float eps, hipStream_t stream) {
    if (rows == 0) return hipSuccess;
    auto go = [&](auto pairs) {
        layer_norm_kernel<decltype(pairs)::value><<<(unsigned)((rows + 3) / 4), 256, 0, stream>>>(
            x, g, b, reinterpret_cast<uint32_t*>(out), rows, D, eps);
    };
    const int P = D / 128;
    if (P <= 4) go(std::integral_constant<int, 4>{});
    else if (P <= 8) go(std::integral_constant<int, 8>{});
    else if (P <= 16) go(std::integral_constant<int, 16>{});
    else go(std::integral_constant<int, kLnMaxPairs>{});
    return hipGetLastError();
}

hipError_t launch_linear(const uint16_t* a, bool a_heads, int L, int H, const uint16_t* w, int64_t M, int N, int K,
                         const float* bias, int out_kind, const float* resid, float sign, float* out_f32,
                         uint16_t* out_bf16, hipStream_t stream) {
    GemmArgs g{a, w, M, N, K, L, H, bias, resid, sign, out_f32, out_bf16};
    if (a_heads) {
        if (out_kind != kLinearResid) return hipErrorInvalidValue;
        return launch_gemm<kInHeads, kOutResid>(g, stream);
    }
    switch (out_kind) {
        case kLinearResid: return launch_gemm<kInRows, kOutResid>(g, stream);
        case kLinearReluBf16: return launch_gemm<kInRows, kOutReluBf16>(g, stream);
        case kLinearHeads: return launch_gemm<kInRows, kOutHeads>(g, stream);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace lsh
