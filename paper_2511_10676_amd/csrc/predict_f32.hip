// Predictor for fp32 storage, any shape: both linear layers (paper section 4.3,
// eq. 3) on the fp32 matrix instruction v_mfma_f32_32x32x2_f32, whose products
// and sums are fp32 like the vector unit's fma.
//
// What bounds it: that instruction, 256 flops per clock and CU (157 TFLOP/s on
// the chip).  It is 16 times slower than the bf16 one while the operands are
// only twice as wide, so small tiles are enough to keep it fed -- a 64 x 64
// tile asks LDS for 16 bytes per clock of the 128 it can deliver -- and the
// tiles are kept small so that a few hundred tokens of one layer already
// spread over every CU.  Vector instructions do not run beside it: a stage of 1024 clocks of products
// took 1030 with nothing else in the loop, 1190 with the LDS reads and their addresses, 1370 with the
// copies, 1500 with the sums in double.  So the loop goes through the ring's stages unrolled (no address
// arithmetic), a chain starts from a zero operand instead of cleared registers and only the last stage's
// copies look for the end of d: 33 tokens of 2048 x 2048, whole call, 53.3 -> 48.9 us, 512 tokens of d = 4096 95.4 -> 85.9.
//
// A workgroup owns BM tokens of one layer and a range of chunks of BN
// hidden units.  Per chunk it forms h^T[BN, BM] = W1[chunk, :] . x^T over stages of
// 32 columns, which travel global -> LDS by direct copies through a ring of NS
// stages (row of 128 bytes = 8 chunks of 16 bytes, chunk c in slot c ^ (row / 2 % 8),
// chosen on the global side; rows past T, r and columns past d lie outside the
// buffer resource and arrive as zeros).  A lane takes its fragment as one
// ds_read_b128, four k-steps of the instruction: the order in which k is walked is
// free as long as both operands agree.  Then h gets bias and activation, goes to
// LDS as [token][unit], and is multiplied by the chunk's columns of W2 into scores that stay
// in accumulators over the chunks.
//   BM = BN = 64   eight waves, two to each 32 x 32 block of h
//   BM = BN = 32   (T <= 32) four waves, all on one block: four times as many workgroups to stream the weights
// Waves that share a block split the columns of each stage and their sums meet in LDS in
// wave order: a second wave on every SIMD covers the other's barriers and LDS reads even where a
// CU has one workgroup (512 tokens of one 2048-wide layer: 48 us with one wave to a block, 46 with two).
// Rounding: the instruction rounds after every product, so a chain of n additions errs like
// sqrt(n / 2) roundings.  Sums over d are therefore chains of 8 to 32 columns (by d, below) that are
// added up in double, sums over r chains of 8 units added up per chunk; with that the scores are no further from
// float64 than those of a lane-split dot product with a butterfly (relative error of the scores, that / chains of 128
// and 64 / here: 512 tokens 2048 x 2048 1.76e-7 / 2.85e-7 / 1.72e-7, 4 x 8192 tokens 1.77e-7 / 8.4e-7 / 1.72e-7, 256 x 64
// 1.06e-7 / 2.9e-7 / 1.05e-7).
// Few token tiles: r is cut over several workgroups per tile, their scores meet in the
// workspace and finalize_kernel adds them; otherwise softmax and top-k follow here, 8 or 16 lanes to a row (a wave
// per row, one after the other: 4 x 1024 tokens of 256 x 64, 16 experts 36.7 us, 22.1 here).  That part costs the 64 x 64 tiles
// registers, also where r is cut: 5 vector registers spilled up to 128 experts at d >= 2048, outside the loop.
// 64 x 64 tiles run two workgroups to a CU up to 256 experts although 129 and more spill 63 to 88 registers (250 bytes a lane),
// and one from 257 on (16 spilled, from 513 on 200).  Two / one, us: 4 x 1024 tokens of 2048 x 2048, 256 experts 401 / 372, 200
// experts 571 / 589; 2 x 1024 of 1024 x 1024, 200 experts 120 / 100, of 512 x 1024, 160 experts 71 / 77; 3 x 1024 of 4096 x 1024, 130
// experts 328 / 331.
// Measured, 512 tokens x (2048 x 2048, 64 experts), whole call: 5200 us for a kernel of vector
// instructions (a wave per hidden unit), 50 us here.
#include <type_traits>

#include "paep_device.h"
#include "paep_internal.h"

namespace paep {

static constexpr int F32_BK = 32;                          // columns of d per stage
static constexpr size_t F32_WORKSPACE_MAX = 16u << 20;     // what predict_static can offer

typedef void __attribute__((address_space(3)))* f32_lds_ptr_t;
typedef __attribute__((ext_vector_type(4))) double f64x4;
__device__ __forceinline__ f32x16 zero16()
{
    f32x16 v;
#pragma unroll
    for (int i = 0; i < 16; ++i) v[i] = 0.0f;
    return v;
}
#define PAEP_F32_VMCNT(n) ((((n) & 0xF) | (((n) >> 4) << 14)) | 0x0F70)
template <int V> using F32IC = std::integral_constant<int, V>;
template <int N, class F> __device__ __forceinline__ void f32_static_for(F&& f)
{
    if constexpr (N > 0) {
        f32_static_for<N - 1>(f);
        f(F32IC<N - 1>{});
    }
}
static constexpr int PAEP_F32_LGKM0 = 0xC07F;              // lgkmcnt(0) and nothing else

// EBW: 32 x 32 score blocks per wave.  CHAIN: columns of d summed in fp32 before the sum is added up in double.
template <int B_, int NS, int EBW, int CHAIN>
__global__ __launch_bounds__(B_ == 64 ? 512 : 256, B_ == 32 || EBW >= 4 ? 2 : 4) void predict_f32_kernel(
    int T, int d, int r, int E, int k, int act, int tiles_per_layer, int groups, int nchunks,
    long long xs, long long w1s, long long w2s, const float* __restrict__ x, const float* __restrict__ W1,
    const float* __restrict__ W2, const float* __restrict__ b1, const float* __restrict__ b2,
    int32_t* __restrict__ idx, float* __restrict__ probs, float* __restrict__ logits, int32_t* __restrict__ counts,
    int prob_mode, float* __restrict__ margin, float* __restrict__ partial)
{
    constexpr int BM = B_, BN = B_;
    constexpr int WAVES = B_ == 64 ? 8 : 4, THREADS = 64 * WAVES;
    constexpr int TBN = BM / 32, NBLK = TBN * TBN;         // 32-token blocks, blocks of h
    constexpr int KPARTS = WAVES / NBLK;                   // waves that share a block
    constexpr int NP = (BM + BN) / 8 / WAVES;              // copy instructions per wave and stage, 8 rows each
    constexpr int STAGE = (BM + BN) * F32_BK * 4;          // bytes
    constexpr int HP = BN + 4;                             // pitch of h: 16 lanes of a fragment read hit all 64 banks
    extern __shared__ __attribute__((aligned(16))) unsigned char fsmem[];
    constexpr int QPW = 4 / KPARTS;                        // quarters of a block that a wave finishes (of a stage: that it multiplies)
    constexpr int RED = (KPARTS - 1) * NBLK * 1024 * 8;    // bytes
    double* red = (double*)fsmem;                          // the waves' sums for one another; reuses the ring
    float* ht = (float*)(fsmem + RED);                     // h of the chunk; reuses the ring
    static_assert(RED + BM * HP * 4 <= NS * STAGE, "sums and h fit in the ring");
    float* zs = (float*)fsmem;                             // 32 rows of scores; reuses everything

    const int grp = blockIdx.x % groups, tile_id = blockIdx.x / groups;
    const int layer = tile_id / tiles_per_layer, t0 = (tile_id - layer * tiles_per_layer) * BM;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l32 = lane & 31, g = lane >> 5;
    const float* xl = x + layer * xs + (long long)t0 * d;
    const float* W1l = W1 + layer * w1s;
    const float* W2l = W2 + layer * w2s;

    // copies: instruction wave * NP + j moves rows 8 * that .. + 7 of the stage; the first half of the waves moves
    // rows of W1, the second half token rows
    const bool moves_w = wave < WAVES / 2;
    const int xrows = T - t0 < BM ? T - t0 : BM;
    uint32_t src_off[NP];
    int lcol[NP];
#pragma unroll
    for (int j = 0; j < NP; ++j) {
        const int row = ((wave % (WAVES / 2)) * NP + j) * 8 + (lane >> 3);
        const int c = (lane & 7) ^ ((row >> 1) & 7);
        src_off[j] = (uint32_t)(row * d + c * 4) * 4u;
        lcol[j] = c * 4;
    }
    const int NKT = (d + F32_BK - 1) / F32_BK;

    f32x16 zacc[EBW];
#pragma unroll
    for (int j = 0; j < EBW; ++j)
#pragma unroll
        for (int i = 0; i < 16; ++i) zacc[j][i] = 0.0f;

    const int n_begin = (int)((long long)grp * nchunks / groups), n_end = (int)((long long)(grp + 1) * nchunks / groups);
#pragma unroll 1
    for (int n = n_begin; n < n_end; ++n) {
        const int u0 = n * BN;
        const int wrows = r - u0 < BN ? r - u0 : BN;
        const __amdgpu_buffer_rsrc_t rsrc = __builtin_amdgcn_make_buffer_rsrc(
            (void*)(moves_w ? W1l + (long long)u0 * d : xl), 0, (moves_w ? wrows : xrows) * d * 4, 0x00020000);
        auto issue_piece = [&](int kt, int slot, int j) {
            if (kt >= NKT) kt = NKT - 1;                   // past the end: the last stage again, into a slot nobody reads
            const int left = d - kt * F32_BK;
            const f32_lds_ptr_t to = (f32_lds_ptr_t)(fsmem + slot * STAGE + (wave * NP + j) * 1024);
            if (left >= F32_BK)
                __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrc, to, 16, (int)src_off[j], kt * (F32_BK * 4), 0, 0);
            else                                           // columns past d: an offset outside the resource
                __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrc, to, 16, (int)(lcol[j] < left ? src_off[j] : 0x70000000u),
                                                         kt * (F32_BK * 4), 0, 0);
        };
        const int blk = wave % NBLK, kpart = wave / NBLK;  // block of h: units (blk / TBN) * 32.., tokens (blk % TBN) * 32..
        f32x16 acc = zero16();
        double tot[16];
#pragma unroll
        for (int i = 0; i < 16; ++i) tot[i] = 0.0;             // 29 more bits: the order of these sums no longer matters
        auto fold = [&]() {
#pragma unroll
            for (int i = 0; i < 16; ++i) tot[i] += (double)acc[i];
        };
        const int arow = (blk / TBN) * 32 + l32;
        const int brow = BN + (blk % TBN) * 32 + l32;
        for (int s = 0; s < NS; ++s)
#pragma unroll
            for (int j = 0; j < NP; ++j) issue_piece(s, s, j);
        // Fragments of the stage being multiplied, replaced one by one by the next stage's (QPW = 1: two, in turn).
        constexpr int NF = 2;
        static_assert(QPW <= NF && NP == 2, "fragments, copies");
        f32x4 fa[NF], fb[NF];
        auto read = [&](auto slot_c, auto q_c, auto buf_c) {
            constexpr int q = decltype(q_c)::value, buf = decltype(buf_c)::value;
            const float* st = (const float*)(fsmem + decltype(slot_c)::value * STAGE);
            const int c = ((2 * (kpart * QPW + q) + g) ^ ((l32 >> 1) & 7)) * 4;
            fa[buf] = *(const f32x4*)(st + arow * F32_BK + c);
            fb[buf] = *(const f32x4*)(st + brow * F32_BK + c);
            __builtin_amdgcn_sched_barrier(0);
        };
        // Step s (8 columns) of the unrolled loop; a chain's first product takes no earlier sum.  COPY: stage kt's copies,
        // into `slot`, between the products.
        auto multiply = [&](auto s_c, auto buf_c, auto copy_c, int kt, int slot) {
            constexpr int buf = decltype(buf_c)::value;
            constexpr bool FIRST = decltype(s_c)::value % (CHAIN / 8) == 0, COPY = decltype(copy_c)::value;
            if constexpr (FIRST) fold();
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                acc = __builtin_amdgcn_mfma_f32_32x32x2f32(fa[buf][i], fb[buf][i], FIRST && i == 0 ? zero16() : acc, 0, 0, 0);
                __builtin_amdgcn_sched_barrier(0);
                if constexpr (COPY)
                    if (i % 2 == 0) issue_piece(kt, slot, i / 2);
                __builtin_amdgcn_sched_barrier(0);
            }
        };
        // from here on the next stage is read and this one's place is copied into: this wave's part of the one has landed,
        // its fragments of the other are in registers; everyone's
        auto hand_over = [&]() {
            __builtin_amdgcn_s_waitcnt(PAEP_F32_VMCNT(NP * (NS - 2)) & PAEP_F32_LGKM0);
            asm volatile("" ::: "memory");
            __builtin_amdgcn_s_barrier();
            asm volatile("" ::: "memory");
        };
        __builtin_amdgcn_s_waitcnt(PAEP_F32_VMCNT(NP * (NS - 1)));
        asm volatile("" ::: "memory");
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
        read(F32IC<0>{}, F32IC<0>{}, F32IC<0>{});
        if constexpr (QPW == 2) read(F32IC<0>{}, F32IC<1>{}, F32IC<1>{});
        static_assert(NS % 2 == 0 && NS * QPW % (CHAIN / 8) == 0, "a chain ends with the unrolled loop");
#pragma unroll 1
        for (int k0 = 0; k0 < NKT; k0 += NS)
            f32_static_for<NS>([&](auto u_c) {
                constexpr int u = decltype(u_c)::value;
                constexpr F32IC<(u + 1) % NS> next{};
                const int kt = k0 + u;
                if (kt < NKT) {
                    if constexpr (QPW == 1) {
                        hand_over();
                        read(next, F32IC<0>{}, F32IC<(u + 1) % 2>{});
                        multiply(F32IC<u>{}, F32IC<u % 2>{}, std::true_type{}, kt + NS, u);
                    } else {
                        multiply(F32IC<2 * u>{}, F32IC<0>{}, std::false_type{}, 0, 0);
                        hand_over();
                        read(next, F32IC<0>{}, F32IC<0>{});
                        multiply(F32IC<2 * u + 1>{}, F32IC<1>{}, std::true_type{}, kt + NS, u);
                        read(next, F32IC<1>{}, F32IC<1>{});
                    }
                }
            });
        fold();
        __builtin_amdgcn_s_waitcnt(PAEP_F32_VMCNT(0));     // no copy may land in the ring once it holds h
        __syncthreads();

        // tot[4q + i] = this wave's part of h[unit (blk / TBN) * 32 + 8q + 4g + i][token (blk % TBN) * 32 + l32]: the waves
        // of a block finish QPW of the four q each, with the others' parts from LDS
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int owner = q / QPW, part = kpart < owner ? kpart : kpart - 1;
            if (kpart != owner)
                *(f64x4*)(red + (((part * NBLK + blk) * 4 + q) * 64 + lane) * 4) = f64x4{tot[4 * q], tot[4 * q + 1], tot[4 * q + 2], tot[4 * q + 3]};
        }
        __syncthreads();
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            if (kpart == q / QPW) {
                f64x4 v = f64x4{tot[4 * q], tot[4 * q + 1], tot[4 * q + 2], tot[4 * q + 3]};
#pragma unroll
                for (int p = 0; p < KPARTS - 1; ++p) v += *(const f64x4*)(red + (((p * NBLK + blk) * 4 + q) * 64 + lane) * 4);
                const int unit = (blk / TBN) * 32 + 8 * q + 4 * g, tok = (blk % TBN) * 32 + l32;
                f32x4 hv;
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    if (b1 && u0 + unit + i < r) v[i] += (double)b1[(long long)layer * r + u0 + unit + i];
                    hv[i] = u0 + unit + i < r ? apply_act((float)v[i], act) : 0.0f;   // rows past r: 0 x infinity in a token is no 0
                }
                *(f32x4*)(ht + tok * HP + unit) = hv;
            }
        }
        __syncthreads();
        // z^T[E, tokens] += W2[:, chunk] . h^T; score block b = wave + WAVES * j is expert block b / TBN, token block b % TBN
#pragma unroll
        for (int j = 0; j < EBW; ++j) {
            const int b = wave + WAVES * j;
            const int e = (b / TBN) * 32 + l32, tok = (b % TBN) * 32 + l32;
            if ((b / TBN) * 32 < E) {                      // wave-uniform
                f32x4 w[BN / 8];
#pragma unroll
                for (int q = 0; q < BN / 8; ++q) {
                    w[q] = f32x4{0.f, 0.f, 0.f, 0.f};
                    if (e < E && u0 + 8 * q < r) w[q] = *(const f32x4*)(W2l + (long long)e * r + u0 + 8 * q + 4 * g);
                }
                f32x16 zc = zero16();
#pragma unroll
                for (int q = 0; q < BN / 8; ++q) {
                    const f32x4 h = *(const f32x4*)(ht + tok * HP + 8 * q + 4 * g);
                    f32x16 zq = zero16();
#pragma unroll
                    for (int i = 0; i < 4; ++i) zq = __builtin_amdgcn_mfma_f32_32x32x2f32(w[q][i], h[i], zq, 0, 0, 0);
                    zc += zq;
                }
                zacc[j] += zc;
            }
            __builtin_amdgcn_sched_barrier(0);             // one block's fetches at a time in registers
        }
        __syncthreads();                                   // h has been read; the ring may be filled again
    }

    // zacc[j][4q + i] = score of expert (b / TBN) * 32 + 8q + 4g + i, token (b % TBN) * 32 + l32
    if (groups > 1) {
#pragma unroll
        for (int j = 0; j < EBW; ++j) {
            const int b = wave + WAVES * j;
            const int t = t0 + (b % TBN) * 32 + l32;
            if (t < T) {
                float* dst = partial + (((long long)layer * groups + grp) * T + t) * E;
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const int e = (b / TBN) * 32 + 8 * q + 4 * g;
                    if (e + 3 < E) {
                        *(f32x4*)(dst + e) = f32x4{zacc[j][4 * q], zacc[j][4 * q + 1], zacc[j][4 * q + 2], zacc[j][4 * q + 3]};
                    } else {
#pragma unroll
                        for (int i = 0; i < 4; ++i)
                            if (e + i < E) dst[e + i] = zacc[j][4 * q + i];
                    }
                }
            }
        }
        return;
    }
    const int ZP = E + 1;
#pragma unroll 1
    for (int tb = 0; tb < TBN; ++tb) {
#pragma unroll
        for (int j = 0; j < EBW; ++j) {
            const int b = wave + WAVES * j;
            if (b % TBN == tb)
#pragma unroll
                for (int i = 0; i < 16; ++i) {
                    const int e = (b / TBN) * 32 + 8 * (i >> 2) + 4 * g + (i & 3);
                    if (e < E) zs[l32 * ZP + e] = zacc[j][i] + (b2 ? b2[(long long)layer * E + e] : 0.0f);
                }
        }
        __syncthreads();
        if (logits)
            for (int i = tid; i < 32 * E; i += THREADS) {
                const int rr = i / E, e = i - rr * E;
                if (t0 + tb * 32 + rr < T) logits[((long long)layer * T + t0 + tb * 32 + rr) * E + e] = zs[rr * ZP + e];
            }
        if (k + (margin && k < E ? 1 : 0) <= 16) {             // G lanes per row, all rows at once
            constexpr int G = THREADS / 32;
            const int rr = tid / G, t = t0 + tb * 32 + rr;
            if (t < T) {
                const long long row = (long long)layer * T + t;
                const float* zrow = zs + rr * ZP;
                const EpilogueOut eo{prob_mode, margin ? margin + row : nullptr,
                                     counts ? counts + (long long)layer * E : nullptr};
                row_softmax_topk_upto16<G, true, Sums::Fine>([&](int e) { return zrow[e]; }, E, k, tid % G, idx + row * k, probs + row * k, eo);
            }
        } else {
            for (int rr = wave; rr < 32; rr += WAVES) {        // longer lists: one wave per row
                const int t = t0 + tb * 32 + rr;
                if (t < T) {
                    constexpr int NV = EBW * WAVES / TBN / 2;  // experts per lane
                    const long long row = (long long)layer * T + t;
                    float z[NV];
#pragma unroll
                    for (int v = 0; v < NV; ++v) {
                        const int e = lane + 64 * v;
                        z[v] = e < E ? zs[rr * ZP + e] : 0.0f;
                    }
                    const EpilogueOut eo{prob_mode, margin ? margin + row : nullptr,
                                         counts ? counts + (long long)layer * E : nullptr};
                    wave_softmax_topk<NV>(z, E, k, lane, idx + row * k, probs + row * k, eo);
                }
            }
        }
        __syncthreads();
    }
}

// tokens (and hidden units) per tile: the small tile while it holds all tokens of a layer
static int f32_tile(const PredictArgs& a) { return a.T <= 32 ? 32 : 64; }

// Workgroups per token tile: up to two per CU (512 in all), which keep the matrix pipe fed between one's chunks;
// more would only add score tiles to add up.
static int f32_groups(const PredictArgs& a)
{
    const int B = f32_tile(a), nchunks = (a.r + B - 1) / B;
    const long long tiles = (long long)((a.T + B - 1) / B) * a.L;
    long long g = (512 + tiles - 1) / tiles;
    if (g > nchunks) g = nchunks;
    const long long per_group = (long long)a.L * a.T * a.E * 4;
    if (g * per_group > (long long)F32_WORKSPACE_MAX) g = (long long)F32_WORKSPACE_MAX / per_group;
    return g < 1 ? 1 : (int)g;
}

// The sizes that fp32 storage has always taken (four rows of tokens, hidden units and scores in 160 KB); byte offsets
// inside a tile's rows stay far below 32 bits.
bool f32_supported(const PredictArgs& a)
{
    return a.dtype == 0 && (long long)a.d + a.r + a.E <= 160 * 1024 / 16;
}

size_t f32_workspace_bytes(const PredictArgs& a)
{
    if (a.T == 0) return 0;
    const int g = f32_groups(a);
    return g == 1 ? 0 : sizeof(float) * (size_t)g * (size_t)a.L * (size_t)a.T * (size_t)a.E;
}

hipError_t launch_predict_f32(const PredictArgs& a)
{
    if (a.T == 0) return hipSuccess;
    const int B = f32_tile(a), tiles = (a.T + B - 1) / B, nchunks = (a.r + B - 1) / B,
              groups = a.workspace && a.workspace_bytes >= f32_workspace_bytes(a) ? f32_groups(a) : 1;
    const size_t epilogue = groups == 1 ? sizeof(float) * 32 * (size_t)(a.E + 1) : 0;
    const int eblocks = (a.E + 31) / 32, waves = B == 64 ? 8 : 4,
              ebw = (eblocks * (B / 32) + waves - 1) / waves;
    hipError_t err;
#define PAEP_LAUNCH_F32_C(BV, NSV, EBV, CV)                                                                        \
    do {                                                                                                           \
        const size_t ring = (size_t)NSV * 2 * BV * F32_BK * 4, lds = ring > epilogue ? ring : epilogue;            \
        auto kern = predict_f32_kernel<BV, NSV, EBV, CV>;                                                            \
        static LdsLimit limit;                                                                                     \
        err = ensure_lds_limit(limit, (const void*)kern, lds);                                                     \
        if (err != hipSuccess) return err;                                                                         \
        hipLaunchKernelGGL(kern, dim3(tiles * a.L * groups), dim3(64 * waves), lds, a.stream, a.T, a.d, a.r, a.E, \
                           a.k, a.act, tiles, groups, nchunks, a.x_stride, a.w1_stride, a.w2_stride,               \
                           (const float*)a.x, (const float*)a.W1, (const float*)a.W2, (const float*)a.b1,          \
                           (const float*)a.b2, a.idx, a.probs, a.logits, a.counts, a.prob_mode, a.margin,          \
                           (float*)a.workspace);                                                                   \
    } while (0)
    // columns in a chain: fewer where d leaves fewer roundings to hide among
#define PAEP_LAUNCH_F32(BV, NSV, EBV)                                                                              \
    do {                                                                                                           \
        if (a.d < 768)       PAEP_LAUNCH_F32_C(BV, NSV, EBV, 8);                                                   \
        else if (a.d < 2048) PAEP_LAUNCH_F32_C(BV, NSV, EBV, 16);                                                  \
        else                 PAEP_LAUNCH_F32_C(BV, NSV, EBV, 32);                                                  \
    } while (0)
    // score blocks per wave the kernel is compiled for
    if (B == 64) {
        if (ebw <= 1)      PAEP_LAUNCH_F32(64, 4, 1);
        else if (ebw <= 2) PAEP_LAUNCH_F32(64, 4, 2);
        else if (ebw <= 4) PAEP_LAUNCH_F32(64, 4, 4);
        else               PAEP_LAUNCH_F32(64, 4, 8);
    } else {
        if (ebw <= 1)      PAEP_LAUNCH_F32(32, 8, 1);
        else if (ebw <= 2) PAEP_LAUNCH_F32(32, 8, 2);
        else               PAEP_LAUNCH_F32(32, 8, 8);
    }
#undef PAEP_LAUNCH_F32
#undef PAEP_LAUNCH_F32_C
    err = hipGetLastError();
    if (err != hipSuccess || groups == 1) return err;
    return launch_finalize(a, (const float*)a.workspace, groups, a.L, a.T, 0, 1);
}

}  // namespace paep
