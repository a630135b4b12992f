// Decode-shaped predictor (T <= 64 tokens per layer), bf16 storage.
//
// At a handful of tokens the predictor is a weight-streaming problem: every
// byte of W1 (r x d) and W2 (E x r) is needed once and the arithmetic per byte
// is tiny, so the kernels are organised around reading the weights from HBM
// exactly once, coalesced, with many loads in flight and nothing in the way.
// One predictor belongs to one layer (paper section 4.2) and a layer is only
// ~8 MB, so all layers of a call are spread over one grid.
//
// Kernel 1 (partial): the inner width r is cut into slices; workgroup (slice,
// layer) owns W1[slice rows, :] and W2[:, slice], forms h^T[slice, T] with
// v_mfma_f32_16x16x32_bf16, rounds it to bf16 (bias and activation applied)
// and multiplies it by the W2 column slice with the same instruction; that is
// the slice's contribution to the scores and goes to the workspace as fp32
// partial[layer][slice][t][e].  Two forms:
//   rows   (r a multiple of 128) slices of 128 hidden units, eight waves that
//          split the ROWS: a wave streams its 16 rows over the whole of d into
//          registers and all waves take the tokens from LDS, where the
//          workgroup puts them once (decode_rows_kernel below).
//   d-split  slices of 64 hidden units, four waves that split d into quarters,
//          weights and tokens both straight into registers, the four partial
//          sums added in LDS wave after wave (decode_partial_kernel).
//   thin   (one layer or a few) slices of 16 or 32 hidden units, eight waves that split d, so that the slices of
//          a single layer already occupy half the chip (decode_thin_kernel).
// In all of them a lane reads 16 contiguous bytes of one row, four neighbouring lanes
// 64 contiguous bytes, and a lane permutation puts the fragment into the
// A-operand layout.
//
// Kernel 2 (finalize.hip): one wave per token adds the slices in ascending order
// and runs softmax and top-k.
#include <type_traits>

#include "paep_device.h"
#include "paep_internal.h"

namespace paep {

static constexpr int DEC_THREADS = 256;
static constexpr int RS = 64;            // hidden units per workgroup
static constexpr int RB = RS / 16;       // 16-row blocks per workgroup
static constexpr int HPAD = 8;

template <int V> using IC = std::integral_constant<int, V>;
template <int N, class F> __device__ __forceinline__ void static_for(F&& f)
{
    if constexpr (N > 0) {
        static_for<N - 1>(f);
        f(IC<N - 1>{});
    }
}

// TB: 16-token blocks (T <= 16 * TB); U: k-steps per load batch; NBUF: load
// batches in the register ring (NBUF - 1 are in flight while one is multiplied).
template <int TB, int U, int NBUF>
__global__ __launch_bounds__(DEC_THREADS) void decode_partial_kernel(
    int T, int d, int r, int E, int act, int S, int total_wgs, long long xs_, long long w1s, long long w2s,
    const uint16_t* __restrict__ x, const uint16_t* __restrict__ W1, const uint16_t* __restrict__ W2,
    const uint16_t* __restrict__ b1, float* __restrict__ partial)
{
    constexpr int TP = 16 * TB;
    __shared__ __attribute__((aligned(16))) float hsum[RB * TB * 64 * 4];          // partial h, summed wave after wave
    __shared__ __attribute__((aligned(16))) uint16_t ht[TP * (RS + HPAD)];        // h as bf16, [token][unit]

    // Work item = (layer, slice), slice fastest.  Workgroups are dealt round-robin
    // to the 8 XCDs; remap so that each XCD walks a contiguous range of items: the
    // workgroups an XCD runs at the same time are then neighbouring slices of one
    // layer and find that layer's tokens in the XCD's L2, and a layer's tokens are
    // fetched from memory by one or two XCDs instead of all eight.
    int item = blockIdx.x;
    {
        const int per = total_wgs / 8, rem = total_wgs % 8;
        const int xcd = item % 8, slot = item / 8;
        item = xcd * per + (xcd < rem ? xcd : rem) + slot;
    }
    const int layer = item / S, slice = item - layer * S;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int m = lane & 15, kg = lane >> 4;
    const uint16_t* xl = x + (long long)layer * xs_;
    const uint16_t* W1l = W1 + (long long)layer * w1s;
    const uint16_t* W2l = W2 + (long long)layer * w2s;

    // this wave's quarter of d
    const int kq = d / 4, k0 = wave * kq;
    const int nsteps = kq / 32;                               // MFMA k-steps per wave
    // Which 16 bytes a lane fetches of a 16-row x 64-byte fragment.  The matrix instruction wants lane
    // (m, kg) to hold row m, bytes 16*kg..; fetched that way, neighbouring lanes touch different rows and
    // every lane is a separate 16-byte access to the vector cache.  So lane l fetches row l/4, bytes
    // 16*(l%4).. instead -- four neighbouring lanes form one 64-byte access -- and the fragment is put
    // into the instruction's layout afterwards by a fixed lane permutation (lane (m, kg) takes from lane
    // 4*m + kg; ds_bpermute moves registers between lanes without touching LDS memory).  Measured on
    // the 26 x (2048 x 2048) bank: -6% time at 1 token, -14% at 64.
    const int lrow = lane >> 2, lchunk = lane & 3;
    const int perm_src = (4 * m + kg) * 4;                   // byte address for ds_bpermute
    const uint16_t* arow = W1l + (long long)(slice * RS + lrow) * d + k0 + lchunk * 8;   // + rb*16*d + step*32
    const uint16_t* brow = xl + (long long)lrow * d + k0 + lchunk * 8;                  // + tb*16*d + step*32
    bool tok_ok[TB];
#pragma unroll
    for (int tb = 0; tb < TB; ++tb) tok_ok[tb] = (tb * 16 + lrow) < T;
    auto to_mfma_layout = [&](const u32x4& f) {
        return u32x4{(uint32_t)__builtin_amdgcn_ds_bpermute(perm_src, (int)f[0]),
                          (uint32_t)__builtin_amdgcn_ds_bpermute(perm_src, (int)f[1]),
                          (uint32_t)__builtin_amdgcn_ds_bpermute(perm_src, (int)f[2]),
                          (uint32_t)__builtin_amdgcn_ds_bpermute(perm_src, (int)f[3])};
    };

    // W2 fragments of this wave's first expert blocks, requested now and used at the very end
    constexpr int NPF = 2;
    const int EB = (E + 15) / 16;
    u32x4 w2pf[NPF][RS / 32];
#pragma unroll
    for (int j = 0; j < NPF; ++j) {
        const int e_row = (wave + 4 * j) * 16 + m;
#pragma unroll
        for (int s = 0; s < RS / 32; ++s) {
            w2pf[j][s] = u32x4{0u, 0u, 0u, 0u};
            if (e_row < E) w2pf[j][s] = *(const u32x4*)(W2l + (long long)e_row * r + slice * RS + s * 32 + kg * 8);
        }
    }

    f32x4 acc[RB][TB];
#pragma unroll
    for (int rb = 0; rb < RB; ++rb)
#pragma unroll
        for (int tb = 0; tb < TB; ++tb) acc[rb][tb] = f32x4{0.f, 0.f, 0.f, 0.f};

    u32x4 fa[NBUF][U][RB], fb[NBUF][U][TB];
    auto load_batch = [&](auto buf_c, int step0) {
        constexpr int buf = decltype(buf_c)::value;
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int off = (step0 + u) * 32;
            const bool live = step0 + u < nsteps;             // wave-uniform; steps past the end multiply zeros
#pragma unroll
            for (int rb = 0; rb < RB; ++rb) {
                fa[buf][u][rb] = u32x4{0u, 0u, 0u, 0u};
                if (live) fa[buf][u][rb] = *(const u32x4*)(arow + (long long)rb * 16 * d + off);
            }
#pragma unroll
            for (int tb = 0; tb < TB; ++tb) {
                fb[buf][u][tb] = u32x4{0u, 0u, 0u, 0u};
                if (live && tok_ok[tb]) fb[buf][u][tb] = *(const u32x4*)(brow + (long long)tb * 16 * d + off);
            }
        }
    };
    auto mma_batch = [&](auto buf_c) {
        constexpr int buf = decltype(buf_c)::value;
#pragma unroll
        for (int u = 0; u < U; ++u) {
            u32x4 pa[RB], pb[TB];
#pragma unroll
            for (int rb = 0; rb < RB; ++rb) pa[rb] = to_mfma_layout(fa[buf][u][rb]);
#pragma unroll
            for (int tb = 0; tb < TB; ++tb) pb[tb] = to_mfma_layout(fb[buf][u][tb]);
#pragma unroll
            for (int rb = 0; rb < RB; ++rb)
#pragma unroll
                for (int tb = 0; tb < TB; ++tb)
                    acc[rb][tb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
                        __builtin_bit_cast(bf16x8, pa[rb]), __builtin_bit_cast(bf16x8, pb[tb]),
                        acc[rb][tb], 0, 0, 0);
        }
    };

    // Ring of NBUF register batches: batch i + NBUF - 1 is requested, then batch i is multiplied,
    // so NBUF - 1 batches of loads are in flight behind the arithmetic.
    static_for<NBUF - 1>([&](auto b_c) { load_batch(b_c, decltype(b_c)::value * U); });
    for (int s0 = 0; s0 < nsteps; s0 += NBUF * U) {
        static_for<NBUF>([&](auto b_c) {
            constexpr int b = decltype(b_c)::value;
            load_batch(IC<(b + NBUF - 1) % NBUF>{}, s0 + (b + NBUF - 1) * U);
            if (s0 + b * U < nsteps) mma_batch(b_c);          // wave-uniform
        });
    }

    // acc[rb][tb][i] = partial h[token tb*16 + m][unit slice*RS + rb*16 + 4*kg + i] over this wave's quarter of d.
    // The four partial sums are added in LDS wave after wave (w0 + w1 + w2 + w3, a fixed order) in one buffer.
#pragma unroll 1
    for (int w = 0; w < 4; ++w) {
        if (wave == w) {
#pragma unroll
            for (int rb = 0; rb < RB; ++rb)
#pragma unroll
                for (int tb = 0; tb < TB; ++tb) {
                    f32x4* slot = (f32x4*)(&hsum[((rb * TB + tb) * 64 + lane) * 4]);
                    f32x4 v = acc[rb][tb];
                    if (w > 0) {
                        const f32x4 o = *slot;
#pragma unroll
                        for (int i = 0; i < 4; ++i) v[i] = o[i] + v[i];
                    }
                    *slot = v;
                }
        }
        __syncthreads();
    }
    for (int q = tid; q < RB * TB * 64; q += DEC_THREADS) {
        const int ln = q & 63, blk = q >> 6, tb = blk % TB, rb = blk / TB;
        const int unit = rb * 16 + 4 * (ln >> 4), tok = tb * 16 + (ln & 15);
        const f32x4 v = *(const f32x4*)(&hsum[q * 4]);
        float h[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            float t = v[i];
            if (b1) t += bf16_bits_to_f32(b1[(long long)layer * r + slice * RS + unit + i]);
            t = round_to_bf16(t);
            if (act != 0) t = round_to_bf16(apply_act_bf16(t, act));
            h[i] = t;
        }
        *(u32x2*)(ht + tok * (RS + HPAD) + unit) = u32x2{pack_bf16x2(h[0], h[1]), pack_bf16x2(h[2], h[3])};
    }
    __syncthreads();

    // scores of this slice: z^T[e, t] = W2[e, slice] . h^T[slice, t]
    auto score_block = [&](int eb, const u32x4 (&wfrag)[RS / 32]) {
#pragma unroll
        for (int tb = 0; tb < TB; ++tb) {
            f32x4 z = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int s = 0; s < RS / 32; ++s) {
                const u32x4 hv = *(const u32x4*)(ht + (tb * 16 + m) * (RS + HPAD) + s * 32 + kg * 8);
                z = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, wfrag[s]),
                                                            __builtin_bit_cast(bf16x8, hv), z, 0, 0, 0);
            }
            // z[i] = score contribution for token tb*16 + m, expert eb*16 + 4*kg + i
            const int t = tb * 16 + m;
            if (t < T) {
                float* dst = partial + (((long long)layer * S + slice) * T + t) * E + eb * 16 + 4 * kg;
                if (eb * 16 + 4 * kg + 3 < E) {
                    *(f32x4*)dst = z;
                } else {
#pragma unroll
                    for (int i = 0; i < 4; ++i)
                        if (eb * 16 + 4 * kg + i < E) dst[i] = z[i];
                }
            }
        }
    };
#pragma unroll
    for (int j = 0; j < NPF; ++j)
        if (wave + 4 * j < EB) score_block(wave + 4 * j, w2pf[j]);
    for (int eb = wave + 4 * NPF; eb < EB; eb += 4) {
        const int e_row = eb * 16 + m;
        u32x4 wfrag[RS / 32];
#pragma unroll
        for (int s = 0; s < RS / 32; ++s) {
            wfrag[s] = u32x4{0u, 0u, 0u, 0u};
            if (e_row < E) wfrag[s] = *(const u32x4*)(W2l + (long long)e_row * r + slice * RS + s * 32 + kg * 8);
        }
        score_block(eb, wfrag);
    }
}

// The row-split form.  What a CU's vector memory path can have in flight, not HBM, is what the d-split kernel
// waits for, and tokens take their share of it: every 64-row slice fetches all T tokens again (at 64 tokens
// as many bytes as the slice itself), and whether they come from L2 or from the CU's own cache makes no
// difference to the time (measured).  Here a workgroup takes 128 hidden units, so the tokens are fetched once
// per 128 rows, and the waves divide the rows instead of d: wave w owns rows 16w..16w+15 of the slice over
// the whole of d and streams them into registers; all eight waves take the tokens from LDS, where each stage
// of 128 columns is put once per workgroup by direct global -> LDS copies (a ring of two or three stages, one
// workgroup barrier per stage: with two workgroups on a CU one stage of requests ahead per wave already
// over-fills the memory pipeline and deeper rings measured 2-3 % slower; with one workgroup per CU two
// stages ahead are 5-9 % faster).  A wave's accumulators are the finished h of its rows: nothing to add up
// across waves.  Token row t of a stage is 256 bytes = 16 chunks of 16 bytes, chunk c in slot c ^ (t % 16)
// (chosen on the global side of the copy), so that the 16 lanes of a fragment read, which take the same
// chunk of 16 different tokens, fall into 16 different slots.  Measured on 26 layers of 2048 x 2048 against
// the d-split kernel: 53.8 -> 49.8 us at 1 token, 58.7 -> 51.2 at 16, 79.7 -> 57.6 at 64.
static constexpr int RW_WAVES = 8;
static constexpr int RW_RS = 16 * RW_WAVES;          // hidden units per workgroup
static constexpr int RW_KST = 128;                   // columns of d per stage

typedef void __attribute__((address_space(3)))* lds_ptr_t;
// s_waitcnt immediate that waits for vmcnt <= n and nothing else (gfx9 encoding)
#define PAEP_DEC_VMCNT(n) ((((n) & 0xF) | (((n) >> 4) << 14)) | 0x0F70)

// TB: 16-token blocks held in LDS, 2 (T <= 32) or 4; RW_NSTG: stages in the ring, 2 or 3
template <int TB, int RW_NSTG>
__global__ __launch_bounds__(RW_WAVES * 64, 4) void decode_rows_kernel(
    int T, int d, int r, int E, int act, int S, int total_wgs, long long xs_, long long w1s, long long w2s,
    const uint16_t* __restrict__ x, const uint16_t* __restrict__ W1, const uint16_t* __restrict__ W2,
    const uint16_t* __restrict__ b1, float* __restrict__ partial)
{
    constexpr int TP = 16 * TB;
    constexpr int STAGE_BYTES = TP * RW_KST * 2;
    constexpr int XJ = TP / 4 / RW_WAVES;            // copy instructions per wave and stage (4 token rows each)
    constexpr int KS = RW_KST / 32;                  // MFMA k-steps per stage
    static_assert(XJ * 4 * RW_WAVES == TP, "token rows divide among the waves");
    extern __shared__ __attribute__((aligned(16))) unsigned char dsmem[];   // the ring; h (bf16) afterwards
    uint16_t* ht = (uint16_t*)dsmem;                                       // [token][unit], TP x (RW_RS + HPAD)
    static_assert(TP * (RW_RS + HPAD) * 2 <= RW_NSTG * STAGE_BYTES, "h fits in the ring");

    int item = blockIdx.x;
    {
        const int per = total_wgs / 8, rem = total_wgs % 8;
        const int xcd = item % 8, slot = item / 8;
        item = xcd * per + (xcd < rem ? xcd : rem) + slot;
    }
    const int layer = item / S, slice = item - layer * S;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int m = lane & 15, kg = lane >> 4;
    const uint16_t* xl = x + (long long)layer * xs_;
    const uint16_t* W1l = W1 + (long long)layer * w1s;
    const uint16_t* W2l = W2 + (long long)layer * w2s;
    const int NST = d / RW_KST;

    // token copies: instruction q = wave * XJ + j moves token rows 4q..4q+3 of a stage; lane l supplies the
    // chunk that belongs in slot l % 16 of row 4q + l / 16.  Rows past T lie outside the resource: zeros.
    const __amdgpu_buffer_rsrc_t rsrc_x =
        __builtin_amdgcn_make_buffer_rsrc((void*)xl, 0, (int)((long long)T * d * 2), 0x00020000);
    uint32_t xlane[XJ];
#pragma unroll
    for (int j = 0; j < XJ; ++j) {
        const int t = (wave * XJ + j) * 4 + (lane >> 4);
        const int c = (lane & 15) ^ (t & 15);
        xlane[j] = (uint32_t)(t * d + c * 8) * 2u;
    }
    auto issue_x = [&](int stage, int slot) {
#pragma unroll
        for (int j = 0; j < XJ; ++j)
            __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrc_x, (lds_ptr_t)(dsmem + slot * STAGE_BYTES + (wave * XJ + j) * 1024),
                                                     16, (int)xlane[j], stage * RW_KST * 2, 0, 0);
    };
    // this wave's 16 rows of W1, fetched as in the kernel above (lane l: row l / 4, bytes 16 * (l % 4) of a
    // 64-byte k-step) and permuted into the A-operand layout
    const int lrow = lane >> 2, lchunk = lane & 3;
    const int perm_src = (4 * m + kg) * 4;
    // (buffer-addressed: base and bounds of the wave's 16 rows in scalar registers, a fixed 32-bit lane offset and
    // a scalar stage offset, so that no vector register is spent on addresses inside the loop)
    const __amdgpu_buffer_rsrc_t rsrc_w = __builtin_amdgcn_make_buffer_rsrc(
        (void*)(W1l + (long long)(slice * RW_RS + wave * 16) * d), 0, 16 * d * 2, 0x00020000);
    const int wlane = (lrow * d + lchunk * 8) * 2;
    auto to_mfma_layout = [&](const u32x4& f) {
        return u32x4{(uint32_t)__builtin_amdgcn_ds_bpermute(perm_src, (int)f[0]),
                     (uint32_t)__builtin_amdgcn_ds_bpermute(perm_src, (int)f[1]),
                     (uint32_t)__builtin_amdgcn_ds_bpermute(perm_src, (int)f[2]),
                     (uint32_t)__builtin_amdgcn_ds_bpermute(perm_src, (int)f[3])};
    };
    u32x4 fa[RW_NSTG][KS];
    auto load_w = [&](auto buf_c, int stage) {
        constexpr int buf = decltype(buf_c)::value;
#pragma unroll
        for (int ks = 0; ks < KS; ++ks)
            fa[buf][ks] = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(rsrc_w, wlane + ks * 64, stage * (RW_KST * 2), 0));
    };

    // W2 fragments of this wave's first expert block, requested now and used at the very end
    const int EB = (E + 15) / 16;
    u32x4 w2pf[RW_RS / 32];
    {
        const int e_row = wave * 16 + m;
#pragma unroll
        for (int s = 0; s < RW_RS / 32; ++s) {
            w2pf[s] = u32x4{0u, 0u, 0u, 0u};
            if (e_row < E) w2pf[s] = *(const u32x4*)(W2l + (long long)e_row * r + slice * RW_RS + s * 32 + kg * 8);
        }
    }

    f32x4 acc[TB];
#pragma unroll
    for (int tb = 0; tb < TB; ++tb) acc[tb] = f32x4{0.f, 0.f, 0.f, 0.f};

    // Stage s: its token copies and this wave's rows are requested RW_NSTG - 1 stages ahead, in that order, so
    // at the top of stage s only the requests of the RW_NSTG - 2 stages after it may still be in flight.  Past
    // the last stage the last one is requested again (into a slot nobody reads any more), which keeps that
    // count the same on every iteration.
    constexpr int WAIT_STAGE = PAEP_DEC_VMCNT((RW_NSTG - 2) * (XJ + KS));
    // Workgroups start at different columns and wrap around (the s-th stage a workgroup works on is columns
    // 128 * ((s + item) % NST) ..): all waves of the chip advance at about the same pace, and with a common
    // starting column the addresses in flight at any moment would differ only in bits 12 and up -- rows are a
    // power of two apart -- which lands them on a few memory channels for some placements of the weights
    // (measured: 58 us against 48 us for one of four identically shaped banks; the same 48 us for all four with
    // the rotation).  The order in which a workgroup adds up d is fixed by its position in the grid.
    const int rot = item % NST;
    auto column_stage = [&](int s) { return s + rot < NST ? s + rot : s + rot - NST; };
    static_for<RW_NSTG - 1>([&](auto b_c) {
        constexpr int b = decltype(b_c)::value;
        const int st = column_stage(b < NST ? b : NST - 1);
        issue_x(st, b);
        __builtin_amdgcn_sched_barrier(0);
        load_w(b_c, st);
        __builtin_amdgcn_sched_barrier(0);
    });
    for (int s0 = 0; s0 < NST; s0 += RW_NSTG) {
        static_for<RW_NSTG>([&](auto b_c) {
            constexpr int b = decltype(b_c)::value;
            const int s = s0 + b;
            if (s < NST) {                                        // uniform over the workgroup
                __builtin_amdgcn_s_waitcnt(WAIT_STAGE);           // this wave's part of stage s has landed
                asm volatile("" ::: "memory");
                __builtin_amdgcn_s_barrier();                     // everyone's has; and everyone is done with stage s - 1
                asm volatile("" ::: "memory");
                const int sn = column_stage(s + RW_NSTG - 1 < NST ? s + RW_NSTG - 1 : NST - 1);
                issue_x(sn, (b + RW_NSTG - 1) % RW_NSTG);
                __builtin_amdgcn_sched_barrier(0);
                load_w(IC<(b + RW_NSTG - 1) % RW_NSTG>{}, sn);
                __builtin_amdgcn_sched_barrier(0);
                const unsigned char* stage = dsmem + b * STAGE_BYTES;
#pragma unroll
                for (int ks = 0; ks < KS; ++ks) {
                    u32x4 pb[TB];
#pragma unroll
                    for (int tb = 0; tb < TB; ++tb)
                        pb[tb] = *(const u32x4*)(stage + (tb * 16 + m) * (RW_KST * 2) + (((ks * 4 + kg) ^ m) << 4));
                    const u32x4 pa = to_mfma_layout(fa[b][ks]);
#pragma unroll
                    for (int tb = 0; tb < TB; ++tb)
                        acc[tb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
                            __builtin_bit_cast(bf16x8, pa), __builtin_bit_cast(bf16x8, pb[tb]), acc[tb], 0, 0, 0);
                }
            }
        });
    }
    // acc[tb][i] = h[token tb*16 + m][unit slice*RW_RS + wave*16 + 4*kg + i].  The ring is handed over to h once
    // every copy still in flight has landed and every wave has read its last fragments.
    __builtin_amdgcn_s_waitcnt(PAEP_DEC_VMCNT(0));
    __syncthreads();
#pragma unroll
    for (int tb = 0; tb < TB; ++tb) {
        const int unit = wave * 16 + 4 * kg, tok = tb * 16 + m;
        float h[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            float t = acc[tb][i];
            if (b1) t += bf16_bits_to_f32(b1[(long long)layer * r + slice * RW_RS + unit + i]);
            t = round_to_bf16(t);
            if (act != 0) t = round_to_bf16(apply_act_bf16(t, act));
            h[i] = t;
        }
        *(u32x2*)(ht + tok * (RW_RS + HPAD) + unit) = u32x2{pack_bf16x2(h[0], h[1]), pack_bf16x2(h[2], h[3])};
    }
    __syncthreads();

    // scores of this slice: z^T[e, t] = W2[e, slice] . h^T[slice, t]; expert blocks dealt to the waves
    auto score_block = [&](int eb, const u32x4 (&wfrag)[RW_RS / 32]) {
#pragma unroll
        for (int tb = 0; tb < TB; ++tb) {
            f32x4 z = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int s = 0; s < RW_RS / 32; ++s) {
                const u32x4 hv = *(const u32x4*)(ht + (tb * 16 + m) * (RW_RS + HPAD) + s * 32 + kg * 8);
                z = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, wfrag[s]),
                                                            __builtin_bit_cast(bf16x8, hv), z, 0, 0, 0);
            }
            const int t = tb * 16 + m;
            if (t < T) {
                float* dst = partial + (((long long)layer * S + slice) * T + t) * E + eb * 16 + 4 * kg;
                if (eb * 16 + 4 * kg + 3 < E) {
                    *(f32x4*)dst = z;
                } else {
#pragma unroll
                    for (int i = 0; i < 4; ++i)
                        if (eb * 16 + 4 * kg + i < E) dst[i] = z[i];
                }
            }
        }
    };
    if (wave < EB) score_block(wave, w2pf);
    for (int eb = wave + RW_WAVES; eb < EB; eb += RW_WAVES) {
        const int e_row = eb * 16 + m;
        u32x4 wfrag[RW_RS / 32];
#pragma unroll
        for (int s = 0; s < RW_RS / 32; ++s) {
            wfrag[s] = u32x4{0u, 0u, 0u, 0u};
            if (e_row < E) wfrag[s] = *(const u32x4*)(W2l + (long long)e_row * r + slice * RW_RS + s * 32 + kg * 8);
        }
        score_block(eb, wfrag);
    }
}

// The form for calls with few hidden units in all (one layer, a decode step): slices of 128 units would leave most
// CUs without a workgroup, and each of the few would stream its half megabyte alone, which takes as long as 26 layers
// on a full chip.  Here a slice is 16 * RB units and the columns of d are dealt out to the eight waves of a workgroup,
// each wave's share (up to SPW stages of 128 columns) requested at once and held in registers, so that the weights of
// a 2048-wide layer are all in flight together.  What remains is latency: one memory round trip, the chain of matrix
// instructions, the launch of the finalize kernel.
// The chain is walked in the row-split kernel's order -- the same stages, starting at the same column, one accumulator
// handed from wave to wave through LDS -- so that h is the same to the bit: a hidden unit whose sum falls on the other
// side of a bf16 rounding boundary moves a score by 1e-4 of its scale, and with one row nothing averages that out.
// (The hand-overs cost 1 us against waves that add their sums up: 12.5 -> 13.4 us for one 2048-wide layer and one
// token, weights from memory; the row-split kernel takes 20.3.)
static constexpr int TH_WAVES = 8;

template <int TB, int RB, int SPW>
__global__ __launch_bounds__(TH_WAVES * 64) void decode_thin_kernel(
    int T, int d, int r, int E, int act, int S, int total_wgs, long long xs_, long long w1s, long long w2s,
    const uint16_t* __restrict__ x, const uint16_t* __restrict__ W1, const uint16_t* __restrict__ W2,
    const uint16_t* __restrict__ b1, float* __restrict__ partial)
{
    constexpr int US = 16 * RB, TP = 16 * TB, KS = RW_KST / 32;
    __shared__ __attribute__((aligned(16))) float hand[RB * TB][64 * 4];           // the accumulators on their way
    __shared__ __attribute__((aligned(16))) uint16_t ht[TP * (US + HPAD)];

    int item = blockIdx.x;
    {
        const int per = total_wgs / 8, rem = total_wgs % 8;
        const int xcd = item % 8, slot = item / 8;
        item = xcd * per + (xcd < rem ? xcd : rem) + slot;
    }
    const int layer = item / S, slice = item - layer * S;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int m = lane & 15, kg = lane >> 4;
    const uint16_t* xl = x + (long long)layer * xs_;
    const uint16_t* W1l = W1 + (long long)layer * w1s;
    const uint16_t* W2l = W2 + (long long)layer * w2s;

    // fragments are fetched as in the kernels above (lane l: row l / 4, bytes 16 * (l % 4) of a 64-byte k-step)
    const int lrow = lane >> 2, lchunk = lane & 3;
    const int perm_src = (4 * m + kg) * 4;
    const uint16_t* arow = W1l + (long long)(slice * US + lrow) * d + lchunk * 8;
    const uint16_t* brow = xl + (long long)lrow * d + lchunk * 8;
    const int NST = d / RW_KST;
    const int rot = (layer * (r / RW_RS) + slice * US / RW_RS) % NST;              // where the row-split kernel starts
    const int s_begin = wave * NST / TH_WAVES, s_end = (wave + 1) * NST / TH_WAVES;   // at most SPW stages
    u32x4 fa[SPW][KS][RB], fb[SPW][KS][TB];
#pragma unroll
    for (int b = 0; b < SPW; ++b) {
        const int s = s_begin + b;
        const bool live = s < s_end;                          // wave-uniform
        const int st = s + rot < NST ? s + rot : s + rot - NST;
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
            const int off = st * RW_KST + ks * 32;
#pragma unroll
            for (int rb = 0; rb < RB; ++rb) {
                fa[b][ks][rb] = u32x4{0u, 0u, 0u, 0u};
                if (live) fa[b][ks][rb] = *(const u32x4*)(arow + (long long)rb * 16 * d + off);
            }
#pragma unroll
            for (int tb = 0; tb < TB; ++tb) {
                fb[b][ks][tb] = u32x4{0u, 0u, 0u, 0u};
                if (live && tb * 16 + lrow < T) fb[b][ks][tb] = *(const u32x4*)(brow + (long long)tb * 16 * d + off);
            }
        }
    }
    // W2 columns of this wave's first expert block: lane (m, kg) holds expert m, units 4 * kg .. + 3 of each 16
    const int EB = (E + 15) / 16;
    u32x2 w2pf[RB];
#pragma unroll
    for (int rb = 0; rb < RB; ++rb) {
        const int e_row = wave * 16 + m;
        w2pf[rb] = u32x2{0u, 0u};
        if (e_row < E) w2pf[rb] = *(const u32x2*)(W2l + (long long)e_row * r + slice * US + rb * 16 + kg * 4);
    }
    // into the operand layout, before the wave's turn
    auto to_mfma_layout = [&](u32x4& f) {
#pragma unroll
        for (int i = 0; i < 4; ++i) f[i] = (uint32_t)__builtin_amdgcn_ds_bpermute(perm_src, (int)f[i]);
    };
#pragma unroll
    for (int b = 0; b < SPW; ++b)
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
#pragma unroll
            for (int rb = 0; rb < RB; ++rb) to_mfma_layout(fa[b][ks][rb]);
#pragma unroll
            for (int tb = 0; tb < TB; ++tb) to_mfma_layout(fb[b][ks][tb]);
        }

#pragma unroll 1
    for (int w = 0; w < TH_WAVES; ++w) {
        if (wave == w) {
            f32x4 acc[RB][TB];
#pragma unroll
            for (int rb = 0; rb < RB; ++rb)
#pragma unroll
                for (int tb = 0; tb < TB; ++tb) {
                    acc[rb][tb] = f32x4{0.f, 0.f, 0.f, 0.f};
                    if (w > 0) acc[rb][tb] = *(const f32x4*)(&hand[rb * TB + tb][lane * 4]);
                }
#pragma unroll
            for (int b = 0; b < SPW; ++b)
                if (s_begin + b < s_end) {
#pragma unroll
                    for (int ks = 0; ks < KS; ++ks)
#pragma unroll
                        for (int rb = 0; rb < RB; ++rb)
#pragma unroll
                            for (int tb = 0; tb < TB; ++tb)
                                acc[rb][tb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
                                    __builtin_bit_cast(bf16x8, fa[b][ks][rb]), __builtin_bit_cast(bf16x8, fb[b][ks][tb]),
                                    acc[rb][tb], 0, 0, 0);
                }
            if (w + 1 < TH_WAVES) {
#pragma unroll
                for (int rb = 0; rb < RB; ++rb)
#pragma unroll
                    for (int tb = 0; tb < TB; ++tb) *(f32x4*)(&hand[rb * TB + tb][lane * 4]) = acc[rb][tb];
            } else {
                // acc[rb][tb][i] = h[token tb*16 + m][unit slice*US + rb*16 + 4*kg + i]
#pragma unroll
                for (int rb = 0; rb < RB; ++rb)
#pragma unroll
                    for (int tb = 0; tb < TB; ++tb) {
                        const int unit = rb * 16 + 4 * kg, tok = tb * 16 + m;
                        float h[4];
#pragma unroll
                        for (int i = 0; i < 4; ++i) {
                            float t = acc[rb][tb][i];
                            if (b1) t += bf16_bits_to_f32(b1[(long long)layer * r + slice * US + unit + i]);
                            t = round_to_bf16(t);
                            if (act != 0) t = round_to_bf16(apply_act_bf16(t, act));
                            h[i] = t;
                        }
                        *(u32x2*)(ht + tok * (US + HPAD) + unit) = u32x2{pack_bf16x2(h[0], h[1]), pack_bf16x2(h[2], h[3])};
                    }
            }
        }
        __syncthreads();
    }

    // scores of this slice: z^T[e, t] = W2[e, slice] . h^T[slice, t]; expert blocks dealt to the waves
    auto score_block = [&](int eb, const u32x2 (&wfrag)[RB]) {
#pragma unroll
        for (int tb = 0; tb < TB; ++tb) {
            f32x4 z = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int rb = 0; rb < RB; ++rb) {
                const u32x2 hv = *(const u32x2*)(ht + (tb * 16 + m) * (US + HPAD) + rb * 16 + kg * 4);
                z = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(__builtin_bit_cast(short4v, wfrag[rb]),
                                                              __builtin_bit_cast(short4v, hv), z, 0, 0, 0);
            }
            const int t = tb * 16 + m;
            if (t < T) {
                float* dst = partial + (((long long)layer * S + slice) * T + t) * E + eb * 16 + 4 * kg;
                if (eb * 16 + 4 * kg + 3 < E) {
                    *(f32x4*)dst = z;
                } else {
#pragma unroll
                    for (int i = 0; i < 4; ++i)
                        if (eb * 16 + 4 * kg + i < E) dst[i] = z[i];
                }
            }
        }
    };
    if (wave < EB) score_block(wave, w2pf);
    for (int eb = wave + TH_WAVES; eb < EB; eb += TH_WAVES) {
        const int e_row = eb * 16 + m;
        u32x2 wfrag[RB];
#pragma unroll
        for (int rb = 0; rb < RB; ++rb) {
            wfrag[rb] = u32x2{0u, 0u};
            if (e_row < E) wfrag[rb] = *(const u32x2*)(W2l + (long long)e_row * r + slice * US + rb * 16 + kg * 4);
        }
        score_block(eb, wfrag);
    }
}

static constexpr int FIN_NV = 8;                          // experts per lane of the finalize kernel at most: E <= 512

bool decode_supported(const PredictArgs& a)
{
    // each wave takes a quarter of d in k-steps of 32
    return a.dtype == 1 && a.T >= 1 && a.T <= 64 && a.r % 64 == 0 && a.d % 128 == 0 && a.E <= 64 * FIN_NV &&
           a.k <= 32;
}

// Units per slice of the thin kernel, or 0 where one of the others runs.  It is the faster one while its slices still
// find a CU each (256 of them); the price of thin slices is that every one fetches all tokens and leaves a score per
// token and expert to be added up, which limits T and E, and that the waves wait for one another, which takes rows
// long enough to make up for.  us for the row-split kernel / 16 / 32 units a slice, weights out of the caches:
//   2048 x 2048, 64 experts: 1 layer, 1 token 20.3 / 13.4 / 16.2; 2 layers, 64 tokens 26.4 / 23.2 / -; 4 layers, 1 token
//   21.2 / 17.1 / 18.3, 16 tokens 22.3 / 19.6 / 19.4, 32 tokens 23.3 / 27.3 / 22.9; 6 layers, 16 tokens 23.4 / 24.2 / 25.3
//   1024 x 4096, 16 experts: 1 layer, 1 token 29.8 / 16.0 / 20.6; 8 layers, 16 tokens 33.4 / 32.0 / 27.1
//   4096 x 2048, 256 experts: 1 layer, 1 token 26.6 / 25.3 / 22.7; 2 layers, 16 tokens 29.2 / 32.3 / 26.2
// and over d (r = 2048, 64 experts unless said; row-split / 16 units):
//   1 token     d = 256 11.1 / 11.2, 512 12.4 / 11.6, 1024 14.9 / 12.2; r = 4096: 512 12.7 / 13.3, 1024 15.4 / 14.2;
//               128 experts: 512 12.9 / 12.8, 768 14.2 / 13.0
//   32 tokens   d = 512 13.5 / 13.8, 1024 16.2 / 14.7; r = 4096: 1024 16.7 / 17.0, 1536 19.8 / 18.2; 128 experts, 2 layers:
//               1024 17.2 / 17.7, 1536 20.3 / 19.0
//   64 tokens   d = 512 15.3 / 17.0, 1024 18.7 / 18.6, 1536 22.6 / 19.7; 128 experts, 2 layers: 1536 23.6 / 24.6, 2048
//               27.1 / 26.9; r = 4096: 2048 28.3 / 29.9
// weights in the caches, 32 units against row-split, 1 token: 256 experts, 1024 x 8 layers d = 1024 1.17 times as long, 2048
// 0.98; 1 to 4 layers d = 768 0.98-1.06, 1024 0.89-1.01 (r = 1024 1.04-1.12); r = 8192 d = 2048 1.21, 4096 1.05; 64 experts d = 768 1.02,
// 1024 0.94
static int decode_thin_units(const PredictArgs& a)
{
    if (a.r % RW_RS != 0) return 0;                           // the order of sums that it keeps is the row-split kernel's
    const long long units = (long long)a.L * a.r;
    // stages of 128 columns a wave can hold in registers, by token blocks
    const int stages = (a.d / RW_KST + TH_WAVES - 1) / TH_WAVES, tb = (a.T + 15) / 16;
    int us = 0;
    if (units <= 256 * 16 && a.E <= 128 && stages <= (tb == 1 ? 6 : tb == 2 ? 4 : 2)) us = 16;
    else if (units <= 256 * 32 && a.E <= 256 && tb == 1 && stages <= 4) us = 32;
    if (us == 0) return 0;
    const bool long_sum = a.r / us >= 256;                    // slices that the finalize kernel adds up for a row
    if (long_sum && a.E > 128) return 0;
    int from = us == 32 || tb == 2 ? 1024 : tb == 1 ? 512 : 1536;
    if (long_sum) from += 512;
    if (a.E > 64) from += us == 32 ? (long_sum || a.L > 4 ? 512 : 0) : tb == 1 ? 256 : 512;
    // (32 to 63 slices are the most that one wave of the finalize kernel adds up by itself)
    if (a.E > 128 && (a.L > 4 || (a.r / us >= 32 && a.r / us < 64))) from += 512;
    return a.d >= from ? us : 0;
}

// the slices' scores in the workspace: of the d-split and the row-split kernel (sized for slices of 64 for both: callers
// know this size), and of the thin one
size_t decode_workspace_min(const PredictArgs& a)
{
    return sizeof(float) * (size_t)a.L * (size_t)(a.r / RS) * (size_t)a.T * (size_t)a.E;
}
static size_t decode_thin_bytes(const PredictArgs& a, int units)
{
    return sizeof(float) * (size_t)a.L * (size_t)(a.r / units) * (size_t)a.T * (size_t)a.E;
}

// What a call runs fastest with; with less, down to the minimum, the thin kernel's calls go to the row-split one.
// Never less for more tokens, so that a workspace for the longest batch serves the shorter ones as well as it can.
size_t decode_workspace_bytes(const PredictArgs& a)
{
    size_t need = decode_workspace_min(a);
    PredictArgs b = a;
    for (int t = 16; t < a.T + 16; t += 16) {                 // the token counts at which the kernel may change
        b.T = t < a.T ? t : a.T;
        const int units = decode_thin_units(b);
        if (units && decode_thin_bytes(b, units) > need) need = decode_thin_bytes(b, units);
    }
    return need;
}

// r in whole slices of 128: the row-split kernel (measured against the d-split kernel at 1 token: 26 layers of
// 2048 x 2048 49.2 against 53.8 us, 32 layers of 1024 x 4096 56.0 against 57.5, 48 layers of 2048 x 2048 equal;
// at 32 and 64 tokens 10-27 % faster)
static bool decode_by_rows(const PredictArgs& a) { return a.r % RW_RS == 0; }

hipError_t launch_predict_decode(const PredictArgs& a)
{
    const bool rows_kernel = decode_by_rows(a);
    int thin = decode_thin_units(a);
    if (thin && a.workspace_bytes < decode_thin_bytes(a, thin)) thin = 0;
    const int S = a.r / (thin ? thin : (rows_kernel ? RW_RS : RS));
    const int total = S * a.L;
    float* partial = (float*)a.workspace;
    const int TB = (a.T + 15) / 16;
    if (thin) {
#define PAEP_LAUNCH_THIN(TBV, RBV, SPWV)                                                                        \
    hipLaunchKernelGGL((decode_thin_kernel<TBV, RBV, SPWV>), dim3(total), dim3(TH_WAVES * 64), 0, a.stream, a.T, \
                       a.d, a.r, a.E, a.act, S, total, a.x_stride, a.w1_stride, a.w2_stride,                    \
                       (const uint16_t*)a.x, (const uint16_t*)a.W1, (const uint16_t*)a.W2,                      \
                       (const uint16_t*)a.b1, partial)
        const bool narrow = a.d <= 2 * 8 * RW_KST;            // two stages a wave
        if (thin == 16) {
            if (TB == 1)      { if (narrow) PAEP_LAUNCH_THIN(1, 1, 2); else if (a.d <= 4 * 8 * RW_KST) PAEP_LAUNCH_THIN(1, 1, 4); else PAEP_LAUNCH_THIN(1, 1, 6); }
            else if (TB == 2) { if (narrow) PAEP_LAUNCH_THIN(2, 1, 2); else PAEP_LAUNCH_THIN(2, 1, 4); }
            else              PAEP_LAUNCH_THIN(4, 1, 2);
        } else {
            if (narrow) PAEP_LAUNCH_THIN(1, 2, 2); else PAEP_LAUNCH_THIN(1, 2, 4);
        }
#undef PAEP_LAUNCH_THIN
    } else if (rows_kernel) {
#define PAEP_LAUNCH_ROWS(TBV, NSV)                                                                          \
        {                                                                                                   \
            constexpr size_t lds = (size_t)NSV * 16 * TBV * RW_KST * 2;                                     \
            static LdsLimit limit;                                                                          \
            const hipError_t e1 = ensure_lds_limit(limit, (const void*)decode_rows_kernel<TBV, NSV>, lds);  \
            if (e1 != hipSuccess) return e1;                                                                \
            hipLaunchKernelGGL((decode_rows_kernel<TBV, NSV>), dim3(total), dim3(RW_WAVES * 64), lds, a.stream, \
                               a.T, a.d, a.r, a.E, a.act, S, total, a.x_stride, a.w1_stride, a.w2_stride,   \
                               (const uint16_t*)a.x, (const uint16_t*)a.W1, (const uint16_t*)a.W2,          \
                               (const uint16_t*)a.b1, partial);                                             \
        }
        // fewer than one and a half workgroups per CU: a deeper ring
        const bool deep = total < 384;
        if (TB <= 2) { if (deep) PAEP_LAUNCH_ROWS(2, 3) else PAEP_LAUNCH_ROWS(2, 2) }
        else         { if (deep) PAEP_LAUNCH_ROWS(4, 3) else PAEP_LAUNCH_ROWS(4, 2) }
#undef PAEP_LAUNCH_ROWS
    } else {
#define PAEP_LAUNCH_DEC(TBV, UV, NBV)                                                                       \
    hipLaunchKernelGGL((decode_partial_kernel<TBV, UV, NBV>), dim3(total), dim3(DEC_THREADS), 0, a.stream,  \
                       a.T, a.d, a.r, a.E, a.act, S, total, a.x_stride, a.w1_stride, a.w2_stride,           \
                       (const uint16_t*)a.x, (const uint16_t*)a.W1, (const uint16_t*)a.W2,                  \
                       (const uint16_t*)a.b1, partial)
    switch (TB) {
    // k-steps per load batch and batches in the ring, by measurement on 26 layers of 2048 x 2048:
    // two k-steps per batch while the registers allow three waves per SIMD, one with a deeper ring beyond
    case 1: PAEP_LAUNCH_DEC(1, 2, 2); break;
    case 2: PAEP_LAUNCH_DEC(2, 2, 2); break;
    case 3: PAEP_LAUNCH_DEC(3, 1, 3); break;
    default: PAEP_LAUNCH_DEC(4, 1, 3); break;
    }
#undef PAEP_LAUNCH_DEC
    }
    const hipError_t err = hipGetLastError();
    if (err != hipSuccess) return err;
    return launch_finalize(a, partial, S, a.L, a.T, 0, 1);
}

}  // namespace paep
