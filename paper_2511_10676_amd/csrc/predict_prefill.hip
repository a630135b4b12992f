// Prefill-shaped predictor (many tokens per layer), bf16 storage: the two
// linear layers of the predictor (paper section 4.3, eq. 3) fused into one
// matrix-core kernel, with softmax and top-k (eq. 1, eq. 4) finished on chip.
//
// A workgroup owns BM tokens of one layer and walks the inner width r in chunks
// of BN hidden units (tile shapes: PfCfg below).  For a chunk it forms
//     h^T[chunk, tokens] = W1[chunk, :] . x[tokens, :]^T
// with v_mfma_f32_32x32x16_bf16, W1 rows as the A operand and token rows as
// the B operand, both copied global -> LDS without staging registers into a
// ring of XOR-swizzled stages of BK elements along d.  The waves form a
// WR x WT grid over (hidden units, tokens).  Written this way round, the
// accumulator of a 32 x 32 block holds, per lane, 16 hidden units of ONE
// token -- which is exactly what the B operand of the next product needs -- so
// the chunk of h goes, after bias, activation and rounding to bf16, straight
// from the accumulator registers into
//     z^T[E, tokens] += W2[:, chunk] . h^T[chunk, tokens]
// without touching LDS; the W2 fragments come from a copy of the chunk's W2
// slice that was brought into LDS while the chunk's first product ran (two
// 8-byte reads per lane, matching the accumulator's row order).  h and z never
// reach HBM.
// After the last chunk the waves that share a token range add their partial
// scores through LDS in a fixed order, and one to four lanes per token run the
// softmax/top-k epilogue.  r may also be split over several workgroups per
// token tile; their partial score tiles then meet in a workspace and the
// finalize kernel adds them in a fixed order.  Long calls of many experts run
// the first layer by itself and the scores as a second kernel (further down).
#include "prefill_common.h"

namespace paep {

// Tile configuration.
//   BM tokens x BN hidden units per workgroup and chunk, BK elements of d per
//   LDS tile, NS LDS stages; WR x WT waves over (hidden units, tokens); OCC
//   workgroups per CU the register budget is sized for.
// Tiles travel global -> LDS with buffer_load_dwordx4 ... lds (no staging
// registers), NS stages deep, so a tile is requested two or three iterations
// before it is used.  An LDS tile row holds BK bf16 = CPR chunks of 16 bytes; chunk c of
// row R sits in slot c ^ swz(R), chosen so that the 16-lane groups of a
// ds_read_b128 touch 64 distinct banks.  The swizzle is applied on the global
// side of the copy (a lane picks which chunk it fetches), because the LDS side
// of that instruction is fixed to lane * 16 bytes from a wave-uniform base.
//   The chunk's slice of W2 (all experts x BN hidden units) is copied to LDS
//   a chunk ahead, behind the stages, and the second layer reads its fragments
//   from there.  Read straight from global memory, every fragment of the second
//   layer is a load the next matrix instruction waits for (no registers are
//   free to request them ahead): measured, the second layer then takes 36-39%
//   of the loop with 128 and 256 experts.
template <int BM_, int BN_, int BK_, int NS_, int WR_, int WT_, int OCC_>
struct PfCfg {
    static constexpr int BM = BM_, BN = BN_, BK = BK_, NS = NS_, WR = WR_, WT = WT_, OCC = OCC_;
    static constexpr int CW = BN / 8;                       // 16-byte chunks per row of the W2 slice
    static constexpr int RPIW = 64 / CW;                    // slice rows moved by one copy instruction
    static constexpr int NW = WR * WT, THREADS = 64 * NW;
    static constexpr int WM = BN / WR, WN = BM / WT;        // wave tile: hidden units x tokens
    static constexpr int MI = WM / 32, NI = WN / 32;        // 32 x 32 blocks per wave
    static constexpr int CPR = BK / 8;                      // 16-byte chunks per tile row
    static constexpr int RPI = 64 / CPR;                    // tile rows moved by one copy instruction
    static constexpr int AJ = BN / RPI / NW, BJ = BM / RPI / NW;   // copy instructions per wave and tile
    static constexpr int STAGE_ELEMS = (BN + BM) * BK;
    static constexpr int TILE_BYTES = NS * STAGE_ELEMS * 2;
    static_assert(BK == 32 || BK == 64, "BK");
    static_assert(AJ >= 1 && BJ >= 1 && AJ * RPI * NW == BN && BJ * RPI * NW == BM, "copy split");
    static_assert(MI >= 1 && NI >= 1, "wave tile");
    static_assert((AJ + BJ) * NS <= 56, "vmcnt budget");
    static __device__ __forceinline__ int swz(int row) { return BK == 32 ? ((row >> 2) & 3) : ((row >> 1) & 7); }
};

// Token rows of the score tile that are staged in LDS at once (<= 128 KB).
template <class C, int EB32>
struct PfZRows {
    static constexpr int value = (C::BM * (EB32 * 32 + 1) * 4 > 128 * 1024) ? C::BM / 2 : C::BM;
};

// EB32: 32-expert blocks (E <= 32 * EB32).  MODE: 0 neither bias b1 nor activation, else act + 1 with an optional b1:
// one kernel for each, because the registers of a form that a call does not use are spilled by the one it does (22
// spills with all forms in one kernel, none without: 26 layers 2048 x 2048, 4096 tokens 932 -> 899 us; 48 layers
// 4096 x 2048, 256 experts 39.6 -> 36.1 ms, both with the late fragments below).
template <class C, int EB32, int MODE>
__global__ __launch_bounds__(C::THREADS, C::OCC) void prefill_kernel(
    int T, int d, int r, int E, int k, int tiles_per_layer, int main_wgs, int main_groups, int tail_wgs,
    int tail_groups, int split_tile0, int nchunks,
    long long xs_, long long w1s, long long w2s,
    const uint16_t* __restrict__ x, const uint16_t* __restrict__ W1, const uint16_t* __restrict__ W2,
    const uint16_t* __restrict__ b1, const uint16_t* __restrict__ b2,
    int32_t* __restrict__ idx, float* __restrict__ probs, float* __restrict__ logits,
    float* __restrict__ zpart, int32_t* __restrict__ counts,
    int prob_mode, float* __restrict__ margin, int tile_fastest)
{
    constexpr int BM = C::BM, BN = C::BN, BK = C::BK, NS = C::NS, WR = C::WR, WT = C::WT;
    constexpr int WM = C::WM, WN = C::WN, MI = C::MI, NI = C::NI, CPR = C::CPR, RPI = C::RPI;
    constexpr int AJ = C::AJ, BJ = C::BJ, STAGE_ELEMS = C::STAGE_ELEMS;

    extern __shared__ __attribute__((aligned(16))) unsigned char smem_raw[];
    uint16_t* tiles = (uint16_t*)smem_raw;
    float* zs = (float*)smem_raw;                         // reused after the main loop

    // A work item is (layer, token tile, group of r-chunks).  Workgroups are
    // dealt round-robin to the 8 XCDs; remap so that each XCD walks a contiguous
    // range of items with the chunk group varying fastest.  The workgroups that
    // run together on an XCD then cover a few token tiles times all chunk groups
    // of one layer: every x tile is shared by `groups` workgroups and every W1
    // chunk by several token tiles through that XCD's L2, instead of each
    // workgroup pulling its own x tile from far memory once per chunk.
    // The grid has two parts: `main_wgs` workgroups that run the first tiles with `main_groups`
    // workgroups per tile, then `tail_wgs` that run the remaining tiles with `tail_groups` each (the
    // tiles that would otherwise form a last, partly filled round of whole-tile workgroups are cut
    // finer so that every CU stays busy to the end).  Each part is remapped by itself.
    int wg = blockIdx.x;
    const bool in_tail = wg >= main_wgs;
    {
        const int part_wgs = in_tail ? tail_wgs : main_wgs;
        if (in_tail) wg -= main_wgs;
        const int per = part_wgs / 8, rem = part_wgs % 8;
        const int xcd = wg % 8, slot = wg / 8;
        wg = xcd * per + (xcd < rem ? xcd : rem) + slot;
    }
    const int groups = in_tail ? tail_groups : main_groups;
    const int cpg = nchunks / groups;
    int cg = wg % groups, tile_id = (in_tail ? main_wgs / main_groups : 0) + wg / groups;   // layer * tiles_per_layer + token tile
    if (tile_fastest) {                                    // of a layer: (group, tile), not (tile, group)
        const int column = wg / tiles_per_layer, l = column / groups;
        cg = column - l * groups;
        tile_id = l * tiles_per_layer + wg - column * tiles_per_layer;
    }
    const int layer = tile_id / tiles_per_layer;
    const int t0 = (tile_id - layer * tiles_per_layer) * BM;

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);   // wave-uniform, kept in a scalar register
    const int wr = wave / WT, wt = wave % WT;
    const int l32 = lane & 31, g = lane >> 5;
    const uint16_t* xl = x + (long long)layer * xs_;
    const uint16_t* W1l = W1 + (long long)layer * w1s;
    const uint16_t* W2l = W2 + (long long)layer * w2s;

    // global -> LDS copy assignment: per tile, wave w moves rows
    // (w*AJ + j)*RPI .. +RPI of the W1 tile (j < AJ) and likewise of the token
    // tile; lane l supplies row l / CPR, slot l % CPR of its instruction.
    // Addresses are a wave-uniform base plus a 32-bit byte offset per lane.
    uint32_t alane[AJ], blane[BJ];
#pragma unroll
    for (int j = 0; j < AJ; ++j) {
        const int row = (wave * AJ + j) * RPI + lane / CPR;
        const int chunk = (lane % CPR) ^ C::swz(row);
        alane[j] = (uint32_t)(row * d + chunk * 8) * 2u;
    }
#pragma unroll
    for (int j = 0; j < BJ; ++j) {
        const int row = (wave * BJ + j) * RPI + lane / CPR;
        const int chunk = (lane % CPR) ^ C::swz(row);
        blane[j] = (uint32_t)(row * d + chunk * 8) * 2u;   // rows past the end of the layer read as zero
    }
    const char* xtile = (const char*)(xl + (long long)t0 * d);

    f32x16 acc1[MI][NI];
    f32x16 acc2[EB32][NI];
#pragma unroll
    for (int mi = 0; mi < MI; ++mi)
#pragma unroll
        for (int ni = 0; ni < NI; ++ni)
#pragma unroll
            for (int i = 0; i < 16; ++i) acc1[mi][ni][i] = 0.f;
#pragma unroll
    for (int eb = 0; eb < EB32; ++eb)
#pragma unroll
        for (int ni = 0; ni < NI; ++ni)
#pragma unroll
            for (int i = 0; i < 16; ++i) acc2[eb][ni][i] = 0.f;

    const int NK = d / BK;
    const int n_begin = cg * cpg, n_end = n_begin + cpg;     // this work item's chunks of r
    // The slice's copies are requested after the first barrier of a chunk and must have landed, for every wave,
    // before a barrier that precedes the chunk's second layer.  A wave's wait before the barrier of tile i lets only
    // the copies of the NS - 1 youngest tiles stay in flight, so with enough tiles per chunk that holds by itself.
    const bool w2_sync = NK < NS + 2;

    // Global -> LDS requests for the next tile in sequence, one copy instruction
    // ("piece") at a time so that they can be spread between the MFMAs instead
    // of holding a wave in a burst of memory instructions.  Pieces 0..AJ-1 move
    // this wave's rows of the W1 tile, AJ..AJ+BJ-1 its rows of the token tile.
    // issue_advance() steps the tile coordinates (counters, no division); past
    // the end it stays on the last tile, which is then re-read into a stage
    // nobody looks at again: the number of copies in flight stays constant, so
    // one s_waitcnt immediate serves every iteration.
    constexpr int NP = AJ + BJ;
    int iss_kt = 0, iss_n = n_begin;
    // Buffer-addressed copies (buffer_load_dwordx4 ... lds): base and bounds in a
    // scalar resource, a 32-bit lane offset, a scalar tile offset.  Token rows
    // past the end of the layer fall outside the resource and read as zero.  (The
    // flat-addressed form of this instruction makes the compiler wait for every
    // outstanding LDS read before the next MFMA, which serialises the pipeline.)
    const __amdgpu_buffer_rsrc_t rsrc_a =
        __builtin_amdgcn_make_buffer_rsrc((void*)W1l, 0, (int)((long long)r * d * 2), 0x00020000);
    const __amdgpu_buffer_rsrc_t rsrc_b =
        __builtin_amdgcn_make_buffer_rsrc((void*)xtile, 0, (int)((long long)(T - t0) * d * 2), 0x00020000);
    auto issue_piece = [&](int slot, auto q_c) {
        constexpr int q = decltype(q_c)::value;
        uint16_t* As = tiles + slot * STAGE_ELEMS;
        if constexpr (q < AJ) {
            const int soff = (iss_n * BN * d + iss_kt * BK) * 2;
            __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrc_a, (lptr_t)(As + (wave * AJ + q) * RPI * BK), 16,
                                                     (int)alane[q], soff, 0, 0);
        } else {
            const int soff = iss_kt * BK * 2;
            __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrc_b, (lptr_t)(As + BN * BK + (wave * BJ + (q - AJ)) * RPI * BK),
                                                     16, (int)blane[q - AJ], soff, 0, 0);
        }
    };
    auto issue_advance = [&]() {
        if (iss_kt + 1 < NK) ++iss_kt;
        else if (iss_n + 1 < n_end) { iss_kt = 0; ++iss_n; }
    };
    auto issue_tile = [&](int slot) {
        static_for<NP>([&](auto q_c) { issue_piece(slot, q_c); });
        issue_advance();
    };

    // The W2 slice of a chunk in LDS, behind the stages: row e (expert) holds BN hidden units = CW
    // chunks of 16 bytes, chunk c in slot c ^ (e % CW) (swizzled on the global side of the copy, like
    // the tiles).  Rows past E lie outside the buffer resource and arrive as zeros.
    constexpr int CW = C::CW, RPIW = C::RPIW, W2ROWS = EB32 * 32;
    constexpr int W2J = W2ROWS / RPIW / C::NW;   // copy instructions per wave and slice
    static_assert(W2J * RPIW * C::NW == W2ROWS, "W2 slice copy split");
    uint16_t* w2lds = tiles + NS * STAGE_ELEMS;
    const __amdgpu_buffer_rsrc_t rsrc_w2 =
        __builtin_amdgcn_make_buffer_rsrc((void*)W2l, 0, (int)((long long)E * r * 2), 0x00020000);
    auto issue_w2 = [&](int n) {
#pragma unroll
        for (int j = 0; j < W2J; ++j) {
            const int row0 = (wave * W2J + j) * RPIW;
            const int e = row0 + lane / CW;
            const int chunk = (lane % CW) ^ (e % CW);
            __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrc_w2, (lptr_t)(w2lds + row0 * BN), 16,
                                                     (int)((uint32_t)(e * r + chunk * 8) * 2u), n * BN * 2, 0, 0);
        }
    };

    // LDS read offsets (elements) of this lane's first A / B fragment at k-step 0.
    // Block mi (ni) is a constant mi*32*BK further on (the swizzle only looks at
    // row bits below 32), and k-step ks flips slot bits: offset ^ (ks * 16).
    constexpr int KS = BK / 16;
    const int arow0 = wr * WM + l32, brow0 = wt * WN + l32;
    const int aoff0 = arow0 * BK + ((g ^ C::swz(arow0)) * 8);
    const int boff0 = BN * BK + brow0 * BK + ((g ^ C::swz(brow0)) * 8);

    // Fragment registers.  B fragments are double-buffered by k-step parity; A
    // fragments are single-buffered and refilled one by one as soon as the
    // MFMAs that use them have been issued ("rolling"), so that LDS reads for
    // the next k-step run under the current k-step's matrix work.
    bf16x8 fa[MI], fb[2][NI];
    auto read_a = [&](const uint16_t* st, auto ks_c, auto mi_c) {
        constexpr int ks = decltype(ks_c)::value, mi = decltype(mi_c)::value;
        fa[mi] = __builtin_bit_cast(bf16x8, *(const u32x4*)(st + ((aoff0 ^ (ks * 16)) + mi * 32 * BK)));
    };
    auto read_b = [&](const uint16_t* st, auto ks_c, auto buf_c) {
        constexpr int ks = decltype(ks_c)::value, buf = decltype(buf_c)::value;
#pragma unroll
        for (int ni = 0; ni < NI; ++ni)
            fb[buf][ni] = __builtin_bit_cast(bf16x8, *(const u32x4*)(st + ((boff0 ^ (ks * 16)) + ni * 32 * BK)));
    };
    auto mfma_row = [&](auto mi_c, auto buf_c) {
        constexpr int mi = decltype(mi_c)::value, buf = decltype(buf_c)::value;
#pragma unroll
        for (int ni = 0; ni < NI; ++ni)
            acc1[mi][ni] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[mi], fb[buf][ni], acc1[mi][ni], 0, 0, 0);
    };
    auto wg_barrier = [&]() {
        asm volatile("" ::: "memory");
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
    };

    // Chunk n of h is complete in acc1: round it to bf16 and feed it to the
    // second layer straight from the accumulator registers, then clear acc1.
    // acc1[mi][ni][i] = h[token wt*WN + ni*32 + l32]
    //                    [unit n*BN + wr*WM + mi*32 + 8*(i/4) + 4*g + i%4]
    // W2 fragment out of the LDS copy of the slice; ubase = first hidden unit of the 16-unit step inside the chunk
    auto w2_fragment_lds = [&](int eb, int ubase) {
        const int e = eb * 32 + l32;
        const char* row = (const char*)w2lds + e * (BN * 2) + 8 * g;
        const int c0 = ubase >> 3, sw = e % CW;
        const u32x2 lo = *(const u32x2*)(row + ((c0 ^ sw) << 4));
        const u32x2 hi = *(const u32x2*)(row + (((c0 + 1) ^ sw) << 4));
        return u32x4{lo[0], lo[1], hi[0], hi[1]};
    };
    // b1 of the layer as 32-bit words in the constant address space (scalar loads); where it starts in the middle of
    // a word, two units are put together from two words
    typedef const __attribute__((address_space(4))) uint32_t* const_words;
    const uintptr_t b1_addr = (uintptr_t)(b1 + (long long)layer * r);
    const const_words b1_words = (const_words)(b1_addr & ~(uintptr_t)3);
    const int b1_odd = (int)(b1_addr >> 1) & 1;
    auto word_pair = [&](const_words w, int i) {
        return (uint32_t)((((uint64_t)w[i + b1_odd] << 32) | w[i]) >> (16 * b1_odd));
    };
    auto second_layer = [&](int n) {
#pragma unroll
        for (int mi = 0; mi < MI; ++mi) {
#pragma unroll
            for (int s = 0; s < 2; ++s) {
                bf16x8 hb[NI];
                if constexpr (MODE == 0) {
#pragma unroll
                    for (int ni = 0; ni < NI; ++ni) {
                        const f32x16& a = acc1[mi][ni];
                        u32x4 pk = u32x4{pack_bf16x2(a[8 * s + 0], a[8 * s + 1]), pack_bf16x2(a[8 * s + 2], a[8 * s + 3]),
                                         pack_bf16x2(a[8 * s + 4], a[8 * s + 5]), pack_bf16x2(a[8 * s + 6], a[8 * s + 7])};
                        hb[ni] = __builtin_bit_cast(bf16x8, pk);
                    }
                } else {
                    uint32_t bias[4] = {0u, 0u, 0u, 0u};                         // pairs of bf16: units +0, +2, +8, +10
                    if (b1) {
                        // the 16 units of this step by scalar loads; the upper half of the wave has units 4 further on
                        // (the offset is opaque so that all steps' loads are not gathered in one place, in registers)
                        int first = __builtin_amdgcn_readfirstlane((n * BN + wr * WM + mi * 32 + 16 * s) >> 1);
                        asm volatile("" : "+s"(first));
                        const const_words w = b1_words + first;
#pragma unroll
                        for (int p = 0; p < 4; ++p) {
                            const int i = (p & 1) + 4 * (p >> 1);
                            bias[p] = g ? word_pair(w, i + 2) : word_pair(w, i);
                        }
                    }
#pragma unroll
                    for (int ni = 0; ni < NI; ++ni) {
                        u32x4 pk;
#pragma unroll
                        for (int p = 0; p < 4; ++p) {
                            float lo = acc1[mi][ni][8 * s + 2 * p] + __uint_as_float(bias[p] << 16);
                            float hi = acc1[mi][ni][8 * s + 2 * p + 1] + __uint_as_float(bias[p] & 0xFFFF0000u);
                            pk[p] = pack_bf16x2(lo, hi);                 // h is stored as bf16 before the activation
                            if constexpr (MODE > 1) {
                                lo = act_bf16<MODE - 1>(__uint_as_float(pk[p] << 16));
                                hi = act_bf16<MODE - 1>(__uint_as_float(pk[p] & 0xFFFF0000u));
                                pk[p] = pack_bf16x2(lo, hi);
                            }
                        }
                        hb[ni] = __builtin_bit_cast(bf16x8, pk);
                    }
                }
                // fragments from LDS, the next one requested before the current one is multiplied
                const int ubase = wr * WM + mi * 32 + 16 * s;
                u32x4 cur = w2_fragment_lds(0, ubase);
#pragma unroll
                for (int eb = 0; eb < EB32; ++eb) {
                    u32x4 nxt = cur;
                    if (eb + 1 < EB32) nxt = w2_fragment_lds(eb + 1, ubase);
                    const bf16x8 wa = __builtin_bit_cast(bf16x8, cur);
#pragma unroll
                    for (int ni = 0; ni < NI; ++ni)
                        acc2[eb][ni] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wa, hb[ni], acc2[eb][ni], 0, 0, 0);
                    cur = nxt;
                }
                __builtin_amdgcn_sched_barrier(0);          // keep the W2 fetches of later steps from piling up in registers
            }
        }
#pragma unroll
        for (int mi = 0; mi < MI; ++mi)
#pragma unroll
            for (int ni = 0; ni < NI; ++ni)
#pragma unroll
                for (int i = 0; i < 16; ++i) acc1[mi][ni][i] = 0.f;
    };

    // Stage recycling.  With four or more stages (LAG) the stage refilled after
    // the barrier inside tile `it` is the one tile it-1 used: every wave has
    // certainly finished reading it (its fragments fed MFMAs issued before this
    // barrier), so no wait on outstanding LDS reads is needed at the barrier.
    // With fewer stages the current tile's own stage is refilled, which requires
    // this wave's last fragment reads to have completed first.
    constexpr bool LAG = (NS >= 4);
    constexpr bool LATE_FRAGS = (MI + EB32) * NI * 16 >= 192;
    constexpr bool DEFER = (NS >= 3) && (NP % 2 == 0) && (NP / 2 <= MI);
    constexpr int HALF = NP / 2;
    constexpr int PRO = LAG ? NS - 1 : NS;                        // tiles requested before the loop
    constexpr int WAIT_LDS = PAEP_LGKM0;
    // next tile landed: the younger tiles that may still be in flight
    constexpr int WAIT_NEXT = LAG ? PAEP_VMCNT(NP * (NS - 3)) : (PAEP_VMCNT(NP * (NS - 2)) & WAIT_LDS);

    // PRO tiles requested up front; tile 0 has landed for everyone after the barrier.
    // (With DEFER the coordinates stay on the last requested tile: the main loop's
    // first deferred half-copy repeats that tile's second half, then advances.)
    issue_w2(n_begin);                                            // oldest copies in flight: landed once tile 0 has
#pragma unroll
    for (int p = 0; p < PRO; ++p) {
        static_for<NP>([&](auto q_c) { issue_piece(p, q_c); });
        if (p + 1 < PRO || !DEFER) issue_advance();
    }
    __builtin_amdgcn_s_waitcnt(PAEP_VMCNT(NP * (PRO - 1)));
    wg_barrier();

    // Main loop.  Per k-step: request the next step's B fragments, then for each
    // 32-unit block issue its MFMAs and immediately refill its A fragment for the
    // next step.  On a tile's last k-step the "next step" is the first of the next
    // tile, so the workgroup barrier that hands over LDS stages sits at the top of
    // that step: by then this wave has all its fragments of the current tile in
    // registers and its copies of the next tile have landed.  The copies that
    // refill the stage freed by that barrier are dealt out one per MFMA pair-row:
    // the first half during this last k-step, the second half during the first
    // k-step of the next tile (DEFER), or all at once when there are only two
    // stages and the data is needed one tile later.
    int slot = 0;                                                 // stage of the tile being multiplied
    int free_slot = LAG ? NS - 1 : 0;                             // stage that the next barrier releases for refilling
    int fill_slot = PRO - 1;                                      // stage whose second half of copies is pending
    {
        static_for<MI>([&](auto mi_c) { read_a(tiles, IC<0>{}, mi_c); });
        read_b(tiles, IC<0>{}, IC<0>{});
        __builtin_amdgcn_s_waitcnt(WAIT_LDS);                     // nothing pending on loop entry
    }
    for (int n = n_begin; n < n_end; ++n) {
        for (int kt = 0; kt < NK; ++kt) {
            const uint16_t* st = tiles + slot * STAGE_ELEMS;
            const int nslot = (slot + 1 == NS) ? 0 : slot + 1;
            const uint16_t* stn = tiles + nslot * STAGE_ELEMS;
            static_for<KS>([&](auto ks_c) {
                constexpr int ks = decltype(ks_c)::value;
                constexpr int cur = ks & 1, nxt = cur ^ 1;
                if constexpr (ks + 1 < KS) {
                    read_b(st, IC<ks + 1>{}, IC<nxt>{});
                    __builtin_amdgcn_sched_barrier(0);
                    static_for<MI>([&](auto mi_c) {
                        constexpr int mi = decltype(mi_c)::value;
                        mfma_row(mi_c, IC<cur>{});
                        __builtin_amdgcn_sched_barrier(0);
                        if constexpr (DEFER && ks == 0 && mi < HALF) {
                            // second half of the copies for the stage released one tile ago
                            // (on the very first tile this repeats copies the prologue made: harmless)
                            issue_piece(fill_slot, IC<HALF + mi>{});
                            if constexpr (mi == HALF - 1) issue_advance();
                        }
                        read_a(st, IC<ks + 1>{}, mi_c);
                        __builtin_amdgcn_sched_barrier(0);
                    });
                } else {
                    __builtin_amdgcn_s_waitcnt(WAIT_NEXT);
                    wg_barrier();
                    // Every wave is past the previous chunk's second layer here, so the slice in LDS may
                    // be replaced by this chunk's; it is read at the end of the chunk, NK - 1 tiles later.
                    if (kt == 0 && n > n_begin) issue_w2(n);
                    if constexpr (!DEFER) issue_tile(free_slot);
                    // With 192 accumulators there is no room to carry the next tile's first fragments
                    // across the second layer: fetch them after it instead.
                    const bool prefetch = !(LATE_FRAGS && kt == NK - 1);
                    if (prefetch) read_b(stn, IC<0>{}, IC<nxt>{});
                    __builtin_amdgcn_sched_barrier(0);
                    static_for<MI>([&](auto mi_c) {
                        constexpr int mi = decltype(mi_c)::value;
                        mfma_row(mi_c, IC<cur>{});
                        __builtin_amdgcn_sched_barrier(0);
                        if constexpr (DEFER && mi < HALF) issue_piece(free_slot, IC<mi>{});
                        if (prefetch) read_a(stn, IC<0>{}, mi_c);
                        __builtin_amdgcn_sched_barrier(0);
                    });
                    fill_slot = free_slot;
                }
            });
            free_slot = LAG ? slot : nslot;
            slot = nslot;
        }
        if (w2_sync) {
            // few tiles per chunk: the slice's copies may still be among the youngest in flight
            __builtin_amdgcn_s_waitcnt(PAEP_VMCNT(0));
            wg_barrier();
        }
        second_layer(n);
        if constexpr (LATE_FRAGS) {
            const uint16_t* stc = tiles + slot * STAGE_ELEMS;
            static_for<MI>([&](auto mi_c) { read_a(stc, IC<0>{}, mi_c); });
            read_b(stc, IC<0>{}, IC<(((KS - 1) & 1) ^ 1)>{});
        }
        __builtin_amdgcn_s_waitcnt(WAIT_LDS);                     // next tile's first fragments have landed
    }
    // all tile reads done, and the copies of the pipeline's end landed, before LDS is reused
    __builtin_amdgcn_s_waitcnt(PAEP_VMCNT(0));
    __syncthreads();

    // Activation counters of this workgroup's rows, kept in LDS behind the score
    // tile and flushed to the layer's counts once at the end: at most E global
    // atomics per workgroup instead of one per selection.
    int32_t* cnt_lds = (int32_t*)(smem_raw + sizeof(float) * (size_t)PfZRows<C, EB32>::value * (size_t)(E + 1));
    if (counts)
        for (int e = tid; e < E; e += C::THREADS) cnt_lds[e] = 0;
    auto flush_counts = [&]() {                              // after a barrier that follows the last row's epilogue
        if (counts)
            for (int e = tid; e < E; e += C::THREADS) {
                const int c = cnt_lds[e];
                if (c) atomicAdd(&counts[(long long)layer * E + e], c);
            }
    };

    // acc2[eb][ni][i] = partial score of token wt*WN + ni*32 + l32,
    //                   expert eb*32 + 8*(i/4) + 4*g + i%4, over this wave's hidden units.
    // The score tile goes to LDS ZROWS tokens at a time (all of it unless E is
    // large); waves that share tokens add their parts there, wr = 0 first.
    constexpr int ZROWS = PfZRows<C, EB32>::value;
    constexpr int ZG = C::THREADS / ZROWS;                 // lanes per token row in the epilogue
    static_assert(ZROWS % WN == 0 && (ZG == 1 || ZG == 2 || ZG == 4), "epilogue split");
    const int ZP = E + 1;
    const bool split = groups > 1;

    // registers -> zs for token rows [zp*ZROWS, (zp+1)*ZROWS); b2 is added here only when r is not split
    auto regs_to_lds = [&](int zp) {
        const bool mine = (wt * WN) / ZROWS == zp;
#pragma unroll
        for (int pass = 0; pass < WR; ++pass) {
            if (mine && wr == pass) {
#pragma unroll
                for (int eb = 0; eb < EB32; ++eb)
#pragma unroll
                    for (int ni = 0; ni < NI; ++ni)
#pragma unroll
                        for (int i = 0; i < 16; ++i) {
                            const int e = eb * 32 + 8 * (i >> 2) + 4 * g + (i & 3);
                            const int tl = wt * WN + ni * 32 + l32 - zp * ZROWS;
                            if (e < E) {
                                float v = acc2[eb][ni][i];
                                if (pass == 0) {
                                    if (b2 && !split) v += bf16_bits_to_f32(b2[(long long)layer * E + e]);
                                } else {
                                    v = zs[tl * ZP + e] + v;
                                }
                                zs[tl * ZP + e] = v;
                            }
                        }
            }
            __syncthreads();
        }
    };
    // zs -> idx, probs (and logits) for the same rows
    auto finish_rows = [&](int zp) {
        const int tbase = t0 + zp * ZROWS;
        if (logits) {
            for (int i = tid; i < ZROWS * E; i += C::THREADS) {
                const int tl = i / E, e = i - tl * E;
                if (tbase + tl < T) logits[((long long)layer * T + tbase + tl) * E + e] = zs[tl * ZP + e];
            }
        }
        const int tl = tid / ZG, gg = tid % ZG;
        // the lanes of a group take the same branch (same token)
        if (tbase + tl < T) {
            const long long row = (long long)layer * T + tbase + tl;
            const EpilogueOut eo{prob_mode, margin ? margin + row : nullptr, counts ? cnt_lds : nullptr};
            const float* zrow = zs + tl * ZP;
            row_softmax_topk_upto16<ZG, (EB32 > 2)>([&](int e) { return zrow[e]; }, E, k, gg, idx + row * k, probs + row * k, eo);
        }
        __syncthreads();
    };

    if (!split) {
#pragma unroll 1
        for (int zp = 0; zp < BM / ZROWS; ++zp) {
            regs_to_lds(zp);
            finish_rows(zp);
        }
        flush_counts();
        return;
    }

    // r is split over `groups` workgroups: park this group's score tile in the workspace as
    // zpart[tile][group][token][expert]; finalize_kernel adds the groups in ascending order and finishes the rows.
    // (The workgroup that arrived last used to do that here: it went through groups x BM x E scores by itself, 8 loads
    // at a time, while the rest of the chip was done -- 512 tokens of a 2048 x 2048 layer in 16 groups 75 -> 36 us.)
    float* zmine = zpart + ((long long)(tile_id - split_tile0) * groups + cg) * BM * E;
#pragma unroll 1
    for (int zp = 0; zp < BM / ZROWS; ++zp) {
        regs_to_lds(zp);
        for (int i = tid; i < ZROWS * E; i += C::THREADS) {
            const int tl = i / E, e = i - tl * E;
            if (t0 + zp * ZROWS + tl < T) zmine[(long long)(zp * ZROWS + tl) * E + e] = zs[tl * ZP + e];
        }
        __syncthreads();
    }
}

// Configurations.  The LDS holds the stages and, behind them, the chunk's W2 slice (E rounded up to 32 rows x BN hidden
// units x 2 bytes):
//   256 x 256 (E <= 128, r a multiple of 256) and 256 tokens x 128 units (65 to 256 experts): prefill256.hip.
//   Flat      256 x 256 for E <= 64 and short rows (flat_wanted), 8 waves: a chunk is a few of prefill256.hip's stages there,
//             and its ends are what counts.
//   Few       128 to 256 tokens x 256 (prefill256.hip): short inputs of up to 128 experts (few_plan).
//   Small     128 x 128, 4 waves, two workgroups per CU (4 x 16 KB + 16 KB slice each): short inputs otherwise
//             and any r that is a multiple of 128.  SmallWide: the same for E > 64 (64 KB slice).
//   Tiny      64 x 64, 4 waves, four 64-wide stages, two workgroups per CU: calls whose 128 x 128 tiles would not reach
//             every CU.  What bounds it is the chain of stages, 0.5 us each whatever is tried on it (eight stages, all
//             of a stage's fragments read a stage ahead: no faster); what the half microsecond consists of is not known.
typedef PfCfg<256, 256, 32, 4, 2, 4, 1> CfgFlat;
struct Cfg256 { static constexpr int BM = 256, BN = 256; };
struct Cfg256x128 { static constexpr int BM = 256, BN = 128; };
typedef PfCfg<128, 128, 32, 4, 2, 2, 2> CfgSmall;
typedef PfCfg<128, 128, 32, 4, 1, 4, 1> CfgSmallWide;
typedef PfCfg<64, 64, 64, 4, 2, 2, 2> CfgTiny;

template <class C, int EB32>
static size_t cfg_lds_bytes(int E)
{
    // score tile of the epilogue, then E activation counters
    const size_t z = sizeof(float) * (size_t)PfZRows<C, EB32>::value * (size_t)(E + 1) + sizeof(int32_t) * (size_t)E;
    // main loop: the stages, then the W2 slice (32 * EB32 rows of BN hidden units)
    const size_t loop = (size_t)C::TILE_BYTES + (size_t)EB32 * 32 * C::BN * 2;
    return z > loop ? z : loop;
}

bool prefill_supported(const PredictArgs& a)
{
    // the copy offsets are 32-bit byte offsets into one layer's W1 and x
    const int list = a.k + ((a.margin && a.k < a.E) ? 1 : 0);     // the epilogue keeps sorted lists of up to 16
    return a.dtype == 1 && a.T >= 1 && a.d % 32 == 0 && a.r % 128 == 0 && a.E <= 256 && list <= 16 &&
           (long long)a.r * a.d * 2 < (1ll << 31) && ((long long)a.T + 256) * a.d * 2 < (1ll << 31);
}

// How many workgroups share one token tile (each takes r / BN / groups chunks
// and the finalize kernel adds their score tiles).
//  * Fewer tiles than CU slots (short inputs, down to a single tile per layer,
//    where the kernel is a weight-streaming problem): split until there are
//    about one and a half workgroups per CU, so that the whole chip pulls on
//    HBM.
//  * Many tiles: splitting lets the workgroups of one XCD share a token tile
//    through L2 instead of each pulling its own from far memory once per chunk
//    (measured: 3.3x fewer bytes fetched past L2 at 8 groups), but every extra
//    group costs a pipeline fill and a score tile written and re-read.  Two
//    groups where the token tile is large (d >= 4096: 2 MB per tile; one / two /
//    four groups, 8192 tokens, us: 32 layers 1024 x 4096, 16 experts 1658 / 1559 / 1598; 2048 x 4096,
//    64 experts 3635 / 3297 / 3245); at d = 2048 there is nothing to gain (1658 / 1669 / 1742; 48 layers,
//    128 experts 2708 / 2698 / 2907).  With more than the least
//    workspace d = 3072 takes two as well (1489 / 1300 / 1378) and d = 5120 four (even_plan).
template <class C>
static int prefill_groups(const PredictArgs& a)
{
    const int NC = a.r / C::BN;
    const long long tiles = (long long)((a.T + C::BM - 1) / C::BM) * a.L;
    if (tiles < 256) {
        int g = 1;
        while (g < NC && (tiles * g < 384 || NC % g != 0)) ++g;
        return g;
    }
    if (NC % 2 != 0) return 1;
    return ((long long)a.d * C::BM * 2 >= (2ll << 20)) ? 2 : 1;
}

// How a launch is laid out: `main_tiles` token tiles with `main_groups` workgroups each, then
// `tail_tiles` with `tail_groups` each.  With whole-tile workgroups (main_groups = 1) the tiles beyond the
// last full round of 256 would keep a fraction of the CUs busy for a whole tile's duration; where it pays
// they are cut along r into pieces short enough to fill every CU evenly, at the price of the score-tile
// exchange.  2048 x 2048 layers of 16 tiles, 64 experts, whole / in 2 / 4 / 8 pieces, us: 17 layers (a tail of 16) 730 / 569 /
// 493 / 474, 20 (64) 764 / 604 / 561 / 560, 24 (128) 795 / 650 / 662 / 678, 26 (160) 811 / 792 / 734 / 730, 28 (192) 837 / 840 /
// 770 / 800, 30 (224) 884 / 842 / 858 / 856; 128 experts 26 layers 864 / 876 / 795 / 800.
struct PfLayout {
    int main_tiles, main_groups, tail_tiles, tail_groups;
    int split_tile0, split_tiles, split_groups;              // the tiles that go through the workspace
};
template <class C>
static PfLayout cfg_layout(const PredictArgs& a)
{
    const int NC = a.r / C::BN;
    const int tiles = ((a.T + C::BM - 1) / C::BM) * a.L;
    PfLayout f{tiles, prefill_groups<C>(a), 0, 1, 0, 0, 1};
    if (f.main_groups > 1) {
        f.split_tiles = tiles;
        f.split_groups = f.main_groups;
        return f;
    }
    constexpr int CUS = 256;
    const int tail = tiles % CUS;
    if (tiles < CUS || tail == 0) return f;
    // Time of the tail in units of one whole-tile workgroup on a full chip: uncut, the tail's workgroups run faster than on
    // a full chip (the clock rises when CUs idle); cut g ways they take 1/g plus about 0.08 each (pipeline fill, the
    // score-tile exchange, and the XCD's workgroups no longer walking the same chunk of W1).  The constants are those of the
    // eight-wave kernels, whose exchange was dearer: tails of 160 to 224 tiles stay whole although cuts in four win above.
    int best = 1;
    double best_t = 0.55 + 0.40 * tail / CUS;
    for (int g = 2; g <= 8 && g <= NC; g *= 2) {
        if (NC % g != 0) continue;
        const double t = (double)((tail * g + CUS - 1) / CUS) * (1.0 / g + 0.08);
        if (t < best_t - 0.05) { best_t = t; best = g; }
    }
    if (best == 1) return f;
    f.main_tiles = tiles - tail;
    f.tail_tiles = tail;
    f.tail_groups = best;
    f.split_tile0 = f.main_tiles;
    f.split_tiles = tail;
    f.split_groups = best;
    return f;
}

template <class C>
static size_t cfg_workspace_bytes(const PredictArgs& a)
{
    const PfLayout f = cfg_layout<C>(a);
    if (f.split_tiles == 0) return 0;
    // score tiles, and a word per tile that nothing uses any more: callers know this size
    return (size_t)f.split_tiles * f.split_groups * C::BM * a.E * sizeof(float) +
           (((size_t)f.split_tiles * sizeof(int) + 15) / 16) * 16;
}

// The order of an XCD's share of the grid where it is less than a layer: chunk groups fastest (many rows of W1, few tokens) or
// token tiles fastest, whichever touches fewer rows in all; they cross to the XCD's L2 once for all its workgroups.  In
// the order of groups / of tiles, us, 2048 x 2048, 64 experts: one layer of 1024 tokens 28.9 / 27.4, 2000 tokens 40.4 / 37.4
// (equally many rows; 256 experts 63.6 / 60.7), r = 4096, d = 1024, 512 tokens 26.4 / 24.4, r = 1024, d = 4096 25.4 / 24.5, 300
// and 512 tokens the same; where the rule keeps groups 4000 tokens 60.6 / 61.7, 20000 tokens 229 / 245.
// Only where the rows that the order of groups touches do not fit the 4 MB of that L2: below 3 MB nothing is gained and up to a
// tenth lost (256 experts, d = 4096, r = 512, 384 tokens 59.4 / 65.5); with more than 64 experts in 64 x 64 tiles, whose score
// tiles are as large as their operands, below 7 MB (128 experts, 4 layers of 512 tokens, 1024 x 1024 30.6 / 34.8; 3 of 256,
// r = 2048 29.0 / 32.2; 2048 x 2048, one of 301 27.4 / 28.4; but one of 700 34.1 / 32.2).  Of hidden units a chunk's rows
// count, not a workgroup's: token rows are read again for every chunk (4 layers of 2310 tokens, 3456 x 4096 in 9 groups of three
// chunks 365 / 441).
static bool tile_fastest(const PredictArgs& a, int bm, int bn, int groups)
{
    const int tiles = (a.T + bm - 1) / bm, share = tiles * a.L * groups / 8;
    if (share == 0 || share >= tiles * groups) return false;
    auto rows = [&](int n, int size, int other) {              // n side by side, of `size` rows each
        return (n < share ? n : share) * size + (share + n - 1) / n * other;
    };
    const int by_groups = rows(groups, bn, bm);
    const long long mb = bm == 64 && a.E > 64 ? 7 : 3;
    return rows(tiles, bm, bn) <= by_groups && 2ll * a.d * by_groups >= mb << 20;
}
template <class C>
static bool tile_fastest(const PredictArgs& a, const PfLayout& f)
{
    return f.tail_tiles == 0 && tile_fastest(a, C::BM, C::BN, f.main_groups);
}

template <class C, int EB32, int MODE>
static hipError_t launch_mode(const PredictArgs& a)
{
    const int tiles = (a.T + C::BM - 1) / C::BM;
    const PfLayout f = cfg_layout<C>(a);
    const int main_wgs = f.main_tiles * f.main_groups, tail_wgs = f.tail_tiles * f.tail_groups;
    const size_t lds = cfg_lds_bytes<C, EB32>(a.E);
    float* zpart = (float*)a.workspace;
    auto kern = prefill_kernel<C, EB32, MODE>;
    static LdsLimit limit;
    hipError_t err = ensure_lds_limit(limit, (const void*)kern, lds);
    if (err != hipSuccess) return err;
    hipLaunchKernelGGL(kern, dim3(main_wgs + tail_wgs), dim3(C::THREADS), lds, a.stream, a.T, a.d, a.r, a.E, a.k,
                       tiles, main_wgs, f.main_groups, tail_wgs, f.tail_groups, f.split_tile0, a.r / C::BN,
                       a.x_stride, a.w1_stride, a.w2_stride, (const uint16_t*)a.x,
                       (const uint16_t*)a.W1, (const uint16_t*)a.W2, (const uint16_t*)a.b1,
                       (const uint16_t*)a.b2, a.idx, a.probs, a.logits, zpart, a.counts, a.prob_mode,
                       a.margin, (int)tile_fastest<C>(a, f));
    err = hipGetLastError();
    if (err != hipSuccess || f.split_tiles == 0) return err;
    return launch_finalize(a, zpart, f.split_groups, f.split_tiles, C::BM, f.split_tile0, tiles);
}

// Tiles of 224 tokens instead of 256 (E <= 64, whole-tile workgroups): where the last round of 256 workgroups is filled better by
// them.  Time in units of a token of a full round; a partly filled round as in cfg_layout.  The same outputs to the bit.
// The same kernel, whole tiles, one box, 2048 x 2048, 64 experts, 256 / 224 tokens, us: 26 x 4096 tokens (416 tiles of 256, 494 of
// 224; 0.93 here) 828 / 759, 26 x 3840 792 / 733, 25 x 4096 786 / 741, with GELU 935 / 879, 26 x 4096, d = 768, r = 512 98 / 92,
// 16 experts, d = 2080, r = 1024 451 / 428; and where the rule keeps 256 (1.07 and more): 32 x 4096 896 / 1134, 27 x 4096 837 / 1061,
// 48 x 4096 1300 / 1516, 44 x 4096, d = 1024 646 / 767.
static bool tiles_of_224_wanted(const PredictArgs& a)
{
    if (a.E > 64) return false;
    auto time = [&](int tokens) {
        const int tiles = ((a.T + tokens - 1) / tokens) * a.L, rounds = tiles / 256, tail = tiles % 256;
        return tokens * (rounds + (tail ? 0.55 + 0.40 * tail / 256 : 0.0));
    };
    return time(224) < 0.97 * time(256);
}

// Flat or prefill256.hip for E <= 64: the latter's stages are 64 columns wide, so that an odd multiple of 32 costs 32 columns
// more, and the ends of a chunk are bare under its one wave per SIMD.  Biases b1 and activations, whose Flat forms spill,
// turn that round.  Flat / prefill256, us: 16 layers of 8192 tokens, d = 64, 16 experts, r = 512 20.6 / 23.9; 32 x 4096 tokens, r = 2048, 64 experts,
// d = 160 120 / 143, 224 143 / 166, 256 155 / 166, 320 183 / 191, 416 222 / 248, 608 307 / 318, with SiLU, r = 1024, d = 160
// 154 / 134, with b1 alone 120 / 99; from d = 384 (an odd multiple of 32: 640) on prefill256 is level or faster.  Split calls of more than 32 experts with one
// or two chunks a workgroup wait for their score tiles, which prefill256 writes faster: 4 x 9000 tokens, r = 1024, 64 experts,
// d = 160 64 / 54, 608 92 / 80.
static bool flat_wanted(const PredictArgs& a)
{
    if (a.d <= 128) return true;
    if (a.act != 0 || a.b1 || a.d > (a.d % 64 != 0 ? 608 : 320)) return false;
    const int groups = prefill_groups<Cfg256>(a);
    return a.E <= 32 || groups == 1 || a.r / Cfg256::BN / groups > 2;
}

static hipError_t launch_tiles_of_224(const PredictArgs& a)
{
    const int tiles = (a.T + 223) / 224;
    return launch_prefill256(a, PrefillGrid{tiles, tiles * a.L, 1, 0, 1, 0, nullptr, 0}, 224, Cfg256::BN, nullptr);
}

template <class C>
static hipError_t launch_cfg256(const PredictArgs& a)
{
    const PfLayout f = cfg_layout<C>(a);
    const int tiles = (a.T + C::BM - 1) / C::BM;
    float* zpart = (float*)a.workspace;
    const PrefillGrid grid{tiles, f.main_tiles * f.main_groups, f.main_groups, f.tail_tiles * f.tail_groups, f.tail_groups,
                           f.split_tile0, zpart, 0};
    const hipError_t err = launch_prefill256(a, grid, C::BM, C::BN, nullptr);
    if (err != hipSuccess || f.split_tiles == 0) return err;
    return launch_finalize(a, zpart, f.split_groups, f.split_tiles, C::BM, f.split_tile0, tiles);
}

template <class C, int EB32>
static hipError_t launch_cfg(const PredictArgs& a)
{
    switch (a.act) {
    case 0: return a.b1 ? launch_mode<C, EB32, 1>(a) : launch_mode<C, EB32, 0>(a);
    case 1: return launch_mode<C, EB32, 2>(a);
    default: return launch_mode<C, EB32, 3>(a);
    }
}

// ---------------------------------------------------------------------------
// Two passes for many experts.  The fused kernel keeps E scores per token in accumulators beside the chunk of h, and
// with more than 64 experts that costs it the tile shape: 256 x 128 tiles (E up to 256) need half as many bytes again
// per flop through the CU's copy path as 256 x 256 ones, which is what the loop waits for, and waves side by side along
// tokens read 1.1-1.25 LDS fragments per matrix instruction.  Here the first layer runs by itself (prefill256.hip),
// h takes a round trip through memory (2 r bytes per token each way, 0.1-0.2 of the layer's bytes at 2048-wide rows),
// and a second kernel forms the scores.
//
// scores_of_h_kernel: a workgroup owns 128 (E <= 128) or 256 tokens, a wave 32 of them and all experts.  h arrives in the
// layout of the matrix instruction, straight into registers, two stages of 64 units ahead, and takes its activation here:
// beside the reading, which bounds this kernel, it costs little, while the first layer's waves have nothing to put beside
// it.  W2's columns of a stage are copied to LDS for all waves (swizzled like the tiles of token rows above), a ring of
// three stages.  Where r is not sliced, a token's scores lie in four lanes' accumulators, which select and write its outputs
// (48 layers of 6011 tokens, 128 experts, GELU 2433 -> 2390 us, of 32768 tokens, 256 experts 23.42 -> 22.99 ms against scores
// through memory); else they go to memory as [tile][slice][256][E] and finalize.hip does the rest.
// Up to 128 experts three workgroups of four waves fit a CU (48 KB of stages each).  Eight waves and two workgroups left half of
// the CUs with one of a batch's 384: 16 layers of 6011 tokens, 2048 x 2048, 128 experts, GELU 860 -> 832 us (both kernels),
// 48 layers 2460 -> 2368; 8 x 20000, d = 3072, r = 512, SiLU 510 -> 488; 32 x 4000, d = 2560, r = 1024 623 -> 615.
// ---------------------------------------------------------------------------
static constexpr int SH_BM = 256, SH_BN = 64, SH_NST = 3;

// EB: blocks of 16 experts
template <int EB> constexpr int sh_waves() { return EB <= 8 ? 4 : 8; }

// what a call writes
struct RowOutputs {
    int k, prob_mode;
    const uint16_t* b2;
    int32_t* idx;
    float *probs, *logits, *margin;
    int32_t* counts;
};

// The outputs of a token by the four lanes, 16 apart, that hold its scores: z[eb][i] is expert 16 eb + 4 g + i.
template <int KMAX, int EB>
__device__ __forceinline__ void finish_token(const f32x4 (&z)[EB], int E, int g, long long row, const RowOutputs& o, int32_t* counts)
{
    TopList<KMAX> top;
    top.clear();
    constexpr int JB = KMAX > 2 ? KMAX / 4 : 1;              // blocks whose keys are sorted together
#pragma unroll
    for (int e0 = 0; e0 < EB; e0 += JB) {
        skey more[JB * 4];
#pragma unroll
        for (int j = 0; j < JB; ++j)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int e = (e0 + j) * 16 + 4 * g + i;
                more[4 * j + i] = e < E ? make_key(z[e0 + j][i], e) : NO_KEY;
            }
        if constexpr (KMAX > 2) {
            top.add(more, e0 == 0);
        } else {
#pragma unroll
            for (int i = 0; i < 4; ++i) top.insert(more[i]);
        }
    }
    top.template merge_group<4, 16>();
    const EpilogueOut eo{o.prob_mode, o.margin ? o.margin + row : nullptr, counts};
    write_selection<KMAX, 4, 16>(top, E, o.k, g, o.idx + row * o.k, o.probs + row * o.k, eo, [&](float m) {
        // four chains: a single one of up to 64 terms rounds more than finalize_rows_kernel's of 16 (256 experts, the first
        // probability against float64, rms: 7.7e-8, here and there 5.4e-8)
        f32x4 s{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int eb = 0; eb < EB; ++eb)
#pragma unroll
            for (int i = 0; i < 4; ++i)
                if (eb * 16 + 4 * g + i < E && z[eb][i] == z[eb][i]) s[i] += __expf(z[eb][i] - m);
        return (s[0] + s[1]) + (s[2] + s[3]);
    });
}

template <int EB, int ACT>
__global__ __launch_bounds__(sh_waves<EB>() * 64, EB <= 8 ? 3 : 2) void scores_of_h_kernel(
    int T, int r, int E, int tiles_per_layer, int slices, long long w2s, const u32x4* __restrict__ h,
    const uint16_t* __restrict__ W2, float* __restrict__ zpart, RowOutputs out)
{
    constexpr int ROWS = EB * 16, STAGE_BYTES = ROWS * SH_BN * 2;
    constexpr int WAVES = sh_waves<EB>(), PARTS = 8 / WAVES; // workgroups per tile of 256 tokens
    constexpr int W2J = ROWS / 8 / WAVES;                   // copy instructions per wave and stage, 8 rows each
    constexpr int KS = SH_BN / 32, NB = SH_BM / 8 / 16;     // steps of 32 units; blocks of 16 tokens per wave
    static_assert(W2J * 8 * WAVES == ROWS, "rows divide among the waves");
    extern __shared__ __attribute__((aligned(16))) unsigned char smem_raw[];

    const int slice = blockIdx.x % slices, tile_id = blockIdx.x / slices / PARTS, part = blockIdx.x / slices % PARTS;
    const int layer = tile_id / tiles_per_layer, t0 = (tile_id - layer * tiles_per_layer) * SH_BM;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l16 = lane & 15, g = lane >> 4;
    const int nst = r / SH_BN;
    const int s_begin = (int)((long long)slice * nst / slices), s_end = (int)((long long)(slice + 1) * nst / slices);
    const int first = (part * WAVES + wave) * NB * 16;      // token in the tile
    const u32x4* hw = h + ((long long)(tile_id * (SH_BM / 16) + first / 16) * (r / 32)) * 64 + lane;

    const __amdgpu_buffer_rsrc_t rsrc_w2 = __builtin_amdgcn_make_buffer_rsrc(
        (void*)(W2 + (long long)layer * w2s), 0, (int)((long long)E * r * 2), 0x00020000);
    uint32_t w2lane[W2J];
#pragma unroll
    for (int j = 0; j < W2J; ++j) {
        const int e = (wave * W2J + j) * 8 + (lane >> 3);
        w2lane[j] = (uint32_t)(e * r + (((lane & 7) ^ ((e >> 1) & 7)) * 8)) * 2u;   // rows past E lie outside the resource: zeros
    }
    auto issue_w2 = [&](int st, int slot) {
#pragma unroll
        for (int j = 0; j < W2J; ++j)
            __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrc_w2, (lptr_t)(smem_raw + slot * STAGE_BYTES + (wave * W2J + j) * 1024),
                                                     16, (int)w2lane[j], st * SH_BN * 2, 0, 0);
    };
    u32x4 hb[SH_NST][KS][NB];
    auto load_h = [&](auto buf_c, int st) {
        constexpr int buf = decltype(buf_c)::value;
#pragma unroll
        for (int ks = 0; ks < KS; ++ks)
#pragma unroll
            for (int b = 0; b < NB; ++b) hb[buf][ks][b] = hw[((long long)b * (r / 32) + st * KS + ks) * 64];
    };
    f32x4 acc[EB][NB];
#pragma unroll
    for (int eb = 0; eb < EB; ++eb)
#pragma unroll
        for (int b = 0; b < NB; ++b) acc[eb][b] = f32x4{0.f, 0.f, 0.f, 0.f};

    // Stage s is requested two stages ahead, W2 first; past the end the last stage is requested again, into a slot
    // nobody reads any more, so that the count of requests in flight stays the same.
    constexpr int WAIT_STAGE = PAEP_VMCNT((SH_NST - 2) * (W2J + KS * NB));
    static_for<SH_NST - 1>([&](auto b_c) {
        constexpr int b = decltype(b_c)::value;
        const int st = s_begin + b < s_end ? s_begin + b : s_end - 1;
        issue_w2(st, b);
        __builtin_amdgcn_sched_barrier(0);
        load_h(b_c, st);
        __builtin_amdgcn_sched_barrier(0);
    });
    for (int s0 = s_begin; s0 < s_end; s0 += SH_NST) {
        static_for<SH_NST>([&](auto b_c) {
            constexpr int b = decltype(b_c)::value, nb = (b + SH_NST - 1) % SH_NST;
            const int st = s0 + b;
            if (st < s_end) {                               // uniform over the workgroup
                __builtin_amdgcn_s_waitcnt(WAIT_STAGE);     // this wave's part of the stage has landed
                asm volatile("" ::: "memory");
                __builtin_amdgcn_s_barrier();               // everyone's has; and everyone is done with the stage before
                asm volatile("" ::: "memory");
                const int sn = st + SH_NST - 1 < s_end ? st + SH_NST - 1 : s_end - 1;
                issue_w2(sn, nb);
                __builtin_amdgcn_sched_barrier(0);
                load_h(IC<nb>{}, sn);
                __builtin_amdgcn_sched_barrier(0);
                const uint16_t* stage = (const uint16_t*)(smem_raw + b * STAGE_BYTES);
#pragma unroll
                for (int ks = 0; ks < KS; ++ks) {
                    bf16x8 hv[NB];
                    if constexpr (ACT > 0) __builtin_amdgcn_sched_barrier(0);    // one step's at a time: registers
#pragma unroll
                    for (int n = 0; n < NB; ++n) {
                        u32x4 v = hb[b][ks][n];
                        if constexpr (ACT > 0)
#pragma unroll
                            for (int q = 0; q < 4; ++q)
                                v[q] = pack_bf16x2(act_bf16<ACT>(__uint_as_float(v[q] << 16)), act_bf16<ACT>(__uint_as_float(v[q] & 0xFFFF0000u)));
                        hv[n] = __builtin_bit_cast(bf16x8, v);
                    }
#pragma unroll
                    for (int eb = 0; eb < EB; ++eb) {
                        const int e = eb * 16 + l16;
                        const bf16x8 w = __builtin_bit_cast(bf16x8, *(const u32x4*)(stage + e * SH_BN + (((4 * ks + g) ^ ((l16 >> 1) & 7)) * 8)));
#pragma unroll
                        for (int n = 0; n < NB; ++n) acc[eb][n] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w, hv[n], acc[eb][n], 0, 0, 0);
                    }
                }
            }
        });
    }
    __builtin_amdgcn_s_waitcnt(PAEP_VMCNT(0));              // no copy may land in this LDS once it belongs to another workgroup
    if (slices == 1) {
        int32_t* cnt_lds = (int32_t*)smem_raw;              // counted per workgroup, flushed once
        if (out.counts) {
            __syncthreads();
            for (int e = tid; e < E; e += WAVES * 64) cnt_lds[e] = 0;
            __syncthreads();
        }
        if (out.b2)
#pragma unroll
            for (int eb = 0; eb < EB; ++eb)
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const int e = eb * 16 + 4 * g + i;
                    const float b = e < E ? bf16_bits_to_f32(out.b2[(long long)layer * E + e]) : 0.0f;
#pragma unroll
                    for (int n = 0; n < NB; ++n) acc[eb][n][i] += b;
                }
        const int need = out.k + ((out.margin && out.k < E) ? 1 : 0);
        static_for<NB>([&](auto n_c) {
            constexpr int n = decltype(n_c)::value;
            const int t = t0 + first + n * 16 + l16;
            if (t < T) {                                    // the lanes of a token together
                const long long row = (long long)layer * T + t;
                f32x4 z[EB];
#pragma unroll
                for (int eb = 0; eb < EB; ++eb) z[eb] = acc[eb][n];
                if (out.logits)
#pragma unroll
                    for (int eb = 0; eb < EB; ++eb)
#pragma unroll
                        for (int i = 0; i < 4; ++i)
                            if (eb * 16 + 4 * g + i < E) out.logits[row * E + eb * 16 + 4 * g + i] = z[eb][i];
                int32_t* counts = out.counts ? cnt_lds : nullptr;
                if (need <= 2)      finish_token<2>(z, E, g, row, out, counts);
                else if (need <= 8) finish_token<8>(z, E, g, row, out, counts);
                else                finish_token<16>(z, E, g, row, out, counts);
            }
        });
        if (out.counts) {
            __syncthreads();
            for (int e = tid; e < E; e += WAVES * 64)
                if (cnt_lds[e]) atomicAdd(&out.counts[(long long)layer * E + e], cnt_lds[e]);
        }
        return;
    }
#pragma unroll
    for (int n = 0; n < NB; ++n) {
        const int tl = first + n * 16 + l16;
        if (t0 + tl >= T) continue;
        float* dst = zpart + (((long long)tile_id * slices + slice) * SH_BM + tl) * E;
#pragma unroll
        for (int eb = 0; eb < EB; ++eb) {
            const int e = eb * 16 + 4 * g;
            if (e + 3 < E) {
                *(f32x4*)(dst + e) = acc[eb][n];
            } else {
#pragma unroll
                for (int i = 0; i < 4; ++i)
                    if (e + i < E) dst[e + i] = acc[eb][n][i];
            }
        }
    }
}

// Layers go through the two kernels in batches whose h takes up to TWO_PASS_BYTES: enough workgroups that the launches'
// ends do not show, no more memory than that buys (batches of 150 / 300 / 600 / 1300 MB, ms: 48 layers 2048 x 2048, 128 experts,
// GELU, 6011 tokens 2.68 / 2.56 / 2.36 / 2.33; 256 experts, 8192 tokens 3.17 / 3.04 / 2.99 / 3.04; 4096 x 2048, 256 experts, 32768
// tokens 23.0 / 23.0 / 22.6 / 22.8).
static constexpr long long TWO_PASS_BYTES = 600ll * 1000 * 1000;
// Workgroups per token tile of the first kernel, each with its share of r: 4 of them and 8 tiles run on an XCD together and
// share their rows of W1 and x through its L2 (1 / 2 / 4 / 8 on the same three: 2.86 / 2.31 / 2.30 / 2.40, 3.61 / 3.10 / 2.98 / 3.07,
// 28.2 / 23.7 / 22.6 / 22.9 ms).
static constexpr int TWO_PASS_GROUPS = 4;
static int two_pass_groups(const PredictArgs& a)
{
    int groups = TWO_PASS_GROUPS;
    while ((a.r / Cfg256::BN) % groups != 0) groups /= 2;
    return groups;
}

// Layers per batch and slices of r in the second kernel.
struct TwoPass { int batch, slices; size_t h_bytes, z_bytes; };
static TwoPass two_pass_layout(const PredictArgs& a)
{
    const long long tiles = (a.T + SH_BM - 1) / SH_BM;
    const long long per_layer = tiles * SH_BM * a.r * 2;
    long long batch = TWO_PASS_BYTES / per_layer;
    if (batch < 1) batch = 1;
    if (batch > a.L) batch = a.L;
    batch = (a.L + (a.L + batch - 1) / batch - 1) / ((a.L + batch - 1) / batch);      // batches of even size
    TwoPass p{(int)batch, 1, (size_t)(batch * per_layer), 0};
    while (tiles * batch * p.slices < 192 && p.slices < 4) p.slices *= 2;
    // (one slice needs none: callers know this size)
    p.z_bytes = (size_t)(batch * tiles) * p.slices * SH_BM * a.E * sizeof(float);
    return p;
}

// Where the fused kernel is the slower one.  What two passes cost goes with r (h written and read again), what they save
// with d, more of it where the fused kernel has to be 128 units wide (E > 128).  Two passes / fused, prefill256.hip on either
// side, r = 512 to 4096, 320 to 1024 tiles unless said:
//   256 experts  d = 256 1.05-1.67, 512 1.00-1.31, 768 0.96-1.17 (r = 4096 1.00-1.17), 1024 0.88-0.96 (1.08 at 320 tiles, r = 4096),
//                2048 0.75-0.91, 4096 0.67-0.80; SiLU and GELU 512 0.90-1.00, 768 0.87-0.94; 192 tiles 0.61-0.98 at any d and r but
//                r = 4096 with d = 256 (1.14)
//   160 experts  d = 768 0.99-1.18, 1024 0.90-1.07, 1536 0.80-0.98, 2048 0.76-0.91
//   128 experts  d = 512 1.02-1.40, 1024 1.06-1.26, 1536 1.02-1.24, 2048 0.97-1.17 (r = 512 0.89-1.00), 2304 0.91-1.10 (1024 tiles
//                0.95-0.98), 2560 0.90-1.06, 4096 0.84-1.04; SiLU 1536 0.99-1.08, 2048 0.92-1.04, 2560 0.86-0.97; GELU 1024
//                0.95-1.06, 1536 0.93-1.00, 2048 0.89-0.99, 2560 0.84-0.95
//   64 experts   slower: with the eight-wave kernels 2048 x 2048, 32 layers x 4096 tokens 1030 / 1101 us fused / two passes
static bool two_pass_wanted(const PredictArgs& a)
{
    const long long tiles = (long long)((a.T + 255) / 256) * a.L;
    if (a.r % Cfg256::BN != 0) return false;
    if (a.E > 128) return tiles >= 128 && (tiles < 256 || a.d >= (a.E < 192 ? 1024 : 768));
    return a.E > 64 && tiles >= 384 && a.d >= (a.act == 2 ? 1536 : a.r <= 512 ? 2048 : tiles >= 1024 ? 2304 : 2560);
}

template <int EB, int ACT>
static hipError_t launch_scores_of_h(const PredictArgs& a, int tiles, int slices, const u32x4* h, float* z)
{
    auto kern = scores_of_h_kernel<EB, ACT>;
    const size_t lds = (size_t)SH_NST * EB * 16 * SH_BN * 2;
    static LdsLimit limit;
    const hipError_t err = ensure_lds_limit(limit, (const void*)kern, lds);
    if (err != hipSuccess) return err;
    hipLaunchKernelGGL(kern, dim3(tiles * a.L * slices * (8 / sh_waves<EB>())), dim3(64 * sh_waves<EB>()), lds, a.stream, a.T, a.r, a.E, tiles, slices,
                       a.w2_stride, h, (const uint16_t*)a.W2, z,
                       RowOutputs{a.k, a.prob_mode, (const uint16_t*)a.b2, a.idx, a.probs, a.logits, a.margin, a.counts});
    return hipGetLastError();
}

static hipError_t launch_two_pass(const PredictArgs& a)
{
    const TwoPass p = two_pass_layout(a);
    const int tiles = (a.T + SH_BM - 1) / SH_BM, groups = two_pass_groups(a);
    u32x4* h = (u32x4*)a.workspace;
    float* z = (float*)((char*)a.workspace + p.h_bytes);
    for (int l0 = 0; l0 < a.L; l0 += p.batch) {
        PredictArgs b = a;                                  // layers l0 .. of the call
        b.L = a.L - l0 < p.batch ? a.L - l0 : p.batch;
        b.x = (const uint16_t*)a.x + l0 * a.x_stride;
        b.W1 = (const uint16_t*)a.W1 + l0 * a.w1_stride;
        b.W2 = (const uint16_t*)a.W2 + l0 * a.w2_stride;
        if (a.b1) b.b1 = (const uint16_t*)a.b1 + (long long)l0 * a.r;
        if (a.b2) b.b2 = (const uint16_t*)a.b2 + (long long)l0 * a.E;
        const long long rows = (long long)l0 * a.T;
        b.idx = a.idx + rows * a.k;
        b.probs = a.probs + rows * a.k;
        if (a.logits) b.logits = a.logits + rows * a.E;
        if (a.margin) b.margin = a.margin + rows;
        if (a.counts) b.counts = a.counts + (long long)l0 * a.E;
        const PrefillGrid grid{tiles, tiles * b.L * groups, groups, 0, 1, 0, nullptr, 0};
        hipError_t err = launch_prefill256(b, grid, Cfg256::BM, Cfg256::BN, h);
        if (err != hipSuccess) return err;
        switch (a.act) {
        case 0: err = a.E <= 128 ? launch_scores_of_h<8, 0>(b, tiles, p.slices, h, z) : launch_scores_of_h<16, 0>(b, tiles, p.slices, h, z); break;
        case 1: err = a.E <= 128 ? launch_scores_of_h<8, 1>(b, tiles, p.slices, h, z) : launch_scores_of_h<16, 1>(b, tiles, p.slices, h, z); break;
        default: err = a.E <= 128 ? launch_scores_of_h<8, 2>(b, tiles, p.slices, h, z) : launch_scores_of_h<16, 2>(b, tiles, p.slices, h, z); break;
        }
        if (err != hipSuccess) return err;
        if (p.slices > 1) err = launch_finalize(b, z, p.slices, tiles * b.L, SH_BM, 0, tiles);
        if (err != hipSuccess) return err;
    }
    return hipSuccess;
}

// The large tiles pay off once they fill a good part of the 256 CUs; below
// that, more and smaller workgroups win.
static bool enough_large_tiles(const PredictArgs& a) { return (long long)((a.T + 255) / 256) * a.L >= 128; }

static bool tiny_wanted(const PredictArgs& a)
{
    // 64 x 64 workgroups for everything, up to two per CU; with more experts the score tiles cost what the tiles gain.
    // Against 128 x 128 tiles, us: 2048 x 2048, 64 experts, one layer, 65 tokens 31.9 / 23.4, 512 tokens 37.3 / 25.3, 1024
    // tokens 47.4 / 39.7, 2048 tokens 49.5 / 50.0; 1024 x 4096, 16 experts, 2048 tokens 46.4 / 36.1; 2048 x 2048, 128
    // experts, 512 tokens 38.8 / 31.2; 4096 x 2048, 256 experts, 512 tokens 61.4 / 69.6
    return a.E <= 128 && a.d % CfgTiny::BK == 0 && (long long)((a.T + 63) / 64) * a.L * (a.r / 64) <= 512;
}
// the fused kernel's tile: 0 small, 1 small wide, 2 big, 3 mid, 4 big wide, 5 tiny (with the workspace for its score tiles)
static int pick_cfg(const PredictArgs& a, bool roomy)
{
    const bool large = enough_large_tiles(a);
    if (roomy && !large && tiny_wanted(a)) return 5;
    if (a.E <= 64) return (large && a.r % 256 == 0) ? 2 : 0;
    if (!large) return 1;
    return (a.E <= 128 && a.r % 256 == 0) ? 4 : 3;
}

// Calls of fewer than 128 tiles of 256 tokens, up to 128 experts, whose 64 x 64 tiles would be too many: prefill256.hip's kernel in
// tiles of 128 to 256 tokens x 256 hidden units (65 to 128 experts: 128 tokens) instead of 128 x 128.  What bounds those is
// LDS: four waves of 64 x 64 read twice as many fragments a product as waves of 128 x 64, and a round of 512 workgroups is
// seldom full.  The size of the tile and the split of r are those of the least time in this model, in us, fitted to 600 timed
// combinations of shape, tile and split: rounds of 256 workgroups (the last one, partly filled, three quarters of one and more), in
// each a stage of 64 columns 0.004 a token and 0.43 on a full chip, 4 for a workgroup's ends; score tiles at 4 TB/s.
// The choice is within 3 % of the best of up to 30 for 34 shapes of 42, within 10 % for all but one of them (13 %).
// 128 x 128 tiles / here, us: 26 layers of 301 tokens, 2048 x 2048, 64 experts 129 / 77, with SiLU 149 / 91; one of 4096 62 / 39;
// 20 of 500, 4096 x 4096 547 / 335-349; 9 of 3000, d = 4096 678 / 357; 10 of 700, 128 experts 113 / 68; 48 of 200 240 / 154; 4 of
// 4000, 1024 x 64 30 / 19.5; 30 of 130, 1536 x 800 53 / 29.  At under 112 workgroups they are level (one of 1500 37.4 / 35.1, one of
// 1024 in 64 x 64 tiles 27.1 / 32.7), and so where the model says so (3 of 1200, 1024 x 4096, 16 experts 48.3 / 52.2; one of 1683,
// 2048 x 4352, 128 experts 58.1 / 63.7).
struct FewPlan { int tokens, groups; };                      // no tokens: the other tiles
static double rounds_of(long long wgs, int slots)
{
    const long long full = wgs / slots, tail = wgs % slots;
    return (double)full + (tail == 0 ? 0.0 : full == 0 ? 1.0 : 0.75 + 0.25 * (double)tail / slots);
}
static double split_us(const PredictArgs& a, long long tiles, int tokens, int groups)
{
    return groups > 1 ? 1.0 + (double)tiles * tokens * groups * a.E * 8 / 4e6 : 0.0;
}
static double time256_us(const PredictArgs& a, int tokens, int groups)
{
    const long long tiles = (long long)((a.T + tokens - 1) / tokens) * a.L, wgs = tiles * groups;
    const double stage = 0.0040 * tokens + 0.43 * (wgs < 256 ? (double)wgs / 256 : 1.0);
    const int chunks = a.r / Cfg256::BN / groups, stages = (a.d + 63) / 64;
    return rounds_of(wgs, 256) * (4 + chunks * (stages * stage + 0.5 + a.E / 64.0)) + split_us(a, tiles, tokens, groups);
}
template <class C>
static double time128_us(const PredictArgs& a)
{
    const int groups = prefill_groups<C>(a), stages = (a.d + 63) / 64;
    const long long tiles = (long long)((a.T + C::BM - 1) / C::BM) * a.L, wgs = tiles * groups;
    const double fill = wgs < 384 ? 0.75 : wgs < 512 ? (double)wgs / 512 : 1.0;
    const double stage = wgs <= 256 ? 0.75 : C::OCC == 1 ? 0.85 : 1.3 * fill;
    const double rounds = C::OCC == 1 ? rounds_of(wgs, 256) : wgs < 512 ? 1.0 : (double)wgs / 512;
    return rounds * (4 + a.r / C::BN / groups * (stages * stage + 0.3)) + split_us(a, tiles, C::BM, groups);
}
static FewPlan few_plan(const PredictArgs& a)
{
    FewPlan best{0, 1};
    if (a.E > 128 || a.r % Cfg256::BN != 0 || enough_large_tiles(a)) return best;
    double least = 0.93 * (a.E > 64 ? time128_us<CfgSmallWide>(a) : time128_us<CfgSmall>(a));
    const int chunks = a.r / Cfg256::BN;
    for (int tokens = 128; tokens <= (a.E > 64 ? 128 : 256); tokens += 32)
        for (int groups = 1; groups <= chunks; ++groups) {
            if (chunks % groups != 0 || (long long)((a.T + tokens - 1) / tokens) * a.L * groups < 112) continue;
            const double t = time256_us(a, tokens, groups);
            if (t < least) {
                least = t;
                best = FewPlan{tokens, groups};
            }
        }
    return best;
}
// Score tiles: the size of the call's scores (tokens rounded up to tiles) times the workgroups that share a tile.  Nothing bounds them
// but that: 48 layers of 32768 tokens, d = 3072, 64 experts ask for 0.8 GB (beside 9.7 GB of token rows); with less a call runs the
// layout of the least workspace.
static size_t few_bytes(const PredictArgs& a, const FewPlan& f)
{
    if (f.groups == 1) return 0;
    return (size_t)((a.T + f.tokens - 1) / f.tokens) * a.L * f.groups * f.tokens * a.E * sizeof(float);
}
static hipError_t launch_few(const PredictArgs& a, const FewPlan& f, bool tiles_first)
{
    const int tiles = (a.T + f.tokens - 1) / f.tokens;
    float* zpart = (float*)a.workspace;
    const PrefillGrid grid{tiles, tiles * a.L * f.groups, f.groups, 0, 1, 0, zpart, (int)tiles_first};
    const hipError_t err = launch_prefill256(a, grid, f.tokens, Cfg256::BN, nullptr);
    if (err != hipSuccess || f.groups == 1) return err;
    return launch_finalize(a, zpart, f.groups, tiles * a.L, f.tokens, 0, tiles);
}

// Calls of 128 to 255 tiles of 256 tokens, and with long rows up to 511: every tile's r split evenly, in tiles of 160 to 256
// tokens (65 to 128 experts: 256), where that beats the split that cfg_layout makes for them by a twentieth in this model of
// the time in us, fitted to 13 shapes of up to 30 (tile, split) each: of them its choice was the best nine times, within
// 4 % else.  (time256_us has other constants for the same kernel below 128 tiles: each is a fit to its own calls, one for both has
// not been tried.)  A stage costs 0.004 a token, 0.55, and from d = 1024 on what the token tile, which does not stay in L2, costs workgroups
// that do not share it; the last round, partly filled, half of one and more.
// cfg_layout / here, us: 16 layers of 1800 tokens, 1536 x 960, 60 experts 115 / 80; 12 of 4096, 2048 x 2048, 64 experts 366 / 316; 20 of
// 3500, d = 3072 820 / 701; 24 of 2000, 3072 x 3584 933 / 806; 48 of 600, d = 4096 549 / 482; 26 of 2600, 1024 x 4096, 16 experts,
// GELU 573 / 503; 12 of 4000, 2048 x 1024, 100 experts 227 / 197.  Beyond those tiles the rounds are many and even by themselves;
// there long rows take two workgroups to a tile, or four, up to 64 experts (16 layers of 8192 tokens,
// 1024 x 3584 833 / 730; 26 of 5120, 2048 x 3072 1561 / 1504, x 5120 in two / in four 2625 / 2334, 20 of 8000, 1024 x 5120 1311 / 1249).
static double even_us(const PredictArgs& a, int tokens, int groups)
{
    const long long tiles = (long long)((a.T + tokens - 1) / tokens) * a.L, wgs = tiles * groups, full = wgs / 256, tail = wgs % 256;
    const double rounds = (double)full + (tail == 0 ? 0.0 : full == 0 ? 1.0 : 0.5 + 0.5 * (double)tail / 256);
    const double shared = a.d > 1024 ? 0.15 * (a.d - 1024) / 1024 / groups * tokens / 256 : 0.0;
    const int chunks = a.r / Cfg256::BN / groups, stages = (a.d + 63) / 64;
    return rounds * (4 + chunks * (stages * (0.0040 * tokens + 0.55 + shared) + 0.5 + a.E / 64.0)) + split_us(a, tiles, tokens, groups);
}
static FewPlan even_plan(const PredictArgs& a)
{
    FewPlan best{0, 1};
    const long long tiles256 = (long long)((a.T + 255) / 256) * a.L;
    if (a.E > 128 || a.r % Cfg256::BN != 0 || tiles256 < 128 || (a.E <= 64 && flat_wanted(a))) return best;
    if (tiles256 >= 512 && a.E <= 64 && a.d >= 3072) {
        const int groups = a.d >= 5120 ? 4 : 2;
        return a.r / Cfg256::BN % groups == 0 && groups != prefill_groups<Cfg256>(a) ? FewPlan{256, groups} : best;
    }
    if (tiles256 >= (a.d >= 3072 ? 512 : 256)) return best;
    double least = 0.95 * even_us(a, 256, prefill_groups<Cfg256>(a));
    const int chunks = a.r / Cfg256::BN;
    for (int tokens = a.E > 64 ? 256 : 160; tokens <= 256; tokens += 32)
        for (int groups = 1; groups <= chunks && groups <= 8; ++groups) {
            if (chunks % groups != 0) continue;
            const double t = even_us(a, tokens, groups);
            if (t < least) {
                least = t;
                best = FewPlan{tokens, groups};
            }
        }
    return best;
}

template <class C>
static void cfg_plan(const PredictArgs& a, int* groups, int* cpg)
{
    const PfLayout f = cfg_layout<C>(a);
    *groups = f.main_groups;
    *cpg = a.r / C::BN / f.main_groups;
}

void prefill_plan(const PredictArgs& a, int* cfg, int* groups, int* chunks_per_group)
{
    if (two_pass_wanted(a)) {
        *cfg = 6;
        *groups = two_pass_groups(a);
        *chunks_per_group = a.r / Cfg256::BN / *groups;
        return;
    }
    *cfg = pick_cfg(a, true);
    if (*cfg == 0 || *cfg == 1) {
        const FewPlan f = few_plan(a);
        if (f.tokens > 0) {
            *cfg = 7;
            *groups = f.groups;
            *chunks_per_group = a.r / Cfg256::BN / f.groups;
            return;
        }
    }
    if (*cfg == 2 || *cfg == 4) {
        const FewPlan f = even_plan(a);
        if (f.tokens > 0) {
            *groups = f.groups;
            *chunks_per_group = a.r / Cfg256::BN / f.groups;
            return;
        }
    }
    switch (*cfg) {
    case 5: cfg_plan<CfgTiny>(a, groups, chunks_per_group); break;
    case 2: cfg_plan<Cfg256>(a, groups, chunks_per_group); break;
    case 3: cfg_plan<Cfg256x128>(a, groups, chunks_per_group); break;
    case 4: cfg_plan<Cfg256>(a, groups, chunks_per_group); break;
    case 1: cfg_plan<CfgSmallWide>(a, groups, chunks_per_group); break;
    default: cfg_plan<CfgSmall>(a, groups, chunks_per_group); break;
    }
}

static size_t fused_workspace_bytes(const PredictArgs& a, bool roomy)
{
    switch (pick_cfg(a, roomy)) {
    case 2: return cfg_workspace_bytes<Cfg256>(a);
    case 3: return cfg_workspace_bytes<Cfg256x128>(a);
    case 4: return cfg_workspace_bytes<Cfg256>(a);
    case 5: return cfg_workspace_bytes<CfgTiny>(a);
    case 1: return cfg_workspace_bytes<CfgSmallWide>(a);
    default: return cfg_workspace_bytes<CfgSmall>(a);
    }
}

// what a call cannot do without
size_t prefill_workspace_min(const PredictArgs& a) { return fused_workspace_bytes(a, false); }

static size_t two_pass_bytes(const PredictArgs& a)
{
    const TwoPass p = two_pass_layout(a);
    return p.h_bytes + p.z_bytes;
}

// The even split asks for more than the least, so that with the least a call runs the layout that this is the size of.
static size_t even_bytes(const PredictArgs& a, const FewPlan& f)
{
    const size_t more = prefill_workspace_min(a) + 16, scores = few_bytes(a, f);
    return f.tokens == 0 ? 0 : scores > more ? scores : more;
}

// what it runs fastest with; calls with less, down to the above, run without what the rest is for
size_t prefill_workspace_bytes(const PredictArgs& a)
{
    size_t need = prefill_workspace_min(a);
    size_t best = two_pass_wanted(a) ? two_pass_bytes(a) : fused_workspace_bytes(a, true);
    const int cfg = pick_cfg(a, true);
    auto ask = [&](size_t bytes) { if (bytes > best) best = bytes; };
    if (cfg == 0 || cfg == 1) ask(few_bytes(a, few_plan(a)));
    if (cfg == 2 || cfg == 4)
        for (const void* b1 : {(const void*)nullptr, (const void*)&a}) {     // a call may have one: of flat_wanted it matters whether
            PredictArgs b = a;
            b.b1 = b1;
            ask(even_bytes(b, even_plan(b)));
        }
    return best > need ? best : need;
}

// The kernel of a call in the workspace it was given: one choice for the launch and for those who ask.
enum class Route { Small, SmallWide, Few, Even, Tiny, Flat, Square, Square224, Long, Short, TwoPass };
static Route route_of(const PredictArgs& a)
{
    if (two_pass_wanted(a) && a.workspace_bytes >= two_pass_bytes(a)) return Route::TwoPass;
    const int cfg = pick_cfg(a, a.workspace_bytes >= fused_workspace_bytes(a, true));
    if (cfg == 0 || cfg == 1) {
        const FewPlan f = few_plan(a);
        if (f.tokens > 0 && a.workspace_bytes >= few_bytes(a, f)) return Route::Few;
    }
    if (cfg == 2 || cfg == 4) {
        const FewPlan f = even_plan(a);
        if (f.tokens > 0 && a.workspace_bytes >= even_bytes(a, f)) return Route::Even;
    }
    switch (cfg) {
    case 5: return Route::Tiny;
    case 4: return Route::Long;
    case 3: return Route::Short;
    case 2:
        if (flat_wanted(a)) return Route::Flat;
        return cfg_layout<Cfg256>(a).split_tiles == 0 && tiles_of_224_wanted(a) ? Route::Square224 : Route::Square;
    case 1: return Route::SmallWide;
    default: return Route::Small;
    }
}

template <class C>
static const char* name_with_order(const PredictArgs& a, const char* groups_first, const char* tiles_first)
{
    return tile_fastest<C>(a, cfg_layout<C>(a)) ? tiles_first : groups_first;
}

static const char* plan_name(const PredictArgs& a, const FewPlan& f, bool tiles_first)
{
    switch (f.tokens) {
    case 128: return tiles_first ? "prefill256_kernel 128x256 tiles first" : "prefill256_kernel 128x256";
    case 160: return tiles_first ? "prefill256_kernel 160x256 tiles first" : "prefill256_kernel 160x256";
    case 192: return tiles_first ? "prefill256_kernel 192x256 tiles first" : "prefill256_kernel 192x256";
    case 224: return tiles_first ? "prefill256_kernel 224x256 tiles first" : "prefill256_kernel 224x256";
    default:
        return tiles_first ? "prefill256_kernel 256x256 tiles first" : a.E > 64 ? "prefill256_kernel 256x256 wide" : "prefill256_kernel 256x256";
    }
}

const char* prefill_kernel_name(const PredictArgs& a)
{
    switch (route_of(a)) {
    case Route::TwoPass: return "prefill256_kernel 256x256 + scores_of_h_kernel";
    case Route::Square: return "prefill256_kernel 256x256";
    case Route::Square224: return "prefill256_kernel 224x256";
    case Route::Long: return "prefill256_kernel 256x256 wide";
    case Route::Short: return "prefill256_kernel 256x128";
    case Route::Flat: return name_with_order<CfgFlat>(a, "prefill_kernel 256x256", "prefill_kernel 256x256 tiles first");
    case Route::Tiny: return name_with_order<CfgTiny>(a, "prefill_kernel 64x64", "prefill_kernel 64x64 tiles first");
    case Route::Few: {
        const FewPlan f = few_plan(a);
        return plan_name(a, f, tile_fastest(a, f.tokens, Cfg256::BN, f.groups));
    }
    case Route::Even: return plan_name(a, even_plan(a), false);
    case Route::SmallWide:
        return name_with_order<CfgSmallWide>(a, "prefill_kernel 128x128 wide", "prefill_kernel 128x128 wide tiles first");
    default: return name_with_order<CfgSmall>(a, "prefill_kernel 128x128", "prefill_kernel 128x128 tiles first");
    }
}

hipError_t launch_predict_prefill(const PredictArgs& a)
{
    switch (route_of(a)) {
    case Route::TwoPass: return launch_two_pass(a);
    case Route::Tiny:
        return a.E <= 32 ? launch_cfg<CfgTiny, 1>(a) : a.E <= 64 ? launch_cfg<CfgTiny, 2>(a) : launch_cfg<CfgTiny, 4>(a);
    case Route::Few: {
        const FewPlan f = few_plan(a);
        return launch_few(a, f, tile_fastest(a, f.tokens, Cfg256::BN, f.groups));
    }
    case Route::Even: return launch_few(a, even_plan(a), false);
    case Route::Flat: return a.E <= 32 ? launch_cfg<CfgFlat, 1>(a) : launch_cfg<CfgFlat, 2>(a);
    case Route::Square224: return launch_tiles_of_224(a);
    case Route::Square:
    case Route::Long: return launch_cfg256<Cfg256>(a);
    case Route::Short: return launch_cfg256<Cfg256x128>(a);
    case Route::SmallWide: return a.E <= 128 ? launch_cfg<CfgSmallWide, 4>(a) : launch_cfg<CfgSmallWide, 8>(a);
    default: return a.E <= 32 ? launch_cfg<CfgSmall, 1>(a) : launch_cfg<CfgSmall, 2>(a);
    }
}

}  // namespace paep
