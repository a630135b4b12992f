// Prefill in tiles of 256 (or 224) tokens x 256 hidden units: the kernel of long calls, fused with the scores for up to 64
// experts, the first layer alone for more (predict_prefill.hip chooses).
//
// Four waves, one per SIMD, own 128 hidden units x 128 tokens of the tile each, as 8 x 8 blocks of
// v_mfma_f32_16x16x32_bf16: W1 rows are the A operand, token rows the B operand, so a lane's accumulators are
// hidden units of one token.  What bounds it is power, then the way from L2 to LDS:
//  * 16x16x32 rather than 32x32x16: registers alone, random operands, all CUs: 2.03 against 1.82 PFLOP/s in a probe (the
//    clock gives way under both).
//  * 128 x 128 per wave: 0.25 fragment reads of 1 KB per matrix instruction of 16384 products-and-sums, a third
//    fewer than 128 x 64 in eight waves.
//  * stages of 64 columns: a copy instruction fetches whole 128-byte lines; stages of 32 columns ask L2 for every line
//    twice (65536 tokens, 2048 x 4096, first layer alone: 144 M requests with the eight waves, 77 M here).
//  * one copy per six matrix instructions.  The copies of a stage in one burst hold the wave at the address unit
//    (57 % of the cycles in matrix instructions, 1100 TFLOP/s), two per six reach 1290, one 1390 (variants on one box).
// First layer alone, 3 layers of 32768 tokens, 2048 x 4096: 1387 us with eight waves of 32x32x16 and five stages of
// 32 columns, 1187 us now; 26 layers of 4096 tokens, 2048 x 2048, 829 -> 707 us (same box).
//
// The accumulators are 256 registers of the upper half of the register file, addressed by inline matrix instructions:
// the compiler's own allocation moves them about (600 moves per tile).  Waits between these instructions and vector
// instructions that the compiler would otherwise insert stand where the two meet.
#include "prefill_common.h"

namespace paep {

namespace {

constexpr int BK = 64;

// A wave's part of the tile in 16 x 16 blocks, MI of hidden units by NI of tokens; WR waves along the units, 4 / WR along
// the tokens; two stages in LDS.
//   Square: 2 x 2 waves of 128 x 128, tiles of 256 x 256: the fewest fragment reads; the first layer alone and E <= 64.
//   Square224: 128 x 112 each, tiles of 256 x 224, for calls whose last round of workgroups is a badly filled one otherwise
//           (predict_prefill.hip): a fourteenth more bytes per flop, and full rounds run at 0.97 of Square's rate (48 x 16 tiles).
//   Few:    128 units x 64 to 96 tokens each, tiles of 256 x 128 to 192, for calls whose larger tiles would leave CUs without one
//           (few_plan in predict_prefill.hip): 0.94 us for a stage of 128 tokens on a full chip, 1.07 of 160, 1.45 of 256.
//   Long:   256 units x 64 tokens each, the same tile: a wave has the chunk's whole contribution to its tokens' scores,
//           which for 65 to 128 experts fit in the registers only so.
//   Short:  128 units x 64 tokens each, tiles of 256 x 128: E up to 256, and r that is no multiple of 256.
// Square and Short keep the chunk's slice of W2 (all experts x BN units) in LDS behind the stages, copied during the chunk's
// first stage; Long, whose slice does not fit, reads its fragments of W2 from memory: 7 % of the time at 128 experts,
// 2048 x 2048.  On short rows, where a chunk's 64 KB weigh most, the kernel still beats the eight-wave one that had the slice in
// LDS: 32 layers of 4096 tokens, r = 2048, d = 64 181 -> 176 us, 256 268 -> 242, 768 515 -> 436; only d = 32, half of whose
// stage is padding, does not (170 -> 176).  (Short from memory too: 256 experts, d = 512 604 us, 178 of them for W2.)
template <int MI_, int NI_, int WR_, bool W2L_> struct Shape {
    static constexpr int MI = MI_, NI = NI_, WR = WR_, WT = 4 / WR_, BN = 16 * MI * WR, BM = 16 * NI * WT;
    static constexpr bool W2L = W2L_;
    static constexpr int STAGE = (BN + BM) * BK;                     // elements: W1 rows, then token rows
    static constexpr int JA = BN / 32, JB = BM / 32, COPIES = JA + JB;   // copy instructions per wave and stage, 8 rows each
    static_assert(MI % 2 == 0, "wave tile");
};
typedef Shape<8, 8, 2, true> Square;
typedef Shape<8, 7, 2, true> Square224;
template <int NI> using Few = Shape<8, NI, 2, true>;
typedef Shape<16, 4, 1, false> Long;
typedef Shape<8, 4, 1, true> Short;

struct Args {
    int T, d, r, E, k, prob_mode;
    PrefillGrid grid;
    long long xs, w1s, w2s;
    const uint16_t *x, *W1, *W2, *b1, *b2;
    int32_t* idx;
    float *probs, *logits, *margin;
    int32_t* counts;
    u32x4* h;
};

// What goes between the matrix instructions (slots) of a stage; two k-steps of K slots.
// A stage is multiplied while the next one lies in LDS and the one after is copied into its place as soon as all its
// fragments are in registers (slot FREE, a barrier); at slot LANDED (a barrier) the next stage's copies have landed
// and its first fragments are read.  Where few accumulators leave room for both k-steps' fragments (ROOM), that frees the
// stage earliest.  Else blocks are walked in two halves of the tokens (4 and 3 blocks of 7), so that fragments retire early and the next
// k-step's move into their registers, half a k-step before they are needed; what no longer fits behind FREE and LANDED
// goes to the front of the next stage.  Short's stages are half as long: it has room for eight fragments more (SOME).
template <class C, int EB> struct Slots {
    static constexpr int MI = C::MI, NI = C::NI, K = MI * NI, F = MI + NI, H = (NI + 1) / 2, K1 = MI * H, N = 2 * K;
    static constexpr bool ROOM = C::WR == 2 && NI >= 7 && EB <= 2, SOME = K == 32;
    static constexpr int mi(int i) { return ROOM ? i / NI : i < K1 ? i / H : (i - K1) / (NI - H); }
    static constexpr int ni(int i) { return ROOM ? i % NI : i < K1 ? i % H : H + (i - K1) % (NI - H); }
    // the q-th fragment to be read: token block 0 .. NI - 1, or NI + unit block
    static constexpr int frag(int q) { return ROOM || q < H ? q : q < H + MI ? q - H + NI : q - MI; }
    // slot of the q-th read of the second k-step's fragments, and of the next stage's first
    static constexpr int half(int q) { return q < H ? K1 + 1 + 2 * q : q < H + MI ? K1 + (NI - H == 3 ? 3 : 2) + (NI - H) * (q - H + 1) : K + 4 + 2 * (q - H - MI); }
    static constexpr int second(int q) { return ROOM || (SOME && q < 8) ? 2 * q : SOME ? 2 * q + 1 : half(q); }
    static constexpr int FREE = ROOM ? 34 : second(F - 1) + 10, LANDED = ROOM ? 94 : K + K / 2, STEP = ROOM ? 6 : SOME ? 3 : 4;
    static constexpr int next(int q) { return ROOM ? LANDED + 2 * q : SOME ? LANDED + 1 + q : K + half(q); }
    static constexpr int read_second(int m) { for (int q = 0; q < F; ++q) if (second(q) == m) return q; return -1; }
    static constexpr int read_next(int m) { for (int q = 0; q < F; ++q) if (next(q) == m) return q; return -1; }
    static constexpr int copy(int m) { return m >= FREE && (m - FREE) % STEP == 0 && (m - FREE) / STEP < C::COPIES ? (m - FREE) / STEP : -1; }
    static constexpr int late_read(int m) { return m < LANDED ? read_next(m + N) : -1; }
    static constexpr int late_copy(int m) { return m < FREE ? copy(m + N) : -1; }
    static constexpr bool LATE = FREE + (C::COPIES - 1) * STEP >= N;
    // copies that may be in flight at LANDED: this stage's own so far
    static constexpr int copies_before(int m) { int c = 0; for (int i = 0; i < m; ++i) c += copy(i) >= 0; return c; }
    // the slice of W2, in a chunk's first stage, from LANDED on: landed with the next stage's copies
    static constexpr int W2COPIES = C::W2L ? EB * 16 * C::BN * 2 / 1024 / 4 : 0, W2STEP = W2COPIES == 0 ? 1 : (N - LANDED) / W2COPIES;
    static constexpr int w2_copy(int m) { return m >= LANDED && (m - LANDED) % W2STEP == 0 && (m - LANDED) / W2STEP < W2COPIES ? (m - LANDED) / W2STEP : -1; }
    static constexpr bool each_read()                    // no two reads of a kind in one slot
    {
        for (int q = 0; q < F; ++q)
            if (read_second(second(q)) != q || read_next(next(q)) != q) return false;
        return true;
    }
    static_assert(each_read(), "one slot each");
    static_assert(next(0) >= LANDED && second(F - 1) < FREE && FREE < LANDED && (C::COPIES - 1) * STEP < N, "one stage's events");
    static_assert(next(F - 1) - N < K / 2 && FREE + (C::COPIES - 1) * STEP - N < LANDED - 16, "in time");
    static_assert(W2STEP > 0, "the slice within the stage");
};

constexpr int pitch(int eb) { return eb * 16 + 1; }      // floats per token of the score tile
// tokens whose scores, of all WR parts, are in LDS at once
template <class C, int EB> constexpr int score_rows() { return C::WR * C::BM * pitch(EB) * 4 > 150 * 1024 ? C::BM / 2 : C::BM; }

// EB: blocks of 16 experts, 0: the first layer alone.  MODE: 0 neither bias b1 nor activation, else act + 1, b1 optional.
template <class C, int EB, int MODE>
__global__ __launch_bounds__(256, 1) void prefill256_kernel(Args p)
{
    typedef Slots<C, EB> S;
    constexpr int MI = C::MI, NI = C::NI, WR = C::WR, WT = C::WT, BN = C::BN, BM = C::BM, STAGE = C::STAGE, COPIES = C::COPIES;
    constexpr int RA = BN / 4, RB = BM / 4;              // rows that a wave copies
    constexpr bool LOW1 = EB > 8;                        // acc1 in the lower half of the register file, acc2 in the upper
    extern __shared__ __attribute__((aligned(16))) unsigned char smem_raw[];
    uint16_t* stages = (uint16_t*)smem_raw;
    const int T = p.T, d = p.d, E = p.E, k = p.k, nchunks = p.r / BN;

    // Work items as in prefill_kernel: (layer, token tile, group of chunks), the group (or the tile) fastest, a contiguous range to each XCD.
    int wg = blockIdx.x;
    const bool in_tail = wg >= p.grid.main_wgs;
    {
        const int part_wgs = in_tail ? p.grid.tail_wgs : p.grid.main_wgs;
        if (in_tail) wg -= p.grid.main_wgs;
        const int per = part_wgs / 8, rem = part_wgs % 8;
        const int xcd = wg % 8, place = wg / 8;
        wg = xcd * per + (xcd < rem ? xcd : rem) + place;
    }
    const int groups = in_tail ? p.grid.tail_groups : p.grid.main_groups;
    const int cpg = nchunks / groups;
    int cg = wg % groups, tile_id = (in_tail ? p.grid.main_wgs / p.grid.main_groups : 0) + wg / groups;
    if (p.grid.tile_fastest) {
        const int column = wg / p.grid.tiles_per_layer, l = column / groups;
        cg = column - l * groups;
        tile_id = l * p.grid.tiles_per_layer + wg - column * p.grid.tiles_per_layer;
    }
    const int layer = tile_id / p.grid.tiles_per_layer;
    const int t0 = (tile_id - layer * p.grid.tiles_per_layer) * BM;
    const int n_begin = cg * cpg, n_end = n_begin + cpg;

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wr = wave / WT, wt = wave % WT;
    const int l16 = lane & 15, g = lane >> 4;

    // Copies: a wave moves RA rows of W1 and RB tokens, 8 rows (lanes / 8) of 8 chunks of 16 bytes an instruction.
    // Chunk c of a row lies in slot c ^ s(row), chosen by the lane on the global side, so that the 16 rows of a
    // fragment read touch all banks: s = bits 1-3 of a token row, bits 1, 3, 4 of a weight row (whose fragments take
    // rows 0-3, 8-11, 16-19, 24-27 of 32 or the other sixteen).  s repeats after 2 instructions of tokens, 4 of weights.
    // Rows past T lie outside the resource and arrive as zeros.
    const __amdgpu_buffer_rsrc_t rsrc_a = __builtin_amdgcn_make_buffer_rsrc(
        (void*)(p.W1 + (long long)layer * p.w1s), 0, (int)((long long)p.r * d * 2), 0x00020000);
    const __amdgpu_buffer_rsrc_t rsrc_b = __builtin_amdgcn_make_buffer_rsrc(
        (void*)(p.x + (long long)layer * p.xs + (long long)t0 * d), 0, (int)((long long)(T - t0) * d * 2), 0x00020000);
    auto swz_a = [](int row) { return ((row >> 1) & 1) | (((row >> 3) & 3) << 1); };
    auto swz_b = [](int row) { return (row >> 1) & 7; };
    uint32_t lane_a[4], lane_b[2];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const int row = wave * RA + j * 8 + (lane >> 3);
        lane_a[j] = (uint32_t)(row * d + ((lane & 7) ^ swz_a(row)) * 8) * 2u;
    }
#pragma unroll
    for (int j = 0; j < 2; ++j) {
        const int row = wave * RB + j * 8 + (lane >> 3);
        lane_b[j] = (uint32_t)(row * d + ((lane & 7) ^ swz_b(row)) * 8) * 2u;
    }
    const int NK = (d + BK - 1) / BK;
    int iss_kt = 0, iss_n = n_begin;
    auto copy_piece = [&](int stage, auto q_c) {
        constexpr int q = decltype(q_c)::value;
        uint16_t* at = stages + stage * STAGE;
        if constexpr (q < C::JB) {
            uint32_t rows = (uint32_t)d * (16u * (q & ~1));
            asm volatile("" : "+s"(rows));               // added here, not kept in a register per piece
            __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrc_b, (lptr_t)(at + BN * BK + (wave * RB + q * 8) * BK), 16,
                                                     (int)(lane_b[q & 1] + rows), iss_kt * BK * 2, 0, 0);
        } else {
            constexpr int j = q - C::JB;
            __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrc_a, (lptr_t)(at + (wave * RA + j * 8) * BK), 16, (int)lane_a[j & 3],
                                                     (iss_n * BN * d + iss_kt * BK + (j & ~3) * 8 * d) * 2, 0, 0);
        }
    };
    // The last stage of a chunk where d is an odd multiple of 32: the upper four chunks of every row are moved out of the
    // resources and arrive as zeros.  (Bit 2 of a lane's chunk is bit 2 of the lane, flipped by bit 2 of s, which for tokens
    // is bit 3 of the row.)
    auto mask_tail = [&]() {
        const uint32_t beyond = (d & 32) && iss_kt == NK - 1 ? 0x80000000u : 0u;
#pragma unroll
        for (int j = 0; j < 4; ++j)
            lane_a[j] = (lane_a[j] & 0x7FFFFFFFu) | ((((uint32_t)lane << 29) ^ ((uint32_t)(j >> 1) << 31)) & beyond);
#pragma unroll
        for (int j = 0; j < 2; ++j)
            lane_b[j] = (lane_b[j] & 0x7FFFFFFFu) | ((((uint32_t)lane << 29) ^ ((uint32_t)(wave * (RB / 8) + j) << 31)) & beyond);
    };
    // past the end the last stage is copied again, to where nobody looks any more: the count in flight stays the same
    auto copy_advance = [&]() {
        if (iss_kt + 1 < NK) ++iss_kt;
        else if (iss_n + 1 < n_end) { iss_kt = 0; ++iss_n; }
        mask_tail();
    };

    // Fragments.  Row 4 a + b of unit block mi is hidden unit 32 (mi / 2) + 8 a + 4 (mi % 2) + b: a lane then holds, of
    // one token, units 8 g .. 8 g + 7 of every 32, the B operand of the second layer (or 16 bytes of h).
    const int arow = wr * MI * 16 + 8 * (l16 >> 2) + (l16 & 3), brow = wt * NI * 16 + l16;
    const int aoff = arow * BK + ((g ^ swz_a(arow)) * 8), boff = BN * BK + brow * BK + ((g ^ swz_b(brow)) * 8);
    bf16x8 fa[2][MI], fb[2][NI];
    auto read = [&](const uint16_t* st, auto ks_c, auto f_c) {
        constexpr int ks = decltype(ks_c)::value, f = decltype(f_c)::value;
        if constexpr (f < NI) fb[ks][f] = __builtin_bit_cast(bf16x8, *(const u32x4*)(st + ((boff ^ (ks * 32)) + f * 16 * BK)));
        else fa[ks][f - NI] = __builtin_bit_cast(bf16x8, *(const u32x4*)(st + ((aoff ^ (ks * 32)) + ((f - NI) / 2 * 32 + ((f - NI) & 1) * 4) * BK)));
    };
    auto barrier = [&]() {
        asm volatile("" ::: "memory");
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
        __builtin_amdgcn_sched_barrier(0);
    };

    constexpr int EBA = EB ? EB : 1;
    f32x4 acc1[MI][NI], acc2[EBA][NI];
#pragma unroll
    for (int eb = 0; eb < EB; ++eb)
#pragma unroll
        for (int ni = 0; ni < NI; ++ni) acc2[eb][ni] = f32x4{0.f, 0.f, 0.f, 0.f};

    // W2: fragment of experts 16 eb + l16, hidden units 8 g .. 8 g + 7 of a step of 32.  Rows past E arrive as zeros.  In LDS row
    // e holds the chunk's BN units, 16 bytes c in slot c ^ (e % 16).
    const __amdgpu_buffer_rsrc_t rsrc_w2 = __builtin_amdgcn_make_buffer_rsrc(
        (void*)(p.W2 + (long long)layer * p.w2s), 0, (int)((long long)E * p.r * 2), 0x00020000);
    uint16_t* w2lds = stages + 2 * STAGE;
    auto w2_copy_piece = [&](int n, auto q_c) {
        constexpr int q = decltype(q_c)::value, CPR = BN / 8, RPI = 64 / CPR;
        int ln = lane;
        asm volatile("" : "+v"(ln));                     // formed here, once a chunk
        const int row0 = (wave * S::W2COPIES + q) * RPI, e = row0 + ln / CPR;
        __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrc_w2, (lptr_t)(w2lds + row0 * BN), 16,
                                                 (int)((uint32_t)(e * p.r + ((ln % CPR) ^ (e % 16)) * 8) * 2u), n * BN * 2, 0, 0);
    };
    constexpr int EG = EB > 8 ? 8 : EBA, GROUPS = EB / EG, STEPS = MI / 2;    // fragments requested together; steps of 32 units
    bf16x8 wf[2][EG];
    auto w2_request = [&](int n, auto i_c) {             // group i % GROUPS of step i / GROUPS
        constexpr int i = decltype(i_c)::value, P = i / GROUPS, eb0 = i % GROUPS * EG;
#pragma unroll
        for (int u = 0; u < EG; ++u) {
            if constexpr (C::W2L)
                wf[i & 1][u] = __builtin_bit_cast(bf16x8, *(const u32x4*)(w2lds + ((eb0 + u) * 16 + l16) * BN +
                                                                          (((wr * STEPS + P) * 4 + g) ^ l16) * 8));
            else
                wf[i & 1][u] = __builtin_bit_cast(bf16x8, __builtin_amdgcn_raw_buffer_load_b128(
                    rsrc_w2, (l16 * p.r + 8 * g) * 2 + (eb0 + u) * 32 * p.r, (n * BN + wr * MI * 16 + P * 32) * 2, 0));
        }
    };
    typedef u32x4 __attribute__((aligned(2))) u32x4_any;  // b1 may start in the middle of a word
    auto bias_of = [&](int n, int P) {
        if (MODE == 0 || !p.b1) return u32x4{0u, 0u, 0u, 0u};
        return (u32x4)*(const u32x4_any*)(p.b1 + (long long)layer * p.r + n * BN + wr * MI * 16 + P * 32 + 8 * g);
    };

    // Chunk n of h is complete in acc1: rounded to bf16, 32 units a step, it goes to memory or into the scores.
    auto second_layer = [&](int n) {
        asm volatile("s_nop 15" ::: "memory");            // the last matrix instructions' results, before they are read
        __builtin_amdgcn_sched_barrier(0);
        u32x4 bias = bias_of(n, 0), bnext = bias;
        if constexpr (EB > 0) w2_request(n, IC<0>{});
        static_for<STEPS>([&](auto P_c) {
            constexpr int P = decltype(P_c)::value;
            if constexpr (P + 1 < STEPS) bnext = bias_of(n, P + 1);
            bf16x8 hb[NI];
#pragma unroll
            for (int ni = 0; ni < NI; ++ni) {
                // the copies out of the accumulators belong here, not where they were last written
                if constexpr (!LOW1) asm volatile("" : "+a"(acc1[2 * P][ni]), "+a"(acc1[2 * P + 1][ni]));
                u32x4 pk;
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    float lo = acc1[2 * P + q / 2][ni][2 * (q % 2)], hi = acc1[2 * P + q / 2][ni][2 * (q % 2) + 1];
                    if constexpr (MODE > 0) {
                        lo += __uint_as_float(bias[q] << 16);
                        hi += __uint_as_float(bias[q] & 0xFFFF0000u);
                    }
                    pk[q] = pack_bf16x2(lo, hi);          // h is stored as bf16 before the activation
                    if constexpr (MODE > 1)
                        pk[q] = pack_bf16x2(act_bf16<MODE - 1>(__uint_as_float(pk[q] << 16)),
                                            act_bf16<MODE - 1>(__uint_as_float(pk[q] & 0xFFFF0000u)));
                }
                hb[ni] = __builtin_bit_cast(bf16x8, pk);
            }
            if constexpr (EB == 0) {
                // h: [block of 16 tokens][step of 32 units][lane], 16 bytes
#pragma unroll
                for (int ni = 0; ni < NI; ++ni)
                    p.h[(((long long)tile_id * (BM / 16) + wt * NI + ni) * (p.r / 32) + n * (BN / 32) + wr * STEPS + P) * 64 + lane] =
                        __builtin_bit_cast(u32x4, hb[ni]);
            } else {
                static_for<GROUPS>([&](auto gr_c) {
                    constexpr int i = P * GROUPS + decltype(gr_c)::value, eb0 = decltype(gr_c)::value * EG;
                    if constexpr (i + 1 < STEPS * GROUPS) w2_request(n, IC<i + 1>{});
                    __builtin_amdgcn_sched_barrier(0);
                    asm volatile("s_nop 1" ::: "memory"); // vector results into matrix instructions
                    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                    for (int u = 0; u < EG; ++u)
#pragma unroll
                        for (int ni = 0; ni < NI; ++ni) {
                            if constexpr (LOW1)
                                asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+a"(acc2[eb0 + u][ni]) : "v"(wf[i & 1][u]), "v"(hb[ni]));
                            else
                                asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+v"(acc2[eb0 + u][ni]) : "v"(wf[i & 1][u]), "v"(hb[ni]));
                        }
                    __builtin_amdgcn_sched_barrier(0);
                });
            }
            bias = bnext;
            __builtin_amdgcn_sched_barrier(0);
        });
    };

    mask_tail();
    static_for<COPIES>([&](auto q) { copy_piece(0, q); });
    copy_advance();
    static_for<COPIES>([&](auto q) { copy_piece(1, q); });
    if (!S::LATE) copy_advance();                         // late copies: the first stage repeats the last of these
    __builtin_amdgcn_s_waitcnt(PAEP_VMCNT(COPIES));
    barrier();
    static_for<S::F>([&](auto f) { read(stages, IC<0>{}, f); });

    int stage = 0;
    // FIRST: the first stage of a chunk, whose first products take no earlier sum
    auto multiply_stage = [&](auto first_c, int n) {
        constexpr bool FIRST = decltype(first_c)::value;
        const uint16_t* st = stages + stage * STAGE;
        const uint16_t* st_next = stages + (stage ^ 1) * STAGE;
        static_for<S::N>([&](auto m_c) {
            constexpr int m = decltype(m_c)::value, ks = m / S::K, mi = S::mi(m % S::K), ni = S::ni(m % S::K);
            // this stage's fragments are in registers; the next stage's copies have landed; everyone's
            if constexpr (m == S::FREE) __builtin_amdgcn_s_waitcnt(PAEP_LGKM0);
            if constexpr (m == S::LANDED) __builtin_amdgcn_s_waitcnt(PAEP_VMCNT(S::copies_before(S::LANDED)));
            if constexpr (m == S::FREE || m == S::LANDED) barrier();
            if constexpr (LOW1) {
                if constexpr (FIRST && ks == 0)
                    asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, 0" : "=v"(acc1[mi][ni]) : "v"(fa[ks][mi]), "v"(fb[ks][ni]));
                else
                    asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+v"(acc1[mi][ni]) : "v"(fa[ks][mi]), "v"(fb[ks][ni]));
            } else {
                if constexpr (FIRST && ks == 0)
                    asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, 0" : "=a"(acc1[mi][ni]) : "v"(fa[ks][mi]), "v"(fb[ks][ni]));
                else
                    asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+a"(acc1[mi][ni]) : "v"(fa[ks][mi]), "v"(fb[ks][ni]));
            }
            __builtin_amdgcn_sched_barrier(0);
            if constexpr (S::read_second(m) >= 0) read(st, IC<1>{}, IC<S::frag(S::read_second(m))>{});
            if constexpr (S::read_next(m) >= 0) read(st_next, IC<0>{}, IC<S::frag(S::read_next(m))>{});
            if constexpr (S::late_read(m) >= 0) read(st, IC<0>{}, IC<S::frag(S::late_read(m))>{});
            if constexpr (S::copy(m) >= 0) copy_piece(stage, IC<S::copy(m)>{});
            if constexpr (FIRST && S::w2_copy(m) >= 0) w2_copy_piece(n, IC<S::w2_copy(m)>{});
            if constexpr (S::late_copy(m) >= 0) {
                copy_piece(stage ^ 1, IC<S::late_copy(m)>{});
                if constexpr (S::late_copy(m) == COPIES - 1) copy_advance();
            }
            __builtin_amdgcn_sched_barrier(0);
        });
        if (!S::LATE) copy_advance();
        stage ^= 1;
    };
    for (int n = n_begin; n < n_end; ++n) {
        multiply_stage(std::true_type{}, n);
        for (int kt = 1; kt < NK; ++kt) multiply_stage(std::false_type{}, n);
        if (C::W2L && EB > 0 && NK == 1) {                // no next stage's wait before the slice is read
            __builtin_amdgcn_s_waitcnt(PAEP_VMCNT(0));
            barrier();
        }
        second_layer(n);
        // the next stage's first fragments again: no register carries them over the second layer
        static_for<S::F>([&](auto f) { read(stages + stage * STAGE, IC<0>{}, f); });
    }
    __builtin_amdgcn_s_waitcnt(PAEP_VMCNT(0));            // the copies of the pipeline's end land in this workgroup's LDS
    if constexpr (EB > 0) {
        asm volatile("s_nop 15" ::: "memory");

        // Scores: acc2[eb][ni][i] is expert 16 eb + 4 g + i of token (wt * NI + ni) * 16 + l16, over this wave's units.  Waves
        // that share tokens meet in LDS, wr = 0 first.
        constexpr int ZP = pitch(EB), ROWS = score_rows<C, EB>(), G = 256 / ROWS, PART = ROWS * ZP;
        float* zs = (float*)smem_raw;
        int32_t* cnt_lds = (int32_t*)(zs + WR * PART);
        const bool split = groups > 1;
        float* zmine = split ? p.grid.zpart + ((long long)(tile_id - p.grid.split_tile0) * groups + cg) * BM * E : nullptr;
        __syncthreads();
        if (p.counts)
            for (int e = tid; e < E; e += 256) cnt_lds[e] = 0;
        const bool biased = p.b2 && !split;
#pragma unroll 1
        for (int r0 = 0; r0 < BM; r0 += ROWS) {
            if (wt * NI * 16 / ROWS == r0 / ROWS) {
#pragma unroll
                for (int eb = 0; eb < EB; ++eb) {
                    f32x4 bias{0.f, 0.f, 0.f, 0.f};
                    if (biased && wr == 0)
#pragma unroll
                        for (int i = 0; i < 4; ++i)
                            if (eb * 16 + 4 * g + i < E) bias[i] = bf16_bits_to_f32(p.b2[(long long)layer * E + eb * 16 + 4 * g + i]);
#pragma unroll
                    for (int ni = 0; ni < NI; ++ni)
#pragma unroll
                        for (int i = 0; i < 4; ++i)
                            zs[wr * PART + ((wt * NI + ni) * 16 + l16 - r0) * ZP + eb * 16 + 4 * g + i] = acc2[eb][ni][i] + bias[i];
                }
            }
            __syncthreads();
            auto score = [&](int tl, int e) {
                float v = zs[tl * ZP + e];
                if constexpr (WR > 1) v += zs[PART + tl * ZP + e];
                return v;
            };
            // One division per pass, not one per score: with them the four waves took twice as long here as the eight of the
            // kernel before, which cost split calls of short rows up to 21 % (16 layers of 3000 tokens, 2048 x 160).
            if (split || p.logits) {
                float* out = split ? zmine + (long long)r0 * E : p.logits + ((long long)layer * T + t0 + r0) * E;
                const int left = T - t0 - r0, n = (left < ROWS ? left : ROWS) * E, rows = 256 / E, rest = 256 - rows * E;
                int tl = tid / E, e = tid - tl * E;
#pragma unroll 4
                for (int i = tid; i < n; i += 256) {
                    out[i] = score(tl, e);
                    tl += rows;
                    e += rest;
                    if (e >= E) { e -= E; ++tl; }
                }
            }
            const int tl = tid / G;
            if (!split && tl < ROWS && t0 + r0 + tl < T) {             // the lanes of a row together
                const long long row = (long long)layer * T + t0 + r0 + tl;
                const EpilogueOut eo{p.prob_mode, p.margin ? p.margin + row : nullptr, p.counts ? cnt_lds : nullptr};
                row_softmax_topk_upto16<G, false, Sums::Chains>([&](int e) { return score(tl, e); }, E, k, tid % G, p.idx + row * k,
                                                  p.probs + row * k, eo);
            }
            __syncthreads();
        }
        if (p.counts && !split)                           // counted per workgroup, flushed once
            for (int e = tid; e < E; e += 256)
                if (cnt_lds[e]) atomicAdd(&p.counts[(long long)layer * E + e], cnt_lds[e]);
    }
}

template <class C, int EB, int MODE>
hipError_t launch_mode(const Args& p, hipStream_t stream)
{
    auto kern = prefill256_kernel<C, EB, MODE>;
    const size_t stages = 2 * sizeof(uint16_t) * C::STAGE + (C::W2L ? sizeof(uint16_t) * EB * 16 * C::BN : 0);
    const size_t scores = sizeof(float) * C::WR * score_rows<C, EB>() * pitch(EB) + sizeof(int32_t) * p.E;
    const size_t lds = EB == 0 || scores < stages ? stages : scores;
    static LdsLimit limit;
    const hipError_t err = ensure_lds_limit(limit, (const void*)kern, lds);
    if (err != hipSuccess) return err;
    hipLaunchKernelGGL(kern, dim3(p.grid.main_wgs + p.grid.tail_wgs), dim3(256), lds, stream, p);
    return hipGetLastError();
}

template <class C, int EB>
hipError_t launch_experts(const Args& p, int act, hipStream_t stream)
{
    switch (act) {
    case 0: return p.b1 ? launch_mode<C, EB, 1>(p, stream) : launch_mode<C, EB, 0>(p, stream);
    case 1: return launch_mode<C, EB, 2>(p, stream);
    default: return launch_mode<C, EB, 3>(p, stream);
    }
}

}  // namespace

hipError_t launch_prefill256(const PredictArgs& a, const PrefillGrid& grid, int tokens, int units, u32x4* h)
{
    const Args p{a.T, a.d, a.r, a.E, a.k, a.prob_mode, grid, a.x_stride, a.w1_stride, a.w2_stride,
                 (const uint16_t*)a.x, (const uint16_t*)a.W1, (const uint16_t*)a.W2, (const uint16_t*)a.b1,
                 (const uint16_t*)a.b2, a.idx, a.probs, a.logits, a.margin, a.counts, h};
    if (h) return a.b1 ? launch_mode<Square, 0, 1>(p, a.stream) : launch_mode<Square, 0, 0>(p, a.stream);
    if (tokens == 128 && a.E > 64) return launch_experts<Few<4>, 8>(p, a.act, a.stream);
    if (tokens == 128)
        return a.E <= 32 ? launch_experts<Few<4>, 2>(p, a.act, a.stream) : launch_experts<Few<4>, 4>(p, a.act, a.stream);
    if (tokens == 160)
        return a.E <= 32 ? launch_experts<Few<5>, 2>(p, a.act, a.stream) : launch_experts<Few<5>, 4>(p, a.act, a.stream);
    if (tokens == 192) return launch_experts<Few<6>, 4>(p, a.act, a.stream);
    if (tokens == 224)
        return a.E <= 32 ? launch_experts<Square224, 2>(p, a.act, a.stream) : launch_experts<Square224, 4>(p, a.act, a.stream);
    if (units == 256)
        return a.E <= 32 ? launch_experts<Square, 2>(p, a.act, a.stream)
             : a.E <= 64 ? launch_experts<Square, 4>(p, a.act, a.stream) : launch_experts<Long, 8>(p, a.act, a.stream);
    return a.E <= 128 ? launch_experts<Short, 8>(p, a.act, a.stream) : launch_experts<Short, 16>(p, a.act, a.stream);
}

}  // namespace paep
