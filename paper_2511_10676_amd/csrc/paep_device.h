// Device-side building blocks shared by the predict kernels (gfx950, wave64).
//
//  * bf16 <-> fp32 conversions on raw bit patterns,
//  * order-preserving packing of (score, expert id) into one 64-bit key, so
//    that one compare implements "higher score first, equal scores by
//    lower expert id" (the tie rule of the C header),
//  * a sorted top-K list kept in registers, filled by streaming over a row of
//    scores and merged across the lanes that share a row with wave shuffles,
//  * the softmax (eq. 1 of the paper) gathered at the selected experts, or one
//    of the other two confidence scores (softmax over the selected experts
//    only; sigmoid, the function the predictor is trained through, section 4.4),
//  * optionally, the margin between the last selected score and the best one
//    left out (the confidence signal of the paper's closing section),
//  * optionally, one integer atomic per selection into activation counters
//    (the histogram that grouping would compute, fused into the epilogue); the
//    counters may live in LDS (one flush per workgroup) or in global memory.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace paep {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(4))) __bf16 bf16x4;
typedef __attribute__((ext_vector_type(4))) short short4v;
typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((ext_vector_type(16))) float f32x16;
typedef __attribute__((ext_vector_type(4))) uint32_t u32x4;
typedef __attribute__((ext_vector_type(2))) uint32_t u32x2;

__device__ __forceinline__ float bf16_bits_to_f32(uint16_t b) { return __uint_as_float(((uint32_t)b) << 16); }

// round-to-nearest-even, by the hardware conversion (v_cvt_pk_bf16_f32)
__device__ __forceinline__ uint16_t f32_to_bf16_bits(float f)
{
    return __builtin_bit_cast(uint16_t, (__bf16)f);
}

__device__ __forceinline__ float round_to_bf16(float f) { return bf16_bits_to_f32(f32_to_bf16_bits(f)); }

// two floats -> packed pair of bf16 (lo in bits 0..15)
__device__ __forceinline__ uint32_t pack_bf16x2(float lo, float hi)
{
    typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
    typedef float f32x2_t __attribute__((ext_vector_type(2)));
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(f32x2_t{lo, hi}, bf16x2_t));
}

__device__ __forceinline__ float apply_act(float v, int act)
{
    if (act == 1) return v / (1.0f + __expf(-v));                        // SiLU
    if (act == 2) return 0.5f * v * (1.0f + erff(v * 0.70710678118654752f));  // exact GELU
    return v;
}

// The same two functions for a v on the bf16 grid whose result is rounded to bf16 again, one instruction stream per
// activation (ACT: 0 identity, 1 SiLU, 2 GELU).  The general forms above spend some 50 vector instructions on a hidden
// unit (erff: both of its ranges; the division: its scaling and correction steps), more than the matrix work of that
// unit leaves idle (26 layers 2048 x 2048, 301 tokens with SiLU: 174 -> 165 us with these and one kernel per activation).
//   SiLU  v / (1 + e^-v) by the hardware reciprocal; 1 + e^-v is scaled by 2^-32 so that neither it nor its
//         reciprocal leaves the normal range before the result does.
//   GELU  v Phi(v), with Phi(-u) = e^(-u^2 / 2) t P(t), t = 1 / (1 + 0.21 u), u = |v| (the form of Abramowitz and
//         Stegun 26.2.17): P of degree 8 fitted to e^(u^2 / 2) Phi(-u) / t over 0 <= u <= 14, relative error 1.6e-8.
// Over the bf16 values of magnitude 2^-60 to 64 whose result is a normal number both give it correctly rounded, or the
// other neighbour within 1e-6 of a rounding boundary; 0.5 v (1 + erff) does not below v = -4.4, where 1 + erff cancels.
// Below v = -13.2, where GELU's results are subnormal, the hardware exponential flushes them to 0; SiLU is 0 below
// v = -88, where e^-v overflows.
template <int ACT> __device__ __forceinline__ float act_bf16(float v)
{
    if constexpr (ACT == 1) {
        const float e = __builtin_amdgcn_exp2f(v * -1.44269504088896341f);
        return v * (__builtin_amdgcn_rcpf(fmaf(e, 0x1p-32f, 0x1p-32f)) * 0x1p-32f);
    } else if constexpr (ACT == 2) {
        const float u = fabsf(v);
        const float t = __builtin_amdgcn_rcpf(fmaf(u, 0.21f, 1.0f));
        float p = -0.0716562569141388f;
        p = fmaf(p, t, 0.28358834981918335f);
        p = fmaf(p, t, -0.330253005027771f);
        p = fmaf(p, t, 0.3494006395339966f);
        p = fmaf(p, t, -0.09392499178647995f);
        p = fmaf(p, t, 0.12487264722585678f);
        p = fmaf(p, t, 0.06919218599796295f);
        p = fmaf(p, t, 0.08506885915994644f);
        p = fmaf(p, t, 0.08371157944202423f);
        const float tail = (p * t) * __builtin_amdgcn_exp2f(u * u * -0.72134752044448170f);
        return v * (v < 0.0f ? tail : 1.0f - tail);
    } else {
        return v;
    }
}
__device__ __forceinline__ float apply_act_bf16(float v, int act)
{
    return act == 1 ? act_bf16<1>(v) : act == 2 ? act_bf16<2>(v) : v;
}

// ---------------------------------------------------------------------------
// (score, expert) -> 64-bit key.  Larger key = better candidate.
// ---------------------------------------------------------------------------
__device__ __forceinline__ uint32_t orderable(float f)
{
    f += 0.0f;                                   // -0 -> +0 so the two zeros tie
    uint32_t u = __float_as_uint(f);
    if (f != f) return 0u;                       // NaN orders below -inf
    return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}

__device__ __forceinline__ float unorderable(uint32_t o)
{
    uint32_t u = (o & 0x80000000u) ? (o & 0x7FFFFFFFu) : ~o;
    return __uint_as_float(u);
}

// The value a score takes part with: NaN for NaN, +0 for both zeros.
__device__ __forceinline__ float ordered_value(float f) { return unorderable(orderable(f)); }

// A key is a double: the ordered score above 30 bits that fall with the expert id, moved to where every pattern is a
// positive normal number, so that the larger and the smaller of two keys are one full-rate instruction each (an unsigned
// 64-bit compare and four selects otherwise).  NO_KEY is below every key.
typedef double skey;
static constexpr skey NO_KEY = 0.0;
__device__ __forceinline__ skey make_key(float score, int e)
{
    const uint32_t o = orderable(score);
    return __hiloint2double((int)((o >> 2) + 0x20000000u), (int)((o << 30) | (0x3FFFFFFFu - (uint32_t)e)));
}
__device__ __forceinline__ int key_expert(skey key) { return (int)(0x3FFFFFFFu - ((uint32_t)__double2loint(key) & 0x3FFFFFFFu)); }
__device__ __forceinline__ float key_score(skey key)
{
    return unorderable((((uint32_t)__double2hiint(key) - 0x20000000u) << 2) | ((uint32_t)__double2loint(key) >> 30));
}
// (fmax and fmin would first make quiet NaNs of their operands' signalling ones, of which there are none)
__device__ __forceinline__ skey key_max(skey a, skey b)
{
    skey r;
    asm("v_max_f64 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
    return r;
}
__device__ __forceinline__ skey key_min(skey a, skey b)
{
    skey r;
    asm("v_min_f64 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
    return r;
}

// Sorted (descending) list of the KMAX best keys seen; NO_KEY marks an empty slot.
template <int KMAX>
struct TopList {
    skey key[KMAX];

    static __device__ __forceinline__ void exchange(skey& a, skey& b)
    {
        const skey hi = key_max(a, b);
        b = key_min(a, b);
        a = hi;
    }
    __device__ __forceinline__ void clear()
    {
#pragma unroll
        for (int j = 0; j < KMAX; ++j) key[j] = NO_KEY;
    }
    __device__ __forceinline__ void insert(skey c)
    {
#pragma unroll
        for (int j = 0; j < KMAX; ++j) exchange(key[j], c);
    }
    // The KMAX best of this list and another one (both sorted): max of the j-th best here and
    // the j-th worst there is a bitonic sequence of the KMAX best, which log2(KMAX) rounds of compare-exchanges
    // sort -- 8 + 12 exchanges for 8 keys where inserting one key after the other takes 64.
    __device__ __forceinline__ void merge(const skey (&other)[KMAX])
    {
        static_assert((KMAX & (KMAX - 1)) == 0, "a power of two");
#pragma unroll
        for (int j = 0; j < KMAX; ++j) key[j] = key_max(other[KMAX - 1 - j], key[j]);
#pragma unroll
        for (int st = KMAX / 2; st > 0; st >>= 1)
#pragma unroll
            for (int j = 0; j < KMAX; ++j)
                if ((j & st) == 0) exchange(key[j], key[j + st]);
    }
    // descending order of KMAX keys by Batcher's odd-even merge sort: 19 compare-exchanges for 8 keys, 63 for 16
    static __device__ __forceinline__ void sort(skey (&k)[KMAX])
    {
#pragma unroll
        for (int p = 1; p < KMAX; p <<= 1)
#pragma unroll
            for (int q = p; q >= 1; q >>= 1)
#pragma unroll
                for (int j = q % p; j + q < KMAX; j += 2 * q)
#pragma unroll
                    for (int i = 0; i < q; ++i)
                        if (i + j + q < KMAX && (i + j) / (2 * p) == (i + j + q) / (2 * p)) exchange(k[i + j], k[i + j + q]);
    }
    // KMAX more keys (NO_KEY: none): sorted by themselves and merged, 39 compare-exchanges where inserting 8 takes 64
    __device__ __forceinline__ void add(skey (&more)[KMAX], bool first)
    {
        sort(more);
        if (first) {
#pragma unroll
            for (int j = 0; j < KMAX; ++j) key[j] = more[j];
        } else {
            merge(more);
        }
    }
    // every lane of a group of G, STRIDE lanes apart, ends with the group's list
    template <int G, int STRIDE = 1> __device__ __forceinline__ void merge_group()
    {
#pragma unroll
        for (int mask = STRIDE; mask < G * STRIDE; mask <<= 1) {
            skey other[KMAX];
#pragma unroll
            for (int j = 0; j < KMAX; ++j) other[j] = __shfl_xor(key[j], mask, 64);
            merge(other);
        }
    }
};

// What the epilogue writes besides idx.
//   prob_mode 0: probs[j] = softmax over all E scores, gathered at the selection (eq. 1)
//             1: probs[j] = softmax over the k selected scores only
//             2: probs[j] = sigmoid of the selected score
//   margin:   nullable; margin[row] = score of the last selected expert minus the best
//             score left out (+inf when k = E)
//   counts:   nullable; counts[e] += 1 per selection of expert e (LDS or global)
struct EpilogueOut {
    int prob_mode;
    float* margin_row;
    int32_t* counts_row;
};

__device__ __forceinline__ float sigmoidf_(float v) { return 1.0f / (1.0f + __expf(-v)); }

// How a row's lanes sum their exponentials.
//   Chain   one after the other
//   Chains  in 4 or 8 chains that are then added in pairs: where a row has one lane, a single chain of its E terms rounds more than
//           the lanes of finalize_rows_kernel, 16 terms each (64 experts, the first probability against float64, rms: 1.2e-7, in
//           chains 5.2e-8, there 5.7e-8).  prefill_kernel keeps the one: its loops, which split calls run alone, are compiled slower
//           beside the others (9 layers of 285 tokens, 896 x 1024, 76 experts 26.3 -> 28.2 us)
//   Fine    ... and of the selected scores in pairs, and quotients instead of products with a reciprocal, as wave_softmax_topk
//           rounds them, for rows of fp32 calls
enum class Sums { Chain, Chains, Fine };

template <int N> __device__ __forceinline__ float sum_in_pairs(float (&t)[N])
{
#pragma unroll
    for (int step = 1; step < N; step <<= 1)
#pragma unroll
        for (int j = 0; j + step < N; j += 2 * step) t[j] += t[j + step];
    return t[0];
}

// The outputs of one row from its merged list `top`, by the G lanes that share it: lane g writes outputs
// j = g, g + G, ... < k.  KMAX >= k, and >= k + 1 when the margin is wanted and k < E.  exp_sum(m) is this lane's
// share of sum(exp(z - m)) over the row's scores.  STRIDE: how far apart the row's lanes are.
template <int KMAX, int G, int STRIDE = 1, Sums SUMS = Sums::Chain, class F>
__device__ __forceinline__ void write_selection(const TopList<KMAX>& top, int E, int k, int g, int32_t* idx_row,
                                                float* probs_row, const EpilogueOut& o, F&& exp_sum)
{
    const float m = key_score(top.key[0]);       // row maximum (NaNs order last)
    float s = 0.0f;
    if (o.prob_mode == 0) {
        s = exp_sum(m);
#pragma unroll
        for (int mask = STRIDE; mask < G * STRIDE; mask <<= 1) s += __shfl_xor(s, mask, 64);
    } else if (o.prob_mode == 1) {               // every lane holds the whole list: same sum, same order
        if constexpr (SUMS == Sums::Fine) {
            float t[KMAX];
#pragma unroll
            for (int j = 0; j < KMAX; ++j) t[j] = j < k ? __expf(key_score(top.key[j]) - m) : 0.0f;
            s = sum_in_pairs(t);
        } else {
#pragma unroll
            for (int j = 0; j < KMAX; ++j)
                if (j < k) s += __expf(key_score(top.key[j]) - m);
        }
    }
    const float inv = 1.0f / s;
#pragma unroll
    for (int j = 0; j < KMAX; ++j) {
        if (j < k && (j % G) == g) {
            const float sc = key_score(top.key[j]);
            idx_row[j] = key_expert(top.key[j]);
            float q = __expf(sc - m) * inv;
            if constexpr (SUMS == Sums::Fine) q = fmaf(fmaf(-q, s, __expf(sc - m)), inv, q);      // a division takes 3 % longer (4 layers of 1024 tokens, 256 x 64, 16 experts, k = 12 25.9 us, 25.3 here)
            probs_row[j] = (o.prob_mode == 2) ? sigmoidf_(sc) : q;
            if (o.counts_row) atomicAdd(&o.counts_row[key_expert(top.key[j])], 1);   // activation counts (exact: integers)
        }
    }
    if (o.margin_row && g == 0) {
        float mg = __builtin_inff();
#pragma unroll
        for (int j = 1; j < KMAX; ++j)
            if (j == k && k < E) mg = key_score(top.key[j - 1]) - key_score(top.key[j]);
        *o.margin_row = mg;
    }
}

// Softmax + top-k of one row of E scores in LDS, z(e) being the e-th, computed by G
// consecutive lanes (G a power of two, the group aligned to G).  Lane g of
// the group scans e = g, g+G, ...; the per-lane lists are merged with
// xor-shuffles so that every lane ends with the row's list.
// SORTED: KMAX scores at a time, sorted and merged, the next ones requested meanwhile; else one inserted after the
// other (fewer registers).  Scores are read in batches: one by one, a lane waits for LDS E / G times.
template <int KMAX, int G, bool SORTED, Sums SUMS = Sums::Chain, class Z>
__device__ __forceinline__ void row_softmax_topk(Z&& z, int E, int k, int g,
                                                 int32_t* idx_row, float* probs_row, const EpilogueOut& o)
{
    TopList<KMAX> top;
    top.clear();
    if constexpr (!SORTED) {
        constexpr int NB = KMAX <= 8 ? 8 : 4;
#pragma unroll 1
        for (int e0 = g; e0 < E; e0 += G * NB) {
            float v[NB];
#pragma unroll
            for (int j = 0; j < NB; ++j) v[j] = e0 + G * j < E ? z(e0 + G * j) : 0.0f;
#pragma unroll
            for (int j = 0; j < NB; ++j)
                if (e0 + G * j < E) top.insert(make_key(v[j], e0 + G * j));
        }
    } else {
        float v[KMAX];
        auto request = [&](int e0) {
#pragma unroll
            for (int j = 0; j < KMAX; ++j) v[j] = e0 + G * j < E ? z(e0 + G * j) : 0.0f;
        };
        request(g);
#pragma unroll 1
        for (int e0 = g; e0 < E; e0 += G * KMAX) {
            skey more[KMAX];
#pragma unroll
            for (int j = 0; j < KMAX; ++j) more[j] = e0 + G * j < E ? make_key(v[j], e0 + G * j) : NO_KEY;
            request(e0 + G * KMAX);
            top.add(more, false);
        }
    }
    top.template merge_group<G>();
    write_selection<KMAX, G, 1, SUMS>(top, E, k, g, idx_row, probs_row, o, [&](float m) {
        constexpr int NB = SORTED || KMAX <= 8 ? 8 : 4, CHAINS = SUMS == Sums::Chain ? 1 : NB;
        float s[CHAINS] = {};
#pragma unroll 1
        for (int e0 = g; e0 < E; e0 += G * NB) {
            float v[NB];
#pragma unroll
            for (int j = 0; j < NB; ++j) v[j] = e0 + G * j < E ? z(e0 + G * j) : 0.0f;
#pragma unroll
            for (int j = 0; j < NB; ++j)
                if (e0 + G * j < E && v[j] == v[j]) s[j % CHAINS] += __expf(v[j] - m);
        }
        return sum_in_pairs(s);
    });
}

// Softmax + top-k of one row held in registers by a whole wave: lane l owns
// z[v] = score of expert l + 64*v (v < NV).  k rounds (one more when the margin
// is wanted) of "wave-wide maximum of the keys still in play"; the lane that
// owns the winner retires it.  Lane j keeps the j-th winner and writes output
// j.  All reductions are xor butterflies, so the result does not depend on
// scheduling.
template <int NV>
__device__ __forceinline__ void wave_softmax_topk(const float (&z)[NV], int E, int k, int lane,
                                                  int32_t* idx_row, float* probs_row, const EpilogueOut& o)
{
    skey key[NV];
#pragma unroll
    for (int v = 0; v < NV; ++v) {
        const int e = lane + 64 * v;
        key[v] = (e < E) ? make_key(z[v], e) : NO_KEY;
    }
    skey mine = NO_KEY;
    const int rounds = k + ((o.margin_row && k < E) ? 1 : 0);
    for (int j = 0; j < rounds; ++j) {
        skey best = key[0];
#pragma unroll
        for (int v = 1; v < NV; ++v) best = key_max(key[v], best);
#pragma unroll
        for (int mask = 1; mask < 64; mask <<= 1) best = key_max(__shfl_xor(best, mask, 64), best);
#pragma unroll
        for (int v = 0; v < NV; ++v) key[v] = (key[v] == best) ? NO_KEY : key[v];
        if (lane == j) mine = best;
    }
    const float m = key_score(__shfl(mine, 0, 64));     // row maximum
    const float sc = key_score(mine);
    float s = 0.0f;
    if (o.prob_mode == 0) {
#pragma unroll
        for (int v = 0; v < NV; ++v) {
            const int e = lane + 64 * v;
            if (e < E && z[v] == z[v]) s += __expf(z[v] - m);
        }
    } else if (o.prob_mode == 1) {
        if (lane < k) s = __expf(sc - m);
    }
    if (o.prob_mode != 2) {
#pragma unroll
        for (int mask = 1; mask < 64; mask <<= 1) s += __shfl_xor(s, mask, 64);
    }
    if (o.margin_row) {
        const float last = key_score(__shfl(mine, k - 1, 64));
        const float next = key_score(__shfl(mine, k < 64 ? k : 63, 64));
        if (lane == 0) *o.margin_row = (k < E) ? last - next : __builtin_inff();
    }
    if (lane < k) {
        idx_row[lane] = key_expert(mine);
        probs_row[lane] = (o.prob_mode == 2) ? sigmoidf_(sc) : __expf(sc - m) / s;
        if (o.counts_row) atomicAdd(&o.counts_row[key_expert(mine)], 1);
    }
}

// The same outputs for a row of at most 64 scores, one per lane, by rank counting:
// every lane learns how many of the row's keys beat its own by walking the 64 lanes' keys
// through scalar registers (v_readlane: no LDS round trip, no dependent chain of shuffles).
// Keys are distinct (the expert id is part of the key), so the ranks are a permutation and the
// lane whose key has rank j < k writes output j.  Selection and order are exactly those of
// wave_softmax_topk; the softmax normaliser is the same butterfly sum.
__device__ __forceinline__ void wave_softmax_topk_rank(float z, int E, int k, int lane,
                                                       int32_t* idx_row, float* probs_row, const EpilogueOut& o)
{
    const skey key = (lane < E) ? make_key(z, lane) : NO_KEY;
    const int khi = __double2hiint(key), klo = __double2loint(key);
    int rank = 0;
    for (int j = 0; j < 64; ++j)                               // uniform: lane j's key, broadcast
        rank += __hiloint2double(__builtin_amdgcn_readlane(khi, j), __builtin_amdgcn_readlane(klo, j)) > key ? 1 : 0;
    // score of the key with a given rank, for every lane (rank < number of valid keys)
    auto score_of_rank = [&](int want) {
        float found = 0.0f;
        const unsigned long long who = __ballot(rank == want && lane < E);
        if (who) found = __uint_as_float((uint32_t)__builtin_amdgcn_readlane(
                     (int)__float_as_uint(z), (int)__builtin_ctzll(who)));
        return found + 0.0f;
    };
    // row maximum as the other routine takes it: the score of the best key (NaNs order last, -0 reads as +0)
    const float m = ordered_value(score_of_rank(0));
    const float sc = ordered_value(z);
    float s = 0.0f;
    if (o.prob_mode == 0) {
        if (lane < E && z == z) s = __expf(z - m);
    } else if (o.prob_mode == 1) {
        if (lane < E && rank < k) s = __expf(sc - m);
    }
    if (o.prob_mode != 2) {
#pragma unroll
        for (int mask = 1; mask < 64; mask <<= 1) s += __shfl_xor(s, mask, 64);
    }
    if (o.margin_row) {
        float mg = __builtin_inff();
        if (k < E) mg = ordered_value(score_of_rank(k - 1)) - ordered_value(score_of_rank(k));
        if (lane == 0) *o.margin_row = mg;
    }
    if (lane < E && rank < k) {
        idx_row[rank] = lane;
        probs_row[rank] = (o.prob_mode == 2) ? sigmoidf_(sc) : __expf(sc - m) / s;
        if (o.counts_row) atomicAdd(&o.counts_row[lane], 1);
    }
}

// row_softmax_topk with the smallest list length that holds k (and the runner-up, when the margin is wanted):
// k <= 16, and k <= 15 when the margin is wanted and k < E.
// LEAN: the caller's registers are full (lists of 16 by insertion).
template <int G, bool LEAN, Sums SUMS = Sums::Chain, class Z>
__device__ __forceinline__ void row_softmax_topk_upto16(Z&& z, int E, int k, int g,
                                                        int32_t* idx_row, float* probs_row, const EpilogueOut& o)
{
    const int need = k + ((o.margin_row && k < E) ? 1 : 0);
    if (need <= 2)      row_softmax_topk<2, G, false, SUMS>(z, E, k, g, idx_row, probs_row, o);
    else if (need <= 8) row_softmax_topk<8, G, true, SUMS>(z, E, k, g, idx_row, probs_row, o);
    else                row_softmax_topk<16, G, !LEAN, SUMS>(z, E, k, g, idx_row, probs_row, o);
}

}  // namespace paep
