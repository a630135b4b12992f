// Last step of every predict call whose inner width r was cut into slices that
// different workgroups worked on: each slice left its contribution to the
// scores in the workspace (fp32); here a row's slices are added in ascending
// order (a fixed order, so the result is reproducible), b2 is added, and softmax
// and top-k (eq. 1 and eq. 4) follow in registers.  Two forms:
//   finalize_kernel       one wave per row, lane l owns experts l, l + 64, ...: the shortest path for
//                         one row, for calls of few rows
//   finalize_rows_kernel  4 to 16 lanes per row, up to 16 scores each as float4 loads, sorted lists merged
//                         between the lanes: fewer instructions per row, for calls of many.  Both move few
//                         bytes; what bounds them at many rows is instructions: 262144 rows of 16 experts
//                         in 2 slices 463 us with a wave per row, 14 us here; 16384 rows of 64 in 8 slices
//                         30 -> 9 us (where the line lies: finalize_rows_from)
//
// The partial scores are laid out [tile][slice][BM][E]: a tile is BM token rows
// of one layer, tiles_per_layer of them to a layer (BM = T and one tile per
// layer where the producer does not tile the tokens).
#include <limits.h>

#include "paep_device.h"
#include "paep_internal.h"

namespace paep {

static constexpr int FIN_THREADS = 256;

// NV: experts per lane, E <= 64 * NV.  WPR: waves per row, 1 or the whole workgroup.
template <int NV, int WPR>
__global__ __launch_bounds__(FIN_THREADS) void finalize_kernel(
    int T, int E, int k, int S, int rows, int BM, int tile0, int tiles_per_layer, const float* __restrict__ partial,
    const void* __restrict__ b2, int b2_f32, int32_t* __restrict__ idx, float* __restrict__ probs,
    float* __restrict__ logits, int32_t* __restrict__ counts, int prob_mode, float* __restrict__ margin)
{
    const int lane = threadIdx.x & 63;
    const int wave = threadIdx.x >> 6;
    const int slot = WPR == 1 ? blockIdx.x * (FIN_THREADS / 64) + wave : blockIdx.x;
    if (slot >= rows) return;
    const int tile = slot / BM, tl = slot - tile * BM;
    const int layer = (tile + tile0) / tiles_per_layer;
    const int t = (tile + tile0 - layer * tiles_per_layer) * BM + tl;
    if (t >= T) return;                                   // the waves of a row leave together
    const long long row = (long long)layer * T + t;
    const long long sstride = (long long)BM * E;
    const float* src = partial + ((long long)tile * S * BM + tl) * E;
    // this wave's slices
    const int s_begin = WPR == 1 ? 0 : wave * S / WPR, s_end = WPR == 1 ? S : (wave + 1) * S / WPR;
    // all of a row's experts at once, CH slices per round: NV * CH loads in flight, added in ascending slice order
    constexpr int CH = (NV >= 8) ? 4 : 32 / NV;
    float z[NV];
#pragma unroll
    for (int v = 0; v < NV; ++v) z[v] = 0.0f;
    for (int s0 = s_begin; s0 < s_end; s0 += CH) {
        float p[NV][CH];
#pragma unroll
        for (int v = 0; v < NV; ++v) {
            const int e = lane + 64 * v;
#pragma unroll
            for (int u = 0; u < CH; ++u) p[v][u] = (e < E && s0 + u < s_end) ? src[(long long)(s0 + u) * sstride + e] : 0.0f;
        }
#pragma unroll
        for (int v = 0; v < NV; ++v)
#pragma unroll
            for (int u = 0; u < CH; ++u)
                if (s0 + u < s_end) z[v] += p[v][u];      // uniform; a skipped slice adds nothing, not even +0
    }
    if constexpr (WPR > 1) {                              // the waves' sums, added in wave order
        __shared__ float part[WPR][64 * NV];
#pragma unroll
        for (int v = 0; v < NV; ++v) part[wave][lane + 64 * v] = z[v];
        __syncthreads();
        if (wave > 0) return;
#pragma unroll
        for (int v = 0; v < NV; ++v)
#pragma unroll
            for (int w = 1; w < WPR; ++w) z[v] += part[w][lane + 64 * v];
    }
#pragma unroll
    for (int v = 0; v < NV; ++v) {
        const int e = lane + 64 * v;
        if (e < E) {
            if (b2) {
                const long long i = (long long)layer * E + e;
                z[v] += b2_f32 ? ((const float*)b2)[i] : bf16_bits_to_f32(((const uint16_t*)b2)[i]);
            }
            if (logits) logits[row * E + e] = z[v];
        }
    }
    const EpilogueOut eo{prob_mode, margin ? margin + row : nullptr, counts ? counts + (long long)layer * E : nullptr};
    // one expert per lane: rank counting; more: k rounds of a wave-wide maximum (measured at 128 experts, k = 8:
    // 6.8 us against 9.6 us for rank counting at 48 rows, 11.6 against 17.7 at 3072 rows)
    if constexpr (NV == 1) wave_softmax_topk_rank(z[0], E, k, lane, idx + row * k, probs + row * k, eo);
    else                   wave_softmax_topk<NV>(z, E, k, lane, idx + row * k, probs + row * k, eo);
}

typedef f32x4 __attribute__((aligned(4))) f32x4_words;

// G lanes per row; lane g owns experts 4 * (j * G + g) + i, j < NJ, i < 4.  Lists of KMAX.  RAGGED: E is no multiple of
// 4; the loads are then aligned to words only, and the last lane's scores past E are left out one by one.
template <int NJ, int G, int KMAX, bool RAGGED>
__global__ __launch_bounds__(FIN_THREADS) void finalize_rows_kernel(
    int T, int E, int k, int S, int rows, int BM, int tile0, int tiles_per_layer, const float* __restrict__ partial,
    const void* __restrict__ b2, int b2_f32, int32_t* __restrict__ idx, float* __restrict__ probs,
    float* __restrict__ logits, int32_t* __restrict__ counts, int prob_mode, float* __restrict__ margin)
{
    const int slot = (blockIdx.x * FIN_THREADS + threadIdx.x) / G, g = threadIdx.x % G;
    if (slot >= rows) return;                             // the lanes of a row leave together
    const int tile = slot / BM, tl = slot - tile * BM;
    const int layer = (tile + tile0) / tiles_per_layer;
    const int t = (tile + tile0 - layer * tiles_per_layer) * BM + tl;
    if (t >= T) return;
    const long long row = (long long)layer * T + t;
    const long long sstride = (long long)BM * E;
    const float* src = partial + ((long long)tile * S * BM + tl) * E + 4 * g;
    f32x4 z[NJ];
#pragma unroll
    for (int j = 0; j < NJ; ++j) z[j] = f32x4{0.f, 0.f, 0.f, 0.f};
    constexpr int CH = 4;                                 // slices in flight
    for (int s0 = 0; s0 < S; s0 += CH) {
        f32x4 p[CH][NJ];
#pragma unroll
        for (int u = 0; u < CH; ++u)
#pragma unroll
            for (int j = 0; j < NJ; ++j)
                if (s0 + u < S && 4 * (j * G + g) < E) {
                    const float* at = src + (s0 + u) * sstride + 4 * j * G;
                    if (!RAGGED) {
                        p[u][j] = *(const f32x4*)at;
                    } else if (4 * (j * G + g) + 3 < E) {
                        p[u][j] = *(const f32x4_words*)at;
                    } else {
#pragma unroll
                        for (int i = 0; i < 4; ++i) p[u][j][i] = 4 * (j * G + g) + i < E ? at[i] : 0.f;
                    }
                }
#pragma unroll
        for (int u = 0; u < CH; ++u)
#pragma unroll
            for (int j = 0; j < NJ; ++j)
                if (s0 + u < S && 4 * (j * G + g) < E) z[j] += p[u][j];
    }
    TopList<KMAX> top;
    top.clear();
    constexpr bool SORTED = KMAX > 2 && NJ * 4 >= KMAX;   // whole lists of keys at a time
    constexpr int JB = SORTED ? KMAX / 4 : 1;
    skey more[JB * 4];
#pragma unroll
    for (int j = 0; j < NJ; ++j) {
        const int e = 4 * (j * G + g);
        if (e < E) {
            if (b2) {
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    if (RAGGED && e + i >= E) continue;
                    const long long c = (long long)layer * E + e + i;
                    z[j][i] += b2_f32 ? ((const float*)b2)[c] : bf16_bits_to_f32(((const uint16_t*)b2)[c]);
                }
            }
            if (logits)
#pragma unroll
                for (int i = 0; i < 4; ++i)
                    if (!RAGGED || e + i < E) logits[row * E + e + i] = z[j][i];
            if constexpr (!SORTED) {
#pragma unroll
                for (int i = 0; i < 4; ++i)
                    if (!RAGGED || e + i < E) top.insert(make_key(z[j][i], e + i));
            }
        }
        if constexpr (SORTED) {
#pragma unroll
            for (int i = 0; i < 4; ++i) more[(j % JB) * 4 + i] = (RAGGED ? e + i : e) < E ? make_key(z[j][i], e + i) : NO_KEY;
            if (j % JB == JB - 1) top.add(more, j < JB);
        }
    }
    top.template merge_group<G>();
    const EpilogueOut eo{prob_mode, margin ? margin + row : nullptr, counts ? counts + (long long)layer * E : nullptr};
    write_selection<KMAX, G>(top, E, k, g, idx + row * k, probs + row * k, eo, [&](float m) {
        float s = 0.0f;
#pragma unroll
        for (int j = 0; j < NJ; ++j)
#pragma unroll
            for (int i = 0; i < 4; ++i)
                if (4 * (j * G + g) + (RAGGED ? i : 0) < E && z[j][i] == z[j][i]) s += __expf(z[j][i] - m);
        return s;
    });
}

// Activation counts of the rows first_row .. L * T - 1 of a call, from their selections: counted in LDS, COUNT_ROWS rows
// of one layer at a time, and added to the layer's counters once.  (One global atomic per selection, as the rows'
// lanes do it where a layer has few rows, meets the others of a popular expert on one address.)
static constexpr int COUNT_ROWS = 2048;
__global__ __launch_bounds__(FIN_THREADS) void count_selected_kernel(int T, int E, int k, long long first_row,
                                                                     const int32_t* __restrict__ idx,
                                                                     int32_t* __restrict__ counts)
{
    extern __shared__ int32_t cnt[];                      // E
    const long long layer = first_row / T + blockIdx.y;
    const long long first = layer * T > first_row ? layer * T : first_row;
    const long long row0 = first + (long long)blockIdx.x * COUNT_ROWS, end = (layer + 1) * T;
    if (row0 >= end) return;
    for (int e = threadIdx.x; e < E; e += FIN_THREADS) cnt[e] = 0;
    __syncthreads();
    const int rows = end - row0 < COUNT_ROWS ? (int)(end - row0) : COUNT_ROWS;
    const int32_t* src = idx + row0 * k;
    for (int i = threadIdx.x; i < rows * k; i += FIN_THREADS) atomicAdd(&cnt[src[i]], 1);
    __syncthreads();
    for (int e = threadIdx.x; e < E; e += FIN_THREADS)
        if (cnt[e]) atomicAdd(&counts[layer * E + e], cnt[e]);
}

// Rows from which on finalize_rows_kernel is the faster form; `need` keys are kept per row.  It takes a row's S slices in
// rounds of four and fewer waves for the same rows, so it wants more of them the more slices there are and the longer the
// lists; the other form takes a row per wave, up to 32 slices at once, and 8192 rows at a time.  us, wave per row /
// several lanes per row:
//   16 experts, k = 2 or 6   1024 rows, 16 slices 6.2 / 4.3-5.7; 32 slices 1024 rows 6.3 / 7.1, 1536 rows 7.4 / 7.1
//   64, k = 6     2 slices: 1536 rows 7.3 / 6.9; 8: 2048 rows 7.4 / 7.9, 3072 rows 8.6 / 7.9; 16: 1664 rows 7.4 / 9.4,
//                 4096 rows 9.7 / 9.5; 32: 4096 rows 10.1 / 13.3, 8192 rows 19.9 / 17.8
//   64, k = 12    2 slices: 4096 rows 9.7 / 9.9; 8: 5120 rows 12.2 / 10.9; 16: 6144 rows 13.8 / 13.0
//   128, k = 8    2 slices: 2048 rows 7.8 / 8.0; 8: 3072 rows 9.0 / 8.9; 16: 4096 rows 10.1 / 11.0, 8192 rows 17.4 / 17.0
//   256, k = 8    2 slices: 2048 rows 8.0 / 8.8, 4096 rows 10.1 / 8.8; 8: 4096 rows 10.4 / 10.2; 16: 8192 rows 25.9 / 26.4,
//                 16384 rows 43.9 / 44.9
// The scores past E of the last lane cost E that is no multiple of 4 a third more rows (62, k = 6: 8 slices 3072 rows
// 8.7 / 9.3, 4096 rows 9.8 / 9.3; 16: 5120 rows 12.4 / 11.9).
static int finalize_rows_from(int E, int S, int need)
{
    int from = need <= 8 ? 1024 : E <= 16 ? 2048 : 4096;
    if (E > 128 && S >= 16) return INT_MAX;
    if (E > 16) from += 192 * S + (E > 64 ? 8 * E : 0);
    else if (S * 48 > from) from = S * 48;
    return E % 4 == 0 ? from : from / 3 * 4;
}

// Rows from which on the counts are taken from the selections, in calls whose layers have more rows than a decode batch
// (or where every row selects most of the experts): one launch more, 2 us, where atomics from the rows' lanes cost
// 0.2 to 1 us for 16 x 64 rows, 12 us for 16 x 512 of 64 experts.
static constexpr int FIN_COUNT_ROWS = 1024;

hipError_t launch_finalize(const PredictArgs& a, const float* partial, int S, int tiles, int BM, int tile0,
                           int tiles_per_layer)
{
    const int rows = tiles * BM;
    const int need = a.k + ((a.margin && a.k < a.E) ? 1 : 0);     // sorted keys per row
    const bool many = a.E <= 256 && need <= 16 && rows >= finalize_rows_from(a.E, S, need);
    if (a.counts && rows >= FIN_COUNT_ROWS && (a.T > 64 || (many && 2 * a.k > a.E))) {
        PredictArgs b = a;
        b.counts = nullptr;
        const hipError_t err = launch_finalize(b, partial, S, tiles, BM, tile0, tiles_per_layer);
        if (err != hipSuccess) return err;
        // the tiles are the call's last ones
        const int layer0 = tile0 / tiles_per_layer;
        const long long first_row = (long long)layer0 * a.T + (long long)(tile0 - layer0 * tiles_per_layer) * BM;
        hipLaunchKernelGGL(count_selected_kernel, dim3((a.T + COUNT_ROWS - 1) / COUNT_ROWS, a.L - layer0),
                           dim3(FIN_THREADS), sizeof(int32_t) * a.E, a.stream, a.T, a.E, a.k, first_row, a.idx, a.counts);
        return hipGetLastError();
    }
    if (many) {
#define PAEP_LAUNCH_FINR(NJV, GV, KV)                                                                            \
    hipLaunchKernelGGL((a.E % 4 == 0 ? finalize_rows_kernel<NJV, GV, KV, false> : finalize_rows_kernel<NJV, GV, KV, true>), \
                       dim3((rows + FIN_THREADS / GV - 1) / (FIN_THREADS / GV)), dim3(FIN_THREADS), 0, a.stream, a.T, a.E, a.k, S, rows, BM, tile0, tiles_per_layer, partial, \
                       a.b2, a.dtype == 0 ? 1 : 0, a.idx, a.probs, a.logits, a.counts, a.prob_mode, a.margin)
#define PAEP_LAUNCH_FINR_K(NJV, GV)                                                                              \
    do {                                                                                                         \
        if (need <= 2)      PAEP_LAUNCH_FINR(NJV, GV, 2);                                                        \
        else if (need <= 8) PAEP_LAUNCH_FINR(NJV, GV, 8);                                                        \
        else                PAEP_LAUNCH_FINR(NJV, GV, 16);                                                       \
    } while (0)
        if (a.E <= 16)       PAEP_LAUNCH_FINR_K(1, 4);
        else if (a.E <= 64)  PAEP_LAUNCH_FINR_K(4, 4);
        else if (a.E <= 128) PAEP_LAUNCH_FINR_K(4, 8);
        else                 PAEP_LAUNCH_FINR_K(4, 16);
#undef PAEP_LAUNCH_FINR_K
#undef PAEP_LAUNCH_FINR
        return hipGetLastError();
    }
    // many slices and few rows: four waves share a row's slices (a wave alone takes them in rounds of 32 loads, one
    // memory round trip each)
    const bool wide = S >= 64 && rows <= 256;
    const int rows_per_wg = wide ? 1 : FIN_THREADS / 64;
#define PAEP_LAUNCH_FIN(NVV)                                                                                     \
    hipLaunchKernelGGL((wide ? finalize_kernel<NVV, 4> : finalize_kernel<NVV, 1>),                              \
                       dim3((rows + rows_per_wg - 1) / rows_per_wg), dim3(FIN_THREADS), 0, a.stream, a.T, a.E,  \
                       a.k, S, rows, BM, tile0, tiles_per_layer, partial, a.b2, a.dtype == 0 ? 1 : 0, a.idx,     \
                       a.probs, a.logits, a.counts, a.prob_mode, a.margin)
    if (a.E <= 64)       PAEP_LAUNCH_FIN(1);
    else if (a.E <= 128) PAEP_LAUNCH_FIN(2);
    else if (a.E <= 256) PAEP_LAUNCH_FIN(4);
    else if (a.E <= 512) PAEP_LAUNCH_FIN(8);
    else                 PAEP_LAUNCH_FIN(16);
#undef PAEP_LAUNCH_FIN
    return hipGetLastError();
}

}  // namespace paep
