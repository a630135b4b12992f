// Last step of every predict call whose inner width r was cut into slices that
// different workgroups worked on: each slice left its contribution to the
// scores in the workspace (fp32), and here one wave per token row adds the
// slices in ascending order (a fixed order, so the result is reproducible),
// adds b2, and runs softmax and top-k (eq. 1 and eq. 4) in registers with wave
// shuffles.  Lane l owns experts l, l + 64, ...
//
// The partial scores are laid out [tile][slice][BM][E]: a tile is BM token rows
// of one layer, tiles_per_layer of them to a layer (BM = T and one tile per
// layer where the producer does not tile the tokens).
#include "paep_device.h"
#include "paep_internal.h"

namespace paep {

static constexpr int FIN_THREADS = 256;

template <int NV>                                         // experts per lane: E <= 64 * NV
__global__ __launch_bounds__(FIN_THREADS) void finalize_kernel(
    int T, int E, int k, int S, int rows, int BM, int tile0, int tiles_per_layer, const float* __restrict__ partial,
    const void* __restrict__ b2, int b2_f32, int32_t* __restrict__ idx, float* __restrict__ probs,
    float* __restrict__ logits, int32_t* __restrict__ counts, int prob_mode, float* __restrict__ margin)
{
    const int lane = threadIdx.x & 63;
    const int slot = blockIdx.x * (FIN_THREADS / 64) + (threadIdx.x >> 6);
    if (slot >= rows) return;
    const int tile = slot / BM, tl = slot - tile * BM;
    const int layer = (tile + tile0) / tiles_per_layer;
    const int t = (tile + tile0 - layer * tiles_per_layer) * BM + tl;
    if (t >= T) return;
    const long long row = (long long)layer * T + t;
    const long long sstride = (long long)BM * E;
    const float* src = partial + ((long long)tile * S * BM + tl) * E;
    // all of a row's experts at once, CH slices per round: NV * CH loads in flight, added in ascending slice order
    constexpr int CH = (NV >= 8) ? 4 : 32 / NV;
    float z[NV];
#pragma unroll
    for (int v = 0; v < NV; ++v) z[v] = 0.0f;
    for (int s0 = 0; s0 < S; s0 += CH) {
        float p[NV][CH];
#pragma unroll
        for (int v = 0; v < NV; ++v) {
            const int e = lane + 64 * v;
#pragma unroll
            for (int u = 0; u < CH; ++u) p[v][u] = (e < E && s0 + u < S) ? src[(long long)(s0 + u) * sstride + e] : 0.0f;
        }
#pragma unroll
        for (int v = 0; v < NV; ++v)
#pragma unroll
            for (int u = 0; u < CH; ++u)
                if (s0 + u < S) z[v] += p[v][u];          // uniform; a skipped slice adds nothing, not even +0
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
    if constexpr (NV == 1) wave_softmax_topk_rank<NV>(z, E, k, lane, idx + row * k, probs + row * k, eo);
    else                   wave_softmax_topk<NV>(z, E, k, lane, idx + row * k, probs + row * k, eo);
}

hipError_t launch_finalize(const PredictArgs& a, const float* partial, int S, int tiles, int BM, int tile0,
                           int tiles_per_layer)
{
    const int rows = tiles * BM;
    const int rows_per_wg = FIN_THREADS / 64;
#define PAEP_LAUNCH_FIN(NVV)                                                                                     \
    hipLaunchKernelGGL(finalize_kernel<NVV>, dim3((rows + rows_per_wg - 1) / rows_per_wg), dim3(FIN_THREADS), 0, \
                       a.stream, a.T, a.E, a.k, S, rows, BM, tile0, tiles_per_layer, partial, a.b2,              \
                       a.dtype == 0 ? 1 : 0, a.idx, a.probs, a.logits, a.counts, a.prob_mode, a.margin)
    if (a.E <= 64)       PAEP_LAUNCH_FIN(1);
    else if (a.E <= 128) PAEP_LAUNCH_FIN(2);
    else if (a.E <= 256) PAEP_LAUNCH_FIN(4);
    else if (a.E <= 512) PAEP_LAUNCH_FIN(8);
    else                 PAEP_LAUNCH_FIN(16);
#undef PAEP_LAUNCH_FIN
    return hipGetLastError();
}

}  // namespace paep
