// What the prefill kernels share: wait counts, the LDS pointer of a direct copy, compile-time loops.
#pragma once

#include <type_traits>

#include "paep_device.h"
#include "paep_internal.h"

namespace paep {

// s_waitcnt immediates (gfx9 encoding): vmcnt <= n and nothing else; lgkmcnt(0) and nothing else
#define PAEP_VMCNT(n) ((((n) & 0xF) | (((n) >> 4) << 14)) | 0x0F70)
static constexpr int PAEP_LGKM0 = 0xC07F;

typedef void __attribute__((address_space(3)))* lptr_t;

template <int V> using IC = std::integral_constant<int, V>;
template <int N, class F> __device__ __forceinline__ void static_for(F&& f)
{
    if constexpr (N > 0) {
        static_for<N - 1>(f);
        f(IC<N - 1>{});
    }
}

// The grid of a prefill launch: the first main_wgs workgroups run whole tiles with main_groups workgroups each, the
// other tail_wgs the remaining tiles with tail_groups each; score tiles from split_tile0 on go through `zpart`.  tile_fastest: of
// a layer, (group, tile) instead of (tile, group).
struct PrefillGrid {
    int tiles_per_layer, main_wgs, main_groups, tail_wgs, tail_groups, split_tile0;
    float* zpart;
    int tile_fastest;
};

// prefill256.hip: tiles of `tokens` x `units` hidden units: 256 tokens x 256 (E <= 128) or 128 (64 < E <= 256), 160, 192 or 224 x 256 (E <= 64),
// 128 x 256 (E <= 128).  h: the first layer alone,
// 256 units, hidden vectors (before the activation) to memory, laid out in fragments for scores_of_h; null: everything.
hipError_t launch_prefill256(const PredictArgs& a, const PrefillGrid& grid, int tokens, int units, u32x4* h);

}  // namespace paep
