// Building blocks shared by the forward and backward kernels.
//
// Edge functions are evaluated in float64. Every operand is an integer below
// 2^51 (snapped coordinates are bounded by 2^24, so products of differences
// are below 2^50), so each value, including the incremental form
// E(x, y) = E(x0, y0) + dx * a + dy * b, is exact and equals the int64 edge
// function of the contract; the tie rule and the conversion to float for the
// barycentrics therefore match it bit for bit.
#pragma once

#include "internal.hpp"

namespace soup {

struct Frag {
    uint64_t key;
    float beta[3];
};

// Perspective-correct barycentrics of vertices 1 and 2 from t_i = beta_i / w_i
// (contract order: r = 1 / ((t0 + t1) + t2), b_i = t_i r).
__device__ __forceinline__ void persp_from_t(float t0, float t1, float t2, float& b1, float& b2) {
    const float r = 1.0f / ((t0 + t1) + t2);
    b1 = t1 * r;
    b2 = t2 * r;
}

// Inclusive scans over the wave on the data-parallel primitives (DPP), with no
// LDS round trip: shifted moves by 1, 2, 4 and 8 lanes within each row of 16
// (a lane with no source in its row keeps its value), then the broadcasts of
// lane 15 into rows 1 and 3 and of lane 31 into rows 2 and 3 (the GFX9
// wave64 controls: row_shr:n = 0x110 + n, row_bcast:15 = 0x142,
// row_bcast:31 = 0x143).
template <int CTRL, int ROWS, class Op>
__device__ __forceinline__ int dpp_step(int v, int identity, Op op) {
    return op(v, __builtin_amdgcn_update_dpp(identity, v, CTRL, ROWS, 0xF, false));
}
template <class Op>
__device__ __forceinline__ int wave_scan_dpp(int v, int identity, Op op) {
    v = dpp_step<0x111, 0xF>(v, identity, op);
    v = dpp_step<0x112, 0xF>(v, identity, op);
    v = dpp_step<0x114, 0xF>(v, identity, op);
    v = dpp_step<0x118, 0xF>(v, identity, op);
    v = dpp_step<0x142, 0xA>(v, identity, op);
    return dpp_step<0x143, 0xC>(v, identity, op);
}
template <int CTRL, int ROWS>
__device__ __forceinline__ uint64_t dpp_max_step_u64(uint64_t v) {
    const uint32_t lo = static_cast<uint32_t>(__builtin_amdgcn_update_dpp(0, static_cast<int>(v), CTRL, ROWS, 0xF, false));
    const uint32_t hi =
        static_cast<uint32_t>(__builtin_amdgcn_update_dpp(0, static_cast<int>(v >> 32), CTRL, ROWS, 0xF, false));
    const uint64_t u = (static_cast<uint64_t>(hi) << 32) | lo;
    return u > v ? u : v;
}

// The largest value over the wave (wave-uniform).
__device__ __forceinline__ uint64_t wave_max_u64(uint64_t v) {
    v = dpp_max_step_u64<0x111, 0xF>(v);
    v = dpp_max_step_u64<0x112, 0xF>(v);
    v = dpp_max_step_u64<0x114, 0xF>(v);
    v = dpp_max_step_u64<0x118, 0xF>(v);
    v = dpp_max_step_u64<0x142, 0xA>(v);
    v = dpp_max_step_u64<0x143, 0xC>(v);
    const uint32_t lo = static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<int>(v), 63));
    const uint32_t hi = static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<int>(v >> 32), 63));
    return (static_cast<uint64_t>(hi) << 32) | lo;
}

// Smallest key any not-yet-processed entry of the tile list can produce.
// Lists are sorted in blocks of kSortBlock, so it is the minimum over the
// current position and the first entry of every later block.
__device__ __forceinline__ uint64_t remaining_min(const uint64_t* __restrict__ entries, int64_t beg, int64_t pos,
                                                  int64_t end) {
    uint64_t m = entries[pos];
    for (int64_t b = beg + ((pos - beg) / kSortBlock + 1) * kSortBlock; b < end; b += kSortBlock) {
        const uint64_t e = entries[b];
        m = e < m ? e : m;
    }
    return m;
}

// View that owns global tile `tile` (views sorted by tile_base).
__device__ __forceinline__ int view_of_tile(const ViewDesc* __restrict__ views, int V, int64_t tile) {
    int lo = 0, hi = V - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (views[mid].tile_base <= tile) lo = mid;
        else hi = mid - 1;
    }
    return lo;
}

}  // namespace soup
