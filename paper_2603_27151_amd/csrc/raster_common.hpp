// Building blocks shared by the forward and backward kernels.
//
// A fragment's edge functions are evaluated in float64. Every operand is an
// integer below 2^51 (snapped coordinates are bounded by 2^24, so products of
// differences are below 2^50), so each value, including the incremental form
// E(x, y) = E(x0, y0) + dx * a + dy * b, is exact and equals the int64 edge
// function of the contract; the conversion to float for the barycentrics
// therefore matches it bit for bit. (Coverage takes its signs, with the tie
// rule, from 32-bit integers: raster_fwd_impl.hpp.)
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
// The largest values over the wave of NB values per lane (wave-uniform): the
// high words first, then the low words of the lanes that hold the largest
// one. Six 32-bit steps each, of one instruction, with the values' steps side
// by side, where 64-bit steps took seven and waited for each other (64 views of
// 50,000 triangles: forward 1.60 -> 1.55 ms).
__device__ __forceinline__ uint32_t max_u32(uint32_t a, uint32_t b) { return a > b ? a : b; }
template <int CTRL, int ROWS, int NB>
__device__ __forceinline__ void dpp_max_step(uint32_t (&v)[NB]) {
#pragma unroll
    for (int b = 0; b < NB; ++b)
        v[b] = max_u32(v[b], static_cast<uint32_t>(__builtin_amdgcn_update_dpp(0, static_cast<int>(v[b]), CTRL, ROWS, 0xF, false)));
}
template <int NB>
__device__ __forceinline__ void wave_max_u32(uint32_t (&v)[NB]) {
    dpp_max_step<0x111, 0xF>(v);
    dpp_max_step<0x112, 0xF>(v);
    dpp_max_step<0x114, 0xF>(v);
    dpp_max_step<0x118, 0xF>(v);
    dpp_max_step<0x142, 0xA>(v);
    dpp_max_step<0x143, 0xC>(v);
#pragma unroll
    for (int b = 0; b < NB; ++b) v[b] = static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<int>(v[b]), 63));
}
template <int NB>
__device__ __forceinline__ void wave_max_u64(const uint64_t (&v)[NB], uint64_t (&out)[NB]) {
    uint32_t hi[NB], lo[NB];
#pragma unroll
    for (int b = 0; b < NB; ++b) hi[b] = static_cast<uint32_t>(v[b] >> 32);
    wave_max_u32(hi);
#pragma unroll
    for (int b = 0; b < NB; ++b) lo[b] = static_cast<uint32_t>(v[b] >> 32) == hi[b] ? static_cast<uint32_t>(v[b]) : 0u;
    wave_max_u32(lo);
#pragma unroll
    for (int b = 0; b < NB; ++b) out[b] = (static_cast<uint64_t>(hi[b]) << 32) | lo[b];
}

// Smallest key any not-yet-processed entry of the tile list can produce.
// Lists are sorted in blocks of kSortBlock, so it is the minimum over the
// current position, whose entry is `first`, and the first entry of every later
// block.
__device__ __forceinline__ uint64_t remaining_min(const uint64_t* __restrict__ entries, int64_t beg, int64_t pos,
                                                  int64_t end, uint64_t first) {
    uint64_t m = first;
    for (int64_t b = beg + ((pos - beg) / kSortBlock + 1) * kSortBlock; b < end; b += kSortBlock) {
        const uint64_t e = entries[b];
        m = e < m ? e : m;
    }
    return m;
}

// The view that owns a global tile, found by the whole wave (views sorted by
// tile_base): lane l stands for view l * step and keeps its first tile, so that
// up to 64 views need no memory access, up to 4096 one.
struct ViewFinder {
    int step, scene = 0;             // views per lane; with one, its scene
    uint32_t base = 0xFFFFFFFFu;     // (tiles are fewer than 2^32 - 1)
    __device__ __forceinline__ void init(const ViewDesc* __restrict__ views, int V, int lane) {
        step = (V + 63) >> 6;
        if (static_cast<int64_t>(lane) * step < V) {
            base = static_cast<uint32_t>(views[lane * step].tile_base);
            if (step == 1) scene = views[lane].scene;
        }
    }
    __device__ __forceinline__ int find(const ViewDesc* __restrict__ views, int V, uint32_t tile, int lane) const {
        int v = (__popcll(__ballot(base <= tile)) - 1) * step;
        for (int n = step; n > 1;) {   // among n views from v
            const int s = (n + 63) >> 6, o = lane * s;
            const bool in = o < n && v + o < V;
            const uint64_t m = __ballot(in && static_cast<uint32_t>(views[in ? v + o : v].tile_base) <= tile);
            v += (__popcll(m) - 1) * s;
            n = s;
        }
        return v;
    }
};

}  // namespace soup
