// Triangle setup and screen-tile binning.
//
// setup:   per (view, triangle): projection, culling, snapping to 1/256 px,
//          bounding box, a lower bound of the depth of any of its fragments;
//          counts its (tile, triangle) pairs per tile (through an LDS
//          histogram per chunk of triangles when the view's tiles fit).
// scan:    exclusive scan of the per-tile counts -> per-tile list offsets.
// scatter: per (view, triangle): writes (zmin << 32 | tri) into the list of
//          every tile its bounding box touches.
// sort:    sorts each tile's list ascending (a wave sorts a short list
//          bitonic in registers; a workgroup sorts a long one likewise,
//          in blocks of kSortBlock entries), so that the raster can walk
//          triangles front to back and stop early.
#include "internal.hpp"

namespace soup {

// One triangle's setup record in one view; whether any pixel centre of the view can be inside it.
__device__ __forceinline__ bool setup_record(const float* __restrict__ p, const ViewDesc& vd, float near_w, TriRec& r) {
    const float* M = vd.M;
    const float hw = 0.5f * static_cast<float>(vd.W), hh = 0.5f * static_cast<float>(vd.H);
    bool ok = true;
#pragma unroll
    for (int i = 0; i < 3; ++i) {
        const float x = p[3 * i], y = p[3 * i + 1], z = p[3 * i + 2];
        float c[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            float a = M[j * 4 + 3];
            a = __builtin_fmaf(M[j * 4 + 0], x, a);
            a = __builtin_fmaf(M[j * 4 + 1], y, a);
            a = __builtin_fmaf(M[j * 4 + 2], z, a);
            c[j] = a;
        }
        ok = ok && (c[3] >= near_w) && __builtin_isfinite(c[0]) && __builtin_isfinite(c[1]) &&
             __builtin_isfinite(c[2]) && __builtin_isfinite(c[3]);
        const float iw = 1.0f / c[3];
        const float sx = __builtin_fmaf(c[0] * iw, hw, hw);
        const float sy = __builtin_fmaf(-(c[1] * iw), hh, hh);
        const float z01 = __builtin_fmaf(c[2] * iw, 0.5f, 0.5f);
        const float fx = sx * 256.0f, fy = sy * 256.0f;
        ok = ok && (__builtin_fabsf(fx) <= kGuard) && (__builtin_fabsf(fy) <= kGuard) && __builtin_isfinite(z01);
        r.X[i] = ok ? static_cast<int32_t>(__builtin_rintf(fx)) : 0;
        r.Y[i] = ok ? static_cast<int32_t>(__builtin_rintf(fy)) : 0;
        r.z01[i] = z01;
        r.iw[i] = iw;
    }
    const int64_t A = static_cast<int64_t>(r.X[1] - r.X[0]) * (r.Y[2] - r.Y[0]) -
                      static_cast<int64_t>(r.Y[1] - r.Y[0]) * (r.X[2] - r.X[0]);
    ok = ok && A != 0;
    const int32_t mnx = min(r.X[0], min(r.X[1], r.X[2])), mxx = max(r.X[0], max(r.X[1], r.X[2]));
    const int32_t mny = min(r.Y[0], min(r.Y[1], r.Y[2])), mxy = max(r.Y[0], max(r.Y[1], r.Y[2]));
    // pixel x is a candidate when mnx <= 256 x + 128 <= mxx
    const int32_t x0 = max((mnx + 127) >> 8, 0), x1 = min((mxx - 128) >> 8, vd.W - 1);
    const int32_t y0 = max((mny + 127) >> 8, 0), y1 = min((mxy - 128) >> 8, vd.H - 1);
    ok = ok && x0 <= x1 && y0 <= y1;
    if (ok) {
        const int64_t aA = A < 0 ? -A : A;
        float rA = 1.0f / static_cast<float>(aA);
        r.rA = A < 0 ? -rA : rA;
        float zm = fminf(r.z01[0], fminf(r.z01[1], r.z01[2]));
        if (!(zm > 0.0f)) zm = 0.0f;
        if (zm > 1.0f) zm = 1.0f;
        const uint32_t zb = __float_as_uint(zm);
        r.zmin = zb > kZminMargin ? zb - kZminMargin : 0u;
        r.x0 = static_cast<int16_t>(x0);
        r.x1 = static_cast<int16_t>(x1);
        r.y0 = static_cast<int16_t>(y0);
        r.y1 = static_cast<int16_t>(y1);
    } else {
        r.rA = 0.0f;
        r.zmin = 0xFFFFFFFFu;
        r.x0 = 1;
        r.x1 = 0;
        r.y0 = 1;
        r.y1 = 0;
    }
    return ok;
}

// Large chunks: one workgroup bins a chunk of `chunk` triangles of one view. When
// the view has at most kHistBins tiles, its (tile, triangle) pairs are counted
// in an LDS histogram, and only the chunk's non-zero tile counts go to the global
// counters (one returning atomic per tile touched: the chunk's first slot in
// that tile's list); otherwise every pair is counted with a global atomic.
__global__ __launch_bounds__(256) void setup_kernel(const ViewDesc* __restrict__ views,
                                                    const SceneDesc* __restrict__ scenes, Opts o, int tile, int chunk,
                                                    TriRec* __restrict__ recs, int32_t* __restrict__ tile_count,
                                                    int32_t* __restrict__ chunk_base, int64_t n_tiles,
                                                    unsigned long long* __restrict__ visible) {
    __shared__ int32_t hist[kHistBins];
    const ViewDesc& vd = views[blockIdx.y];
    const int t_beg = blockIdx.x * chunk;
    if (t_beg >= vd.T) return;
    const int t_end = min(t_beg + chunk, vd.T);
    const int nb = vd.tiles_x * vd.tiles_y;
    const bool local = nb <= kHistBins;
    if (local) {
        for (int b = threadIdx.x; b < nb; b += blockDim.x) hist[b] = 0;
        __syncthreads();
    }
    const SceneDesc sc = scenes[vd.scene];
    for (int t = t_beg + static_cast<int>(threadIdx.x); t < t_end; t += blockDim.x) {
        TriRec r;
        const bool ok = setup_record(sc.verts + static_cast<size_t>(t) * 9, vd, o.near_w, r);
        if (ok) {
            const int tx0 = r.x0 / tile, tx1 = r.x1 / tile, ty0 = r.y0 / tile, ty1 = r.y1 / tile;
            for (int ty = ty0; ty <= ty1; ++ty)
                for (int tx = tx0; tx <= tx1; ++tx) {
                    const int b = ty * vd.tiles_x + tx;
                    if (local) atomicAdd(&hist[b], 1);
                    else atomicAdd(&tile_count[vd.tile_base + b], 1);
                }
        }
        recs[vd.rec_base + t] = r;
        if (visible) {
            const uint64_t m = __ballot(ok);
            if (lane_id() == __builtin_ctzll(__ballot(1)) && m)
                atomicAdd(visible, static_cast<unsigned long long>(__popcll(m)));
        }
    }
    if (local) {
        __syncthreads();
        int32_t* base = chunk_base + static_cast<int64_t>(blockIdx.x) * n_tiles + vd.tile_base;
        for (int b = threadIdx.x; b < nb; b += blockDim.x) {
            const int n = hist[b];
            if (n) base[b] = atomicAdd(&tile_count[vd.tile_base + b], n);
        }
    }
}

// Writes (zmin << 32 | tri) into the list of every tile a triangle's bounding
// box touches, over the same chunks as the setup. A view binned in LDS takes
// its positions from an LDS cursor per tile, started at the tile's list offset
// plus the chunk's first slot; other views take them from a global atomic.
__global__ __launch_bounds__(256) void scatter_kernel(const ViewDesc* __restrict__ views, int tile, int chunk,
                                                      const TriRec* __restrict__ recs,
                                                      const int64_t* __restrict__ tile_start, int64_t n_tiles,
                                                      const int32_t* __restrict__ chunk_base,
                                                      int32_t* __restrict__ tile_fill,
                                                      uint64_t* __restrict__ entries, int64_t cap) {
    __shared__ unsigned long long cur[kHistBins];
    const ViewDesc& vd = views[blockIdx.y];
    const int t_beg = blockIdx.x * chunk;
    if (t_beg >= vd.T) return;
    const int64_t total = tile_start[n_tiles];
    if (total == 0) return;   // no entries, or lists emptied by the static capacity check
    const int t_end = min(t_beg + chunk, vd.T);
    const int nb = vd.tiles_x * vd.tiles_y;
    const bool local = nb <= kHistBins;
    if (local) {
        // bins this chunk does not touch hold stale offsets and are never used
        const int32_t* base = chunk_base + static_cast<int64_t>(blockIdx.x) * n_tiles + vd.tile_base;
        for (int b = threadIdx.x; b < nb; b += blockDim.x)
            cur[b] = static_cast<unsigned long long>(tile_start[vd.tile_base + b] + base[b]);
        __syncthreads();
    }
    for (int t = t_beg + static_cast<int>(threadIdx.x); t < t_end; t += blockDim.x) {
        const TriRec r = recs[vd.rec_base + t];
        if (r.x0 > r.x1) continue;
        const uint64_t e = (static_cast<uint64_t>(r.zmin) << 32) | static_cast<uint32_t>(t);
        const int tx0 = r.x0 / tile, tx1 = r.x1 / tile, ty0 = r.y0 / tile, ty1 = r.y1 / tile;
        for (int ty = ty0; ty <= ty1; ++ty)
            for (int tx = tx0; tx <= tx1; ++tx) {
                const int b = ty * vd.tiles_x + tx;
                int64_t at;
                if (local) {
                    at = static_cast<int64_t>(atomicAdd(&cur[b], 1ull));
                } else {
                    const int64_t g = vd.tile_base + b;
                    at = tile_start[g] + atomicAdd(&tile_fill[g], 1);
                }
                if (at < cap) entries[at] = e;   // false only in lists longer than the buffer (which are made again)
            }
    }
}

// The (tile, triangle) pairs of a small chunk (at most 256 triangles), dealt to
// the whole workgroup: thread t leaves its triangle's tile rectangle, the counts
// are scanned, and pair p belongs to the triangle whose run of pairs holds p.
// Each thread then has a few independent atomics in flight, however many tiles
// one triangle touches. (One triangle per thread, its tiles in a loop, waited
// for a returning atomic per tile, a wave as long as its largest triangle: 64
// large triangles took 20 us to scatter, now 4; four views of 50,000 triangles
// 90 us for the setup and 126 us for the scatter, now 50 and 44 with the spread
// counters. The LDS of the histogram chunks, which the same kernel held, also
// left two workgroups per CU.)
struct PairRuns {
    int incl[256];      // inclusive scan of the triangles' tile counts
    int16_t x0[256], y0[256], nx[256];
    int wsum[4];
    // n = this thread's tile count; the total over the workgroup
    __device__ __forceinline__ int scan(int n) {
        const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
        int v = n;
#pragma unroll
        for (int d = 1; d < 64; d <<= 1) {
            const int u = __shfl_up(v, d, 64);
            if (lane >= d) v += u;
        }
        if (lane == 63) wsum[w] = v;
        __syncthreads();
        int total = 0;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            if (i < w) v += wsum[i];
            total += wsum[i];
        }
        incl[tid] = v;
        __syncthreads();
        return total;
    }
    // the triangle of pair p (the first whose inclusive count exceeds p) and the pair's tile
    __device__ __forceinline__ int find(int p, int tiles_x, int& tile) const {
        int lo = 0, hi = 255;
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const int mid = (lo + hi) >> 1;
            if (incl[mid] > p) hi = mid;
            else lo = mid + 1;
        }
        const uint32_t k = static_cast<uint32_t>(p - (hi ? incl[hi - 1] : 0)), wide = static_cast<uint32_t>(nx[hi]);
        const uint32_t ty = k / wide;
        tile = (y0[hi] + static_cast<int>(ty)) * tiles_x + x0[hi] + static_cast<int>(k - ty * wide);
        return hi;
    }
    // this thread's rectangle (pixels x0..x1, y0..y1; none if x0 > x1) in tiles; the
    // total (every thread of the workgroup calls it: it holds barriers)
    __device__ __forceinline__ int put(int px0, int py0, int px1, int py1, int tile) {
        const int tid = threadIdx.x;
        int n = 0;
        if (px0 <= px1) {
            const int tx0 = px0 / tile, ty0 = py0 / tile, w = px1 / tile - tx0 + 1;
            n = w * (py1 / tile - ty0 + 1);
            x0[tid] = static_cast<int16_t>(tx0);
            y0[tid] = static_cast<int16_t>(ty0);
            nx[tid] = static_cast<int16_t>(w);
        }
        return scan(n);
    }
};

__global__ __launch_bounds__(256) void setup_small_kernel(const ViewDesc* __restrict__ views,
                                                          const SceneDesc* __restrict__ scenes, Opts o, int tile,
                                                          int chunk, TriRec* __restrict__ recs,
                                                          int32_t* __restrict__ tile_count, int stride,
                                                          unsigned long long* __restrict__ visible) {
    __shared__ PairRuns s;
    const ViewDesc& vd = views[blockIdx.y];
    const int tid = threadIdx.x, t = blockIdx.x * chunk + tid;
    if (blockIdx.x * chunk >= vd.T) return;
    TriRec r;
    r.x0 = r.y0 = 1;   // an empty box (a culled triangle's record has one too)
    r.x1 = r.y1 = 0;
    bool ok = false;
    if (tid < chunk && t < vd.T) {
        ok = setup_record(scenes[vd.scene].verts + static_cast<size_t>(t) * 9, vd, o.near_w, r);
        recs[vd.rec_base + t] = r;
    }
    if (visible) {
        const uint64_t m = __ballot(ok);
        if (m && lane_id() == 0) atomicAdd(visible, static_cast<unsigned long long>(__popcll(m)));
    }
    const int total = s.put(r.x0, r.y0, r.x1, r.y1, tile);
    for (int p = tid; p < total; p += 256) {
        int b;
        s.find(p, vd.tiles_x, b);
        atomicAdd(&tile_count[(vd.tile_base + b) * stride], 1);
    }
}

__global__ __launch_bounds__(256) void scatter_small_kernel(const ViewDesc* __restrict__ views, int tile, int chunk,
                                                            const TriRec* __restrict__ recs,
                                                            const int64_t* __restrict__ tile_start, int64_t n_tiles,
                                                            int32_t* __restrict__ tile_fill, int stride,
                                                            uint64_t* __restrict__ entries, int64_t cap) {
    __shared__ PairRuns s;
    __shared__ uint32_t zmin[256];
    const ViewDesc& vd = views[blockIdx.y];
    const int tid = threadIdx.x, t0 = blockIdx.x * chunk, t = t0 + tid;
    if (t0 >= vd.T) return;
    const int64_t n_entries = tile_start[n_tiles];
    if (n_entries == 0) return;   // no entries, or lists emptied by the static capacity check
    uint4 q = make_uint4(0u, 0u, 1u, 0u);   // (area, zmin, x0 | y0 << 16, x1 | y1 << 16): an empty box
    if (tid < chunk && t < vd.T) q = reinterpret_cast<const uint4*>(recs + vd.rec_base + t)[3];
    zmin[tid] = q.y;
    const int total = s.put(static_cast<int16_t>(q.z & 0xFFFFu), static_cast<int16_t>(q.z >> 16),
                            static_cast<int16_t>(q.w & 0xFFFFu), static_cast<int16_t>(q.w >> 16), tile);
    constexpr int U = 4;   // pairs in flight per thread
    for (int p0 = tid; p0 < total; p0 += U * 256) {
        int64_t at[U];
        uint64_t e[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int p = p0 + u * 256;
            at[u] = cap;
            e[u] = 0;
            if (p < total) {
                int b;
                const int j = s.find(p, vd.tiles_x, b);
                const int64_t g = vd.tile_base + b;
                e[u] = (static_cast<uint64_t>(zmin[j]) << 32) | static_cast<uint32_t>(t0 + j);
                at[u] = tile_start[g] + atomicAdd(&tile_fill[g * stride], 1);
            }
        }
#pragma unroll
        for (int u = 0; u < U; ++u)
            if (at[u] < cap) entries[at[u]] = e[u];   // false past the pairs, and in lists longer than the buffer
    }
}

// The value of lane (lane ^ J), J = 1, 2, 4 .. 32, by lane permutations within
// the vector ALU (through the LDS a general shuffle waits for its round trip).
template <int J>
__device__ __forceinline__ uint32_t xor_lane(uint32_t v) {
    auto dpp = [](uint32_t x, auto ctrl) __attribute__((always_inline)) {
        return static_cast<uint32_t>(__builtin_amdgcn_mov_dpp(static_cast<int>(x), decltype(ctrl)::value, 0xF, 0xF, true));
    };
    if constexpr (J == 1) {
        return dpp(v, std::integral_constant<int, 0xB1>{});        // quad_perm 1 0 3 2
    } else if constexpr (J == 2) {
        return dpp(v, std::integral_constant<int, 0x4E>{});        // quad_perm 2 3 0 1
    } else if constexpr (J == 4) {                                 // ^7 (row_half_mirror), then ^3 (quad_perm 3 2 1 0)
        return dpp(dpp(v, std::integral_constant<int, 0x141>{}), std::integral_constant<int, 0x1B>{});
    } else if constexpr (J == 8) {
        return dpp(v, std::integral_constant<int, 0x128>{});       // row_ror:8
    } else if constexpr (J == 16) {   // rows (0, 0, 2, 2) and (1, 1, 3, 3)
        const auto q = __builtin_amdgcn_permlane16_swap(v, v, false, false);
        return lane_id() & 16 ? q[0] : q[1];
    } else {                          // halves (lo, lo) and (hi, hi)
        static_assert(J == 32);
        const auto q = __builtin_amdgcn_permlane32_swap(v, v, false, false);
        return lane_id() & 32 ? q[0] : q[1];
    }
}
template <int J>
__device__ __forceinline__ uint64_t xor_lane(uint64_t v) {
    const uint32_t lo = xor_lane<J>(static_cast<uint32_t>(v)), hi = xor_lane<J>(static_cast<uint32_t>(v >> 32));
    return (static_cast<uint64_t>(hi) << 32) | lo;
}

// Bitonic sort of up to 64 R W entries by W waves, held in registers: entry e =
// 64 R w + 64 r + lane is register r of its lane in wave w (the slots past n
// hold the largest key and stay at the end). A compare-exchange at distance j
// pairs e with e ^ j: between lanes for j < 64, between two registers of one
// lane for 64 <= j < 64 R, between two waves, through the LDS, for the three
// steps at j >= 64 R of four waves. Entry e keeps the smaller key when it is
// the lower of its pair in an ascending run (e & k == 0) or the upper of its
// pair in a descending one.
template <int R, int J>
__device__ __forceinline__ void exchange_lanes(uint64_t (&v)[R], int e0, int k) {
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const int e = e0 + 64 * r;
        const uint64_t a = v[r], b = xor_lane<J>(a);
        const bool keep_min = ((e & J) == 0) == ((e & k) == 0);
        v[r] = (a < b) == keep_min ? a : b;
    }
}
template <int R, int W>
__device__ __forceinline__ void bitonic_sort(uint64_t* __restrict__ list, int n, int w, uint64_t* __restrict__ s) {
    const int lane = lane_id(), e0 = 64 * R * w + lane;
    constexpr int N = 64 * R * W;
    uint64_t v[R];
#pragma unroll
    for (int r = 0; r < R; ++r) v[r] = e0 + 64 * r < n ? list[e0 + 64 * r] : kBgKey;
#pragma unroll
    for (int k = 2; k <= N; k <<= 1) {
#pragma unroll
        for (int j = k >> 1; j >= 64; j >>= 1) {
            if (j >= 64 * R) {
                __syncthreads();   // the last exchange's reads are done
#pragma unroll
                for (int r = 0; r < R; ++r) s[e0 + 64 * r] = v[r];
                __syncthreads();
#pragma unroll
                for (int r = 0; r < R; ++r) {
                    const int e = e0 + 64 * r;
                    const uint64_t a = v[r], b = s[e ^ j];
                    const bool keep_min = ((e & j) == 0) == ((e & k) == 0);
                    v[r] = (a < b) == keep_min ? a : b;
                }
            } else {
                const int jr = j >> 6;
#pragma unroll
                for (int r = 0; r < R; ++r) {
                    if (r & jr) continue;   // the pair (r, r + jr), seen from its lower register
                    const uint64_t a = v[r], b = v[r | jr];
                    const bool up = ((e0 + 64 * r) & k) == 0, swap = (a < b) != up;
                    v[r] = swap ? b : a;
                    v[r | jr] = swap ? a : b;
                }
            }
        }
        if (k > 32) exchange_lanes<R, 32>(v, e0, k);
        if (k > 16) exchange_lanes<R, 16>(v, e0, k);
        if (k > 8) exchange_lanes<R, 8>(v, e0, k);
        if (k > 4) exchange_lanes<R, 4>(v, e0, k);
        if (k > 2) exchange_lanes<R, 2>(v, e0, k);
        exchange_lanes<R, 1>(v, e0, k);
    }
#pragma unroll
    for (int r = 0; r < R; ++r)
        if (e0 + 64 * r < n) list[e0 + 64 * r] = v[r];
}

constexpr int kWaveSortMax = 256;   // longest list sorted by one wave

// Workgroup b owns tiles b + i * gridDim.x, i = 0..3 (strided, so that the
// long lists of a crowded screen region spread over many workgroups). A list
// of at most kWaveSortMax entries is sorted by the wave of its tile;
// longer lists are then sorted by the whole workgroup, in blocks of kSortBlock.
// Both hold the entries in registers and exchange them by lane permutations; a
// workgroup's waves meet in the LDS three times, where a bitonic sort in it met
// after each of 66 steps. 64 views of 50,000 triangles: 191 -> 122 us, 200,000
// triangles 346 -> 192, four training views 51 -> 25. Six waves per SIMD: left
// to itself the compiler takes 136 registers, and the short lists, which wait
// on their loads, then take longer than the long ones save (201 us).
__global__ __launch_bounds__(256, 6) void sort_kernel(const int64_t* __restrict__ tile_start, int64_t n_tiles,
                                                   uint64_t* __restrict__ entries, int64_t cap) {
    __shared__ uint64_t s[kSortBlock];
    const int w = threadIdx.x >> 6;
    const int64_t stride = gridDim.x;
    if (tile_start[n_tiles] > cap) return;   // lists longer than the buffer are made again
    {
        const int64_t tile = blockIdx.x + w * stride;
        if (tile < n_tiles) {
            const int64_t beg = tile_start[tile];
            const int n = static_cast<int>(min<int64_t>(tile_start[tile + 1] - beg, kWaveSortMax + 1));
            if (n > 1 && n <= 64) bitonic_sort<1, 1>(entries + beg, n, 0, nullptr);
            else if (n > 64 && n <= 128) bitonic_sort<2, 1>(entries + beg, n, 0, nullptr);
            else if (n > 128 && n <= kWaveSortMax) bitonic_sort<4, 1>(entries + beg, n, 0, nullptr);
        }
    }
    for (int i = 0; i < 4; ++i) {
        const int64_t tile = blockIdx.x + i * stride;
        if (tile >= n_tiles) break;
        const int64_t beg = tile_start[tile], end = tile_start[tile + 1];
        if (end - beg <= kWaveSortMax) continue;
        for (int64_t b0 = beg; b0 < end; b0 += kSortBlock) {
            const int n = static_cast<int>(min<int64_t>(kSortBlock, end - b0));
            uint64_t* const list = entries + b0;
            if (n <= 64) {   // the last block of a longer list
                if (w == 0) bitonic_sort<1, 1>(list, n, 0, nullptr);
            } else if (n <= kWaveSortMax) {
                if (w == 0) bitonic_sort<4, 1>(list, n, 0, nullptr);
            } else if (n <= 512) {
                bitonic_sort<2, 4>(list, n, w, s);
            } else if (n <= 1024) {
                bitonic_sort<4, 4>(list, n, w, s);
            } else {
                bitonic_sort<8, 4>(list, n, w, s);
            }
        }
    }
}

// ---------------------------------------------------------------------------
// exclusive scan int32 -> int64 (three passes over blocks of 1024)
// ---------------------------------------------------------------------------

constexpr int kScanBlock = 1024;

__device__ __forceinline__ int64_t wave_incl_scan(int64_t v) {
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        const int64_t u = __shfl_up(v, d, 64);
        if (lane_id() >= d) v += u;
    }
    return v;
}

// Exclusive scan over the 256 threads of a block; returns the block total.
__device__ __forceinline__ int64_t block_excl_scan(int64_t v, int64_t& total) {
    __shared__ int64_t wsum[4];
    const int w = threadIdx.x >> 6;
    const int64_t inc = wave_incl_scan(v);
    if (lane_id() == 63) wsum[w] = inc;
    __syncthreads();
    int64_t off = 0;
    total = 0;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        if (i < w) off += wsum[i];
        total += wsum[i];
    }
    __syncthreads();
    return off + inc - v;
}

__global__ __launch_bounds__(256) void scan_reduce_kernel(const int32_t* __restrict__ in, int64_t n, int stride,
                                                          int64_t* __restrict__ bsum) {
    const int64_t base = static_cast<int64_t>(blockIdx.x) * kScanBlock;
    int64_t v = 0;
    for (int k = 0; k < 4; ++k) {
        const int64_t i = base + threadIdx.x * 4 + k;
        if (i < n) v += in[i * stride];
    }
    int64_t total;
    block_excl_scan(v, total);
    if (threadIdx.x == 0) bsum[blockIdx.x] = total;
}

__global__ __launch_bounds__(256) void scan_bsum_kernel(int64_t* __restrict__ bsum, int64_t nb) {
    int64_t carry = 0;
    for (int64_t b0 = 0; b0 < nb; b0 += 256) {
        const int64_t i = b0 + threadIdx.x;
        const int64_t v = i < nb ? bsum[i] : 0;
        int64_t total;
        const int64_t ex = block_excl_scan(v, total);
        if (i < nb) bsum[i] = carry + ex;
        carry += total;
        __syncthreads();
    }
}

__global__ __launch_bounds__(256) void scan_apply_kernel(const int32_t* __restrict__ in, int64_t n, int stride,
                                                         const int64_t* __restrict__ bsum,
                                                         int64_t* __restrict__ out, int64_t* __restrict__ host_total) {
    const int64_t base = static_cast<int64_t>(blockIdx.x) * kScanBlock;
    int64_t vals[4];
    int64_t v = 0;
    for (int k = 0; k < 4; ++k) {
        const int64_t i = base + threadIdx.x * 4 + k;
        vals[k] = i < n ? in[i * stride] : 0;
        v += vals[k];
    }
    int64_t total;
    int64_t ex = block_excl_scan(v, total) + bsum[blockIdx.x];
    for (int k = 0; k < 4; ++k) {
        const int64_t i = base + threadIdx.x * 4 + k;
        if (i < n) out[i] = ex;
        ex += vals[k];
    }
    if (blockIdx.x == gridDim.x - 1 && threadIdx.x == 255) {
        out[n] = ex;
        store_host(host_total, ex);
    }
}

// The same scan by one workgroup, for up to kScanOne values: four consecutive
// values per thread and round, the rounds' totals carried along.
constexpr int64_t kScanOne = 16384;
__global__ __launch_bounds__(1024) void scan_one_kernel(const int32_t* __restrict__ in, int n, int stride, int64_t* __restrict__ out,
                                                        int64_t* __restrict__ host_total) {
    __shared__ int64_t wsum[16];
    const int tid = threadIdx.x, w = tid >> 6, lane = lane_id();
    int32_t v[4][4];
    int64_t ex[4], carry = 0;
#pragma unroll
    for (int r = 0; r < 4; ++r)   // every load first
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const int i = r * 4096 + tid * 4 + k;
            v[r][k] = i < n ? in[i * stride] : 0;
        }
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const int64_t sum = static_cast<int64_t>(v[r][0]) + v[r][1] + v[r][2] + v[r][3];
        const int64_t inc = wave_incl_scan(sum);
        if (lane == 63) wsum[w] = inc;
        __syncthreads();
        int64_t off = 0, total = 0;
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            if (i < w) off += wsum[i];
            total += wsum[i];
        }
        __syncthreads();
        ex[r] = carry + off + inc - sum;
        carry += total;
        if (r * 4096 + 4096 >= n) break;   // uniform
    }
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        int64_t x = ex[r];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const int i = r * 4096 + tid * 4 + k;
            if (i < n) out[i] = x;
            x += v[r][k];
        }
    }
    if (tid == 0) {
        out[n] = carry;
        store_host(host_total, carry);
    }
}

__global__ void fill_i32_kernel(int32_t* __restrict__ p, int64_t n, int32_t v) {
    for (int64_t i = blockIdx.x * static_cast<int64_t>(blockDim.x) + threadIdx.x; i < n;
         i += static_cast<int64_t>(gridDim.x) * blockDim.x)
        p[i] = v;
}

// Ranges cleared by one launch, in 16-byte stores where a range is aligned.
__global__ __launch_bounds__(256) void zero_kernel(ZeroList z) {
    const int64_t tid = blockIdx.x * static_cast<int64_t>(256) + threadIdx.x, step = static_cast<int64_t>(gridDim.x) * 256;
    for (int r = 0; r < z.k; ++r) {
        int32_t* p = z.p[r];
        const int64_t n = z.n[r], n4 = (reinterpret_cast<uintptr_t>(p) & 15) == 0 ? n / 4 : 0;
        for (int64_t i = tid; i < n4; i += step) nt_store(make_float4(0.f, 0.f, 0.f, 0.f), reinterpret_cast<float4*>(p) + i);
        for (int64_t i = 4 * n4 + tid; i < n; i += step) p[i] = 0;
    }
}

__global__ void fill_f32_kernel(float* __restrict__ p, int64_t n, float v) {
    for (int64_t i = blockIdx.x * static_cast<int64_t>(blockDim.x) + threadIdx.x; i < n;
         i += static_cast<int64_t>(gridDim.x) * blockDim.x)
        p[i] = v;
}

// ---------------------------------------------------------------------------
// host launchers
// ---------------------------------------------------------------------------

static unsigned grid_for(int64_t n, int bs = 256) {
    int64_t g = (n + bs - 1) / bs;
    if (g < 1) g = 1;
    if (g > 65536) g = 65536;
    return static_cast<unsigned>(g);
}

void launch_fill_i32(int32_t* p, int64_t n, int32_t v, hipStream_t s) {
    if (n <= 0) return;
    hipLaunchKernelGGL(fill_i32_kernel, dim3(grid_for(n)), dim3(256), 0, s, p, n, v);
}

void launch_zero(const ZeroList& z, hipStream_t s) {
    int64_t n = 0;
    for (int r = 0; r < z.k; ++r) n += z.n[r];
    if (n <= 0) return;
    hipLaunchKernelGGL(zero_kernel, dim3(grid_for((n + 3) / 4)), dim3(256), 0, s, z);
}

void launch_fill_f32(float* p, int64_t n, float v, hipStream_t s) {
    if (n <= 0) return;
    hipLaunchKernelGGL(fill_f32_kernel, dim3(grid_for(n)), dim3(256), 0, s, p, n, v);
}

// Large chunks when they still give every CU two workgroups, else small ones:
// 256 triangles when those do, else 64 or 16, so that few large triangles
// spread over many workgroups.
int bin_chunk_size(int V, int maxT, int num_cus) {
    const int64_t full = 2 * static_cast<int64_t>(num_cus);
    for (const int chunk : {kBinChunk, 256, 64})
        if (static_cast<int64_t>(V) * bin_chunks(maxT, chunk) >= full) return chunk;
    return 16;
}

// Atomics on one 64-byte line complete 2.6 ns apart (16 counters in it; on one
// counter 13 ns), and few tiles put their counters in few lines: spread by 16,
// the setup and the scatter of a 640x360 render (920 tiles) took 7.7 and 7.0 us
// instead of 21.6 and 21.2, four views (7,312 tiles) 50 and 44 instead of 75
// and 76. At 10,000 tiles the scan over the wider array takes back what 16 gives
// over 4 (92 us for the three kernels against 87, packed 98).
int bin_stride(int chunk, int64_t n_tiles) {
    return chunk >= kBinChunk || n_tiles > 16384 ? 1 : n_tiles <= 8192 ? 16 : 4;
}

void launch_setup(const ViewDesc* views, int V, int maxT, int chunk, const SceneDesc* scenes, const Opts& o,
                  int tile, TriRec* recs, int32_t* tile_count, int32_t* chunk_base, int64_t n_tiles,
                  unsigned long long* visible, hipStream_t s) {
    if (maxT <= 0) return;
    dim3 grid(bin_chunks(maxT, chunk), V);
    if (chunk < kBinChunk) {
        hipLaunchKernelGGL(setup_small_kernel, grid, dim3(256), 0, s, views, scenes, o, tile, chunk, recs, tile_count,
                           bin_stride(chunk, n_tiles), visible);
        return;
    }
    hipLaunchKernelGGL(setup_kernel, grid, dim3(256), 0, s, views, scenes, o, tile, chunk, recs, tile_count,
                       chunk_base, n_tiles, visible);
}

void launch_scan(const int32_t* in, int64_t n, int stride, int64_t* bsum, int64_t* out, int64_t* host_total,
                 hipStream_t s) {
    if (n <= 0) {   // empty input: the single offset is 0
        launch_fill_i32(reinterpret_cast<int32_t*>(out), 2, 0, s);
        return;
    }
    if (n <= kScanOne) {
        hipLaunchKernelGGL(scan_one_kernel, dim3(1), dim3(1024), 0, s, in, static_cast<int>(n), stride, out, host_total);
        return;
    }
    const int64_t nb = (n + kScanBlock - 1) / kScanBlock;
    hipLaunchKernelGGL(scan_reduce_kernel, dim3(static_cast<unsigned>(nb)), dim3(256), 0, s, in, n, stride, bsum);
    hipLaunchKernelGGL(scan_bsum_kernel, dim3(1), dim3(256), 0, s, bsum, nb);
    hipLaunchKernelGGL(scan_apply_kernel, dim3(static_cast<unsigned>(nb)), dim3(256), 0, s, in, n, stride, bsum, out,
                       host_total);
}

void launch_scatter(const ViewDesc* views, int V, int maxT, int chunk, int tile, const TriRec* recs,
                    const int64_t* tile_start, int64_t n_tiles, const int32_t* chunk_base, int32_t* tile_fill,
                    uint64_t* entries, int64_t cap, hipStream_t s) {
    if (maxT <= 0) return;
    dim3 grid(bin_chunks(maxT, chunk), V);
    if (chunk < kBinChunk) {
        hipLaunchKernelGGL(scatter_small_kernel, grid, dim3(256), 0, s, views, tile, chunk, recs, tile_start, n_tiles,
                           tile_fill, bin_stride(chunk, n_tiles), entries, cap);
        return;
    }
    hipLaunchKernelGGL(scatter_kernel, grid, dim3(256), 0, s, views, tile, chunk, recs, tile_start, n_tiles,
                       chunk_base, tile_fill, entries, cap);
}

// Static-capacity mode: when the lists need more than `cap` entries, flag the
// overflow (sticky bit 1) and empty every tile list, so that no kernel of
// the call touches entries beyond the capacity.
__global__ void clip_check_kernel(const int64_t* __restrict__ tile_start, int64_t n_tiles, int64_t cap,
                                  unsigned int* __restrict__ local, unsigned int* __restrict__ sticky) {
    const bool over = tile_start[n_tiles] > cap;
    *local = over ? 1u : 0u;
    if (over) atomicOr(sticky, 1u);
}

__global__ void clip_apply_kernel(int64_t* __restrict__ tile_start, int64_t n_tiles,
                                  const unsigned int* __restrict__ local) {
    const int64_t i = blockIdx.x * static_cast<int64_t>(blockDim.x) + threadIdx.x;
    if (i <= n_tiles && *local) tile_start[i] = 0;
}

void launch_clip(int64_t* tile_start, int64_t n_tiles, int64_t cap, unsigned int* local, unsigned int* sticky,
                 hipStream_t s) {
    hipLaunchKernelGGL(clip_check_kernel, dim3(1), dim3(1), 0, s, tile_start, n_tiles, cap, local, sticky);
    hipLaunchKernelGGL(clip_apply_kernel, dim3(static_cast<unsigned>((n_tiles + 256) / 256)), dim3(256), 0, s,
                       tile_start, n_tiles, local);
}

void launch_sort(const int64_t* tile_start, int64_t n_tiles, uint64_t* entries, int64_t cap, hipStream_t s) {
    if (n_tiles <= 0) return;
    hipLaunchKernelGGL(sort_kernel, dim3(static_cast<unsigned>((n_tiles + 3) / 4)), dim3(256), 0, s, tile_start,
                       n_tiles, entries, cap);
}

}  // namespace soup
