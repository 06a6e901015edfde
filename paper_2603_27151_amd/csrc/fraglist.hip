// Backward, part 1 (Supplement Algorithm A1, part 2): the fragments the
// backward needs -- the winner of each pixel and, where the pixel carries a
// score weight, every fragment in front of it (Eq. (9)) -- sorted by triangle.
//
// They come from a log with one region per wave of the raster that wrote it:
// the forward's, which holds every fragment it decoded (every fragment with key
// <= the winner's was, since the forward's best key never falls below the
// winner's), or that of a raster walk with the winners known (a backward
// without the forward's log). count_kernel decides what is kept (two 64-bit
// masks per 64 entries) and counts per triangle; after a scan, place_kernel
// writes the kept fragments to their places. The log is read twice and the
// list written once: a filtered copy between the two would be written and read
// again (64 views of 50,000 triangles: 0.51 ms for the two kernels, 0.58 with it).
#include "internal.hpp"

namespace soup {

// Total and largest region count of a log; an overflow sets kOverflowFragments in
// *sticky (when not null). One workgroup, n <= kMaxRegions.
__global__ __launch_bounds__(1024) void log_summary_kernel(const uint32_t* __restrict__ counts, int n, uint32_t region,
                                                           unsigned long long* __restrict__ summary,
                                                           unsigned int* __restrict__ sticky) {
    __shared__ unsigned long long s_tot[16];
    __shared__ uint32_t s_max[16];
    const int t = threadIdx.x;
    unsigned long long tot = 0;
    uint32_t mx = 0;
#pragma unroll
    for (int i = 0; i < kMaxRegions / 1024; ++i) {
        const int r = i * 1024 + t;
        const uint32_t c = r < n ? counts[r] : 0u;
        tot += c;
        mx = c > mx ? c : mx;
    }
#pragma unroll
    for (int d = 32; d > 0; d >>= 1) {
        tot += __shfl_xor(tot, d, 64);
        const uint32_t m = __shfl_xor(mx, d, 64);
        mx = m > mx ? m : mx;
    }
    if ((t & 63) == 0) {
        s_tot[t >> 6] = tot;
        s_max[t >> 6] = mx;
    }
    __syncthreads();
    if (t == 0) {
        for (int i = 1; i < 16; ++i) {
            tot += s_tot[i];
            mx = s_max[i] > mx ? s_max[i] : mx;
        }
        if (summary) {
            store_host(&summary[0], tot);
            store_host(&summary[1], static_cast<unsigned long long>(mx));
        }
        if (sticky && mx > region) atomicOr(sticky, kOverflowFragments);
    }
}

void launch_log_summary(const uint32_t* counts, int n, uint32_t region, unsigned long long* summary,
                        unsigned int* sticky, hipStream_t s) {
    hipLaunchKernelGGL(log_summary_kernel, dim3(1), dim3(1024), 0, s, counts, n, region, summary, sticky);
}

__global__ __launch_bounds__(256) void count_kernel(FragLogView L, FragSelect sel, ulonglong2* __restrict__ masks,
                                                    int32_t* __restrict__ tri_count) {
    const int lane = threadIdx.x & 63;
    const uint32_t slots = log_slots(L.region);
    for_log_batches(L, [&](uint32_t r, uint32_t b, uint32_t n) {
        const uint64_t at = static_cast<uint64_t>(r) * L.region + b + lane;
        uint32_t tri = 0xFFFFFFFFu;
        bool keep = false, win = false;
        if (b + lane < n) {
            const uint4 e = L.frag[at];
            tri = e.y;
            sel.decide(e, keep, win);
        }
        const uint64_t km = __ballot(keep), wm = __ballot(win);
        if (lane == 0) masks[static_cast<uint64_t>(r) * slots + b / 64] = make_ulonglong2(km, wm);
        // one atomic per run of equal triangles among consecutive lanes
        const uint32_t tp = __shfl_up(tri, 1, 64);
        const bool head = lane == 0 || tp != tri;
        const uint64_t heads = __ballot(head);
        if (head && tri != 0xFFFFFFFFu) {
            const int k = __popcll(km & run_of(heads, lane));
            if (k) atomicAdd(&tri_count[tri], k);
        }
    });
}

void launch_count(const FragLogView& L, const FragSelect& sel, ulonglong2* masks, int32_t* tri_count, hipStream_t s) {
    hipLaunchKernelGGL(count_kernel, dim3(log_blocks(L)), dim3(256), 0, s, L, sel, masks, tri_count);
}

// Triangle t's winners go to sorted[tri_off[t] + k] and its other fragments to
// sorted[tri_off[t + 1] - 1 - k], k from a per-triangle pair of fill counters
// (one 64-bit atomic per run of equal triangles among consecutive lanes), so
// that most 64-fragment batches of the decode hold winners only or none.
__global__ __launch_bounds__(256) void place_kernel(FragLogView L, const float* __restrict__ grad_logp,
                                                    const ulonglong2* __restrict__ masks,
                                                    const int64_t* __restrict__ tri_off,
                                                    unsigned long long* __restrict__ tri_fill,
                                                    FragRec* __restrict__ sorted) {
    const int lane = threadIdx.x & 63;
    const uint32_t slots = log_slots(L.region);
    for_log_batches(L, [&](uint32_t r, uint32_t b, uint32_t n) {
        const ulonglong2 m = masks[static_cast<uint64_t>(r) * slots + b / 64];
        const uint64_t km = m.x, wm = m.y;
        const uint64_t at = static_cast<uint64_t>(r) * L.region + b + lane;
        const bool keep = (km >> lane) & 1u, win = (wm >> lane) & 1u;
        uint4 e = make_uint4(0u, 0xFFFFFFFFu, 0u, 0u);
        uint2 bc = make_uint2(0u, 0u);
        float gl = 0.0f;
        if (b + lane < n) e = nt_load(L.frag + at);
        if (keep) {
            bc = nt_load(L.bary + at);
            if (grad_logp) gl = grad_logp[e.x];
        }
        const uint32_t tri = e.y;
        const uint32_t tp = __shfl_up(tri, 1, 64);
        const bool head = lane == 0 || tp != tri;
        const uint64_t heads = __ballot(head);
        const uint64_t run = run_of(heads, 63 - __builtin_clzll(heads & upto_mask(lane)));   // this lane's run
        const int hl = __builtin_ctzll(run);
        unsigned long long base = 0;
        if (head) {
            const unsigned long long nw = static_cast<unsigned long long>(__popcll(wm & run));
            const unsigned long long nf = static_cast<unsigned long long>(__popcll(km & run)) - nw;
            if (nw | nf) base = atomicAdd(&tri_fill[tri], nw | (nf << 32));
        }
        const unsigned long long hb = __shfl(base, hl, 64);
        if (keep) {
            const uint64_t before = run & lanemask_lt();
            const int w_before = __popcll(wm & before), k_before = __popcll(km & before);
            const int64_t dst = win ? tri_off[tri] + static_cast<int64_t>(hb & 0xFFFFFFFFull) + w_before
                                    : tri_off[tri + 1] - 1 - static_cast<int64_t>(hb >> 32) - (k_before - w_before);
            FragRec fr;
            fr.p0 = make_uint2(e.x, tri | (win ? 0x80000000u : 0u));
            fr.p1 = bc;
            fr.x = make_uint2(__float_as_uint(gl), e.w);
            sorted[dst] = fr;
        }
    });
}

void launch_place(const FragLogView& L, const float* grad_logp, const ulonglong2* masks, const int64_t* tri_off,
                  unsigned long long* tri_fill, FragRec* sorted, hipStream_t s) {
    hipLaunchKernelGGL(place_kernel, dim3(log_blocks(L)), dim3(256), 0, s, L, grad_logp, masks, tri_off, tri_fill,
                       sorted);
}

}  // namespace soup
