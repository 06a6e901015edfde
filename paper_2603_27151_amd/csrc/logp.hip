// log p(f*) of Eq. (6) per pixel: the sum of log(1 - alpha) over the fragments
// in front of the winner and log(alpha) of the winner, from the forward's log
// (one fragment per lane, the decode of the forward, atomics per pixel).
#include "fwd_mfma.hpp"

namespace soup {

template <class S>
__global__ __launch_bounds__(256) void logp_kernel(FragLogView L, FragSelect sel, const float* __restrict__ feats_p,
                                                   const float* __restrict__ mlp, const float* __restrict__ weights,
                                                   int G, float* __restrict__ logp) {
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    gfloat* feats = as_global(uniform_ptr(feats_p));
    __shared__ f4v s_w[4][FwdWeights<S>::kLds];
    FwdRegs<S> wregs;
    gf4v* wops = as_gf4v(reinterpret_cast<const f4v*>(weights));
    if constexpr (FwdWeights<S>::kRegs) wregs.load(wops, s_w[w], lane);
    for_log_batches(L, [&](uint32_t r, uint32_t b, uint32_t n) {
        const uint64_t at = static_cast<uint64_t>(r) * L.region + b + lane;
        uint4 e = make_uint4(0u, 0u, 0u, 0u);
        bool keep = false, win = false;
        if (b + lane < n) {
            e = L.frag[at];
            sel.decide(e, keep, win);
        }
        if (__ballot(keep) == 0) return;
        float x[S::C], o[4];
#pragma unroll
        for (int k = 0; k < S::C; ++k) x[k] = 0.0f;
        if (keep) {
            const uint2 bc = L.bary[at];
            fetch_feature<S::C>(feats, e.y, G, cell_of(__uint_as_float(bc.x), __uint_as_float(bc.y), G), x);
        }
        // opaque copies of the weight pointers per batch: the compiler may not hoist
        // the weights' loads out of the batch loop
        if constexpr (FwdWeights<S>::kMfma) {
            gf4v* wg = as_gf4v(opaque_ptr(reinterpret_cast<const f4v*>(weights)));
            if constexpr (FwdWeights<S>::kRegs) mfma_logits<S>(wregs, wg, s_w[w], x, o, lane);
            else mfma_logits<S>(wregs, wg, wg + FwdWeights<S>::kWo, x, o, lane);
        } else {
            mlp_logits<S>(as_const(opaque_ptr(mlp)), x, o);
        }
        const float alpha = sigmoid_c(o[3]);
        if (keep) atomicAdd(&logp[e.x], win ? logf(alpha) : log1pf(-alpha));
    });
}

template <class S>
static void launch_logp_s(const LogpArgs& a, hipStream_t s) {
    hipLaunchKernelGGL(logp_kernel<S>, dim3(log_blocks(a.log)), dim3(256), 0, s, a.log, a.sel, a.feats, a.mlp,
                       a.weights, a.G, a.logp);
}

void launch_logp(const LogpArgs& a, MlpKind k, hipStream_t s) {
    switch (k) {
        case MlpKind::k8_16_1: launch_logp_s<MlpShape<8, 16, 1>>(a, s); break;
        case MlpKind::k16_32_2: launch_logp_s<MlpShape<16, 32, 2>>(a, s); break;
        case MlpKind::k32_64_2: launch_logp_s<MlpShape<32, 64, 2>>(a, s); break;
        default: break;
    }
}

}  // namespace soup
