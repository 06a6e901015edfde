#pragma once
// The forward's MLP decode of a 64-fragment batch on the matrix cores, in the
// contract's float32 sequence.
//
// v_mfma_f32_32x32x2f32 evaluates D = fma(A[.][1], B[1][.], fma(A[.][0],
// B[0][.], C)), one rounding per step, denormals kept, bit for bit as two
// fmaf (checked on gfx950 over normal, tiny, denormal and arbitrary bit
// patterns). Steps over input pairs (2m, 2m + 1), m ascending, are therefore
// exactly the contract's chain h = b; h = fma(W[j][k], x[k], h), k ascending.
//
// Operand layout (lane l, half h = l >> 5): the lane supplies A[l & 31][h] and
// B[h][l & 31] and holds D[8 (r >> 2) + 4 h + (r & 3)][l & 31] in register r.
// The weights' rows are ordered so that register r of half h is unit
// 32 rb + 2 r + h of row block rb: register r of one layer's D is then the B
// operand of step 16 rb + r of the next layer, and nothing moves between
// layers. Fragments 0..31 and 32..63 of the batch are two column blocks; one
// half swap per input pair takes the lanes' own features (lane = fragment) to
// their operands. The output layer runs on v_mfma_f32_4x4x1f32 (sixteen blocks
// of four lanes: lane = fragment in and out), after one half swap per unit
// pair back.
//
// What bounds it: 64 fragments of 16->32->32->4 are 48 products of 64 cycles
// and 32 of 8, 3.3 k cycles of a SIMD's matrix pipe, where the same chain on
// the vector ALU was 1,664 instructions of 4 cycles (6.7 k). (The walk's vector
// work of the SIMD's other waves does not run beside the products: float32
// matrix and vector instructions take turns.) The weights are laid out as A operands once per call and
// read by 16-byte loads, four steps each: a wave keeps those of 16->32->32->4
// in registers while it stays with one scene and reads the 26 KB of
// 32->64->64->4 from the caches. Forward kernels before and now: 64 views,
// 50,000 triangles, 2.23 -> 1.83 ms; 16 views 1080p, 200,000 triangles,
// 32->64->64->4, 5.49 -> 3.87 ms; 16 serving requests 1.32 -> 1.14 ms.
#include "decode_mfma.hpp"

namespace soup {

typedef float f16v __attribute__((ext_vector_type(16)));

// The weights of one scene as A operands (16-byte groups, offsets in groups).
template <class S>
struct FwdWeights {
    static constexpr bool kMfma = S::H >= 32;   // 8->16->4 fills half a product's rows: vector ALU
    static constexpr int NB = S::H / 32;               // row blocks
    static constexpr int J0 = S::C / 8, J1 = S::H / 8; // groups of four steps per row block
    static constexpr int kW0 = 0;                      // [rb][j][64]: step 4 j + e: W0[32 rb + u(l & 31)][2 (4 j + e) + h]
    static constexpr int kW1 = kW0 + NB * J0 * 64;     // [rb][j][64]
    static constexpr int kWo = kW1 + NB * J1 * 64;     // [t][4]: W_out[l & 3][4 t + e]
    static constexpr int kB0 = kWo + S::H;             // [rb][h][4]: register 4 i + e: b0[32 rb + 2 (4 i + e) + h]
    static constexpr int kB1 = kB0 + NB * 8;
    static constexpr int kBo = kB1 + NB * 8;           // b_out
    static constexpr int kGroups = kBo + 1;
    static_assert(!kMfma || S::NH == 2, "two hidden layers");
    // One row block: a wave keeps both hidden layers' operands in registers
    // (24 for 16->32->32->4) and the groups from kWo on in its LDS; read again for
    // every batch, their latency was a third of the wave's time (the forward of 64
    // views, 50,000 triangles: 2.08 ms against 1.83). Two row blocks (96 registers)
    // are read from the caches.
    static constexpr bool kRegs = kMfma && NB == 1;
    static constexpr int kLds = kRegs ? kGroups - kWo : 1;   // groups a wave keeps in LDS

    // the flat parameter index of element e of group g
    __device__ static int source(int g, int e) {
        const bool l1 = g >= kW1;
        if (g < kWo) {
            const int q = l1 ? g - kW1 : g, J = l1 ? J1 : J0;
            const int l = q & 63, j = (q >> 6) % J, rb = (q >> 6) / J;
            const int row = l & 31, unit = 8 * (row >> 3) + 2 * (row & 3) + ((row >> 2) & 1);
            return S::w_off(l1 ? 1 : 0) + (32 * rb + unit) * S::din(l1 ? 1 : 0) + 2 * (4 * j + e) + (l >> 5);
        }
        if (g < kB0) return S::w_off(2) + ((g - kWo) & 3) * S::H + 4 * ((g - kWo) >> 2) + e;
        if (g < kBo) {
            const int q = (g - kB0) % (NB * 8), rb = q >> 3, h = (q >> 2) & 1, i = q & 3;
            return S::b_off(g < kB1 ? 0 : 1) + 32 * rb + 2 * (4 * i + e) + h;
        }
        return S::b_off(2) + e;
    }
};

// The operand groups in global memory: through a generic pointer they were flat
// loads, whose waits are for all of them (and for the LDS) at once (200,000
// triangles, 32-64-64-4: forward 3.23 -> 3.17 ms).
#if defined(__HIP_DEVICE_COMPILE__)
using gf4v = const f4v __attribute__((address_space(1)));
#else
using gf4v = const f4v;
#endif
__device__ __forceinline__ gf4v* as_gf4v(const f4v* p) { return reinterpret_cast<gf4v*>(reinterpret_cast<uintptr_t>(p)); }

// A wave's copy of its scene's weights.
template <class S>
struct FwdRegs {
    f4v w0[FwdWeights<S>::kRegs ? FwdWeights<S>::J0 : 1], w1[FwdWeights<S>::kRegs ? FwdWeights<S>::J1 : 1];
    __device__ __forceinline__ void load(gf4v* __restrict__ wg, f4v* __restrict__ lds, int lane) {
        using FW = FwdWeights<S>;
        static_assert(FW::kLds <= 64, "one group per lane");
#pragma unroll
        for (int j = 0; j < FW::J0; ++j) w0[j] = wg[FW::kW0 + j * 64 + lane];
#pragma unroll
        for (int j = 0; j < FW::J1; ++j) w1[j] = wg[FW::kW1 + j * 64 + lane];
        if (lane < FW::kLds) lds[lane] = wg[FW::kWo + lane];
        wave_fence();
    }
};

__device__ __forceinline__ f16v mfma32(float a, float b, const f16v& c) {
    return __builtin_amdgcn_mfma_f32_32x32x2f32(a, b, c, 0, 0, 0);
}

// The accumulators of one row block, started at its biases.
template <class P>
__device__ __forceinline__ f16v bias16(P* __restrict__ b) {
    f16v d;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const f4v v = b[i];
#pragma unroll
        for (int e = 0; e < 4; ++e) d[4 * i + e] = v[e];
    }
    return d;
}

__device__ __forceinline__ void relu16(f16v& d, float inf) {
#pragma unroll
    for (int r = 0; r < 16; ++r) d[r] = relu(d[r], inf);
}

// Logits of the wave's 64 fragments (lane = fragment; every lane takes part).
// wl: the groups from kWo on (the wave's LDS where the layers have one row block).
// Two product chains run side by side: the two column blocks where the layers
// have one row block (they share the weights), the two row blocks otherwise
// (they share the activations).
template <class S, class P>
__device__ __forceinline__ void mfma_logits(const FwdRegs<S>& wr, gf4v* __restrict__ wg,
                                            P* __restrict__ wl, const float (&x)[S::C], float (&o)[4],
                                            int lane) {
    using FW = FwdWeights<S>;
    constexpr int NB = FW::NB;
    const float inf = opaque_inf();
    gf4v* __restrict__ w = wg + lane;
    P* __restrict__ bh = wl - FW::kWo + 4 * (lane >> 5);
    float xs[2][S::C / 2];   // per column block: inputs 2m (lanes 0..31) and 2m + 1 (lanes 32..63)
#pragma unroll
    for (int m = 0; m < S::C / 2; ++m) {
        const U2 q = swap32(__float_as_uint(x[2 * m]), __float_as_uint(x[2 * m + 1]));
        xs[0][m] = __uint_as_float(q.a);
        xs[1][m] = __uint_as_float(q.b);
    }
    f16v h2[2][NB];          // [column block][row block]
    if constexpr (NB == 1) {
        f16v d0 = bias16(bh + FW::kB0), d1 = d0;
#pragma unroll
        for (int j = 0; j < FW::J0; ++j) {
            const f4v a = wr.w0[j];
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                d0 = mfma32(a[e], xs[0][4 * j + e], d0);
                d1 = mfma32(a[e], xs[1][4 * j + e], d1);
            }
        }
        relu16(d0, inf);
        relu16(d1, inf);
        f16v e0 = bias16(bh + FW::kB1), e1 = e0;
#pragma unroll
        for (int j = 0; j < FW::J1; ++j) {
            const f4v a = wr.w1[j];
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                e0 = mfma32(a[e], d0[4 * j + e], e0);
                e1 = mfma32(a[e], d1[4 * j + e], e1);
            }
        }
        h2[0][0] = e0;
        h2[1][0] = e1;
    } else {
        static_assert(NB <= 2, "one or two row blocks");
#pragma unroll
        for (int cb = 0; cb < 2; ++cb) {
            f16v d[2] = {bias16(bh + FW::kB0), bias16(bh + FW::kB0 + 8)};
#pragma unroll
            for (int j = 0; j < FW::J0; ++j) {
                const f4v a0 = w[FW::kW0 + j * 64], a1 = w[FW::kW0 + (FW::J0 + j) * 64];
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    d[0] = mfma32(a0[e], xs[cb][4 * j + e], d[0]);
                    d[1] = mfma32(a1[e], xs[cb][4 * j + e], d[1]);
                }
            }
            relu16(d[0], inf);
            relu16(d[1], inf);
            f16v e0 = bias16(bh + FW::kB1), e1 = bias16(bh + FW::kB1 + 8);
#pragma unroll
            for (int j = 0; j < FW::J1; ++j) {
                const f4v a0 = w[FW::kW1 + j * 64], a1 = w[FW::kW1 + (FW::J1 + j) * 64];
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const float b = d[j >> 2][4 * (j & 3) + e];
                    e0 = mfma32(a0[e], b, e0);
                    e1 = mfma32(a1[e], b, e1);
                }
            }
            h2[cb][0] = e0;
            h2[cb][NB - 1] = e1;
        }
    }
    f4v out = wl[FW::kBo - FW::kWo];
#pragma unroll
    for (int rb = 0; rb < NB; ++rb) {
        relu16(h2[0][rb], inf);
        relu16(h2[1][rb], inf);
#pragma unroll
        for (int t = 0; t < 8; ++t) {   // units 32 rb + 4 t .. + 3
            const f4v a = wl[4 * (8 * rb + t) + (lane & 3)];
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                const U2 q = swap32(__float_as_uint(h2[0][rb][2 * t + i]), __float_as_uint(h2[1][rb][2 * t + i]));
                out = mfma4x4(a[2 * i], __uint_as_float(q.a), out);
                out = mfma4x4(a[2 * i + 1], __uint_as_float(q.b), out);
            }
        }
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) o[i] = out[i];
}

}  // namespace soup
