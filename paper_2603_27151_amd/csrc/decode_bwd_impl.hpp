#pragma once
// Backward, part 2 (Supplement Algorithm A1, part 2; Eq. (8), (9)): decode of
// the fragment list.
//
// The backward walks the fragment list sorted by triangle: every wave takes a
// contiguous range of 64-fragment batches. For each batch:
//   - recompute the bilinear feature and the MLP (the forward's float32
//     sequence, so its hidden layers and ReLU decisions are the forward's);
//   - logit gradients: winner -> colour path g_C sigma'(o_rgb) and score
//     g_L (1 - alpha); fragment in front -> score -g_L alpha (Eq. (9) through
//     the sigmoid);
//   - back-propagate through the MLP; the weight gradient sum_f delta_f a_f^T
//     runs on the matrix cores over the batch (activations and deltas staged
//     through LDS); each wave writes its sums once, at the end, to its own row
//     of a partial-sum buffer (rows are reduced later in a fixed order);
//   - for the winner, the gradient of its triangle's world-space vertices
//     from its colour logits only (the score term moves no vertex, Section
//     3.2): the feature gradient of the colour logits (a second data backward
//     where the winner also carries a score weight) dotted with the texture's
//     derivative along the cell position, then through the perspective-
//     correct and screen barycentrics, the screen positions and 1/w, and the
//     view-projection; the edge term of Section 3.2 (the pixel's edge weights
//     times its screen barycentrics) joins it in screen space;
//   - the feature gradient (bilinear weights of the four texels) and the
//     vertex gradient are summed into the wave's LDS copy of the current
//     triangle's G x G x C grid; when the triangle changes, the grid goes to
//     HBM once (a plain store when the wave holds all of the triangle's
//     fragments, float atomics for a triangle split between waves).
//
// What bounds it: the products themselves and the vector instructions between
// them. A SIMD's float32 matrix and vector instructions take turns, also where
// they come from two waves (a wave of products beside a wave of fused
// multiply-adds took 447 us where each alone took 228 and 237), so a batch costs
// the sum of both: the steps around the products are kept few (per-fragment
// data through LDS instead of lane moves, ReLU in one instruction), and within
// a block the stage of each weight gradient is written before, and read behind,
// a data backward. 64 views of 50,000 triangles, 16-32-32-4: 2.71 -> 2.65 ms;
// 200,000 triangles, 32-64-64-4: 8.60 -> 8.33 ms (its products alone: 5.6 ms).
// Two blocks side by side spilled registers; the grid as a matrix product
// (texels x fragments x channels) took 2.83 and 8.66 ms.
#include "decode_mfma.hpp"

namespace soup {

constexpr int kStageRows = 16;   // fragments staged per transpose pass
// floats after a wave's gradient grid: the current triangle's nine vertex
// gradient sums, as doubles
constexpr int kGridTail = 32;

// 1/x in double: the hardware estimate refined by two Newton steps (about one
// ulp; the backward needs no correctly rounded quotient)
__device__ __forceinline__ double rcp64(double x) {
    double r = __builtin_amdgcn_rcp(x);
    double e = __builtin_fma(-x, r, 1.0);
    r = __builtin_fma(r, e, r);
    e = __builtin_fma(-x, r, 1.0);
    return __builtin_fma(r, e, r);
}

// The sigmoid of the backward's recompute, from the hardware exp2 and
// reciprocal (a few ulp; only the forward's mask decision is bit-exact)
__device__ __forceinline__ float sigmoid_fast(float x) { return __builtin_amdgcn_rcpf(1.0f + __expf(-x)); }

template <class S>
struct StageCfg {
    static constexpr int kMax2(int a, int b) { return a > b ? a : b; }
    // the widest pair of staged rows (in, d), each row padded by kRowPad floats
    static constexpr int kWidth = kMax2(kMax2(S::C + S::H, 2 * S::H), S::H + 4) + 2 * kRowPad;
};

// Accumulators of one layer's weight gradient dW[DOUT][DIN] += sum_f d_f a_f^T
// on the matrix cores: the contraction runs over fragments, four per
// v_mfma_f32_16x16x4f32 (A[m][k] = d[f_k][m], B[k][n] = a[f_k][n]); dW is
// tiled in 16x16 blocks held in registers (4 per lane per block), padded
// with zeros where DIN or DOUT is below 16. The bias gradient sum_f d_f is
// kept per lane in the unit-major layout of d (units 16 bo + 4 i + grp of the
// lane's fragments; for the output layer, OUTL, output grp in element 0) and
// summed over the lanes of a lane group at the end. Staged rows of hidden units
// are in position order (UIN: the inputs are hidden units, else channels); the
// outputs are hidden units except in the output layer.
template <int DIN, int DOUT, bool UIN, bool OUTL = false>
struct LayerAcc {
    static constexpr int BI = (DIN + 15) / 16;
    static constexpr int BO = (DOUT + 15) / 16;
    static constexpr int NB = BI * BO;
    static_assert(!OUTL || DOUT == 4, "the output layer has four outputs, one per lane group");
    f4v w[NB];
    f4v bs[BO];
    __device__ __forceinline__ void zero() {
#pragma unroll
        for (int i = 0; i < NB; ++i) w[i] = f4v{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int i = 0; i < BO; ++i) bs[i] = f4v{0.f, 0.f, 0.f, 0.f};
    }
    __device__ __forceinline__ void add_bias(const f4v (&d)[BO]) {
        if (OUTL) {
            bs[0][0] += d[0][0];
        } else {
#pragma unroll
            for (int i = 0; i < BO; ++i) bs[i] += d[i];
        }
    }
    // kStageRows (16) staged fragments: in[r][DIN] and d[r][DOUT] in LDS, rows
    // padded by kRowPad. The operands of all steps are read first: their wait
    // can then lie behind other products.
    static constexpr int KS = kStageRows / 4;
    struct Operands {
        float av[KS][BO], bv[KS][BI];
    };
    __device__ __forceinline__ static void load(Operands& o, const float* __restrict__ in, const float* __restrict__ d, int lane) {
        const int col = lane & 15, kq = lane >> 4;
#pragma unroll
        for (int kk = 0; kk < KS; ++kk) {
            const int r = 4 * kk + kq;
#pragma unroll
            for (int bo = 0; bo < BO; ++bo) {
                const int m = 16 * bo + col;
                o.av[kk][bo] = m < DOUT ? d[r * (DOUT + kRowPad) + m] : 0.0f;
            }
#pragma unroll
            for (int bi = 0; bi < BI; ++bi) {
                const int n = 16 * bi + col;
                o.bv[kk][bi] = n < DIN ? in[r * (DIN + kRowPad) + n] : 0.0f;
            }
        }
    }
    __device__ __forceinline__ void accumulate(const Operands& o) {
#pragma unroll
        for (int kk = 0; kk < KS; ++kk)
#pragma unroll
            for (int bo = 0; bo < BO; ++bo)
#pragma unroll
                for (int bi = 0; bi < BI; ++bi)
                    w[bo * BI + bi] =
                        __builtin_amdgcn_mfma_f32_16x16x4f32(o.av[kk][bo], o.bv[kk][bi], w[bo * BI + bi], 0, 0, 0);
    }
    // D of a 16x16 block: lane l holds column l % 16, rows 4 (l / 16) + i
    __device__ __forceinline__ void store(float* __restrict__ row, int w_off, int b_off, int lane) const {
#pragma unroll
        for (int bo = 0; bo < BO; ++bo)
#pragma unroll
            for (int bi = 0; bi < BI; ++bi)
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const int m = 16 * bo + (OUTL ? 4 * (lane >> 4) + i : 4 * i + (lane >> 4));
                    const int n = 16 * bi + (UIN ? unit_of(lane & 15) : lane & 15);
                    if (m < DOUT && n < DIN) row[w_off + m * DIN + n] = w[bo * BI + bi][i];
                }
        // bias: sum over the 16 lanes (fragments) of each lane group
#pragma unroll
        for (int bo = 0; bo < BO; ++bo) {
            f4v v = bs[bo];
#pragma unroll
            for (int sh = 1; sh < 16; sh <<= 1)
#pragma unroll
                for (int i = 0; i < 4; ++i) v[i] += __shfl_xor(v[i], sh, 64);
            if ((lane & 15) == 0) {
                if (OUTL) {
                    row[b_off + (lane >> 4)] = v[0];
                } else {
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        const int m = 16 * bo + 4 * i + (lane >> 4);
                        if (m < DOUT) row[b_off + m] = v[i];
                    }
                }
            }
        }
    }
};

// The output layer's weight gradient dW[4][DIN] += sum_f d_f a_f^T on
// v_mfma_f32_4x4x1f32: block b (lanes 4b .. 4b + 3) accumulates the 4 x 4
// tile of positions 4 (b % 8) .. + 3 over the fragments of half b / 8 of the 16
// staged rows, one fragment per product (A = the fragment's four output
// deltas, B = its four units); the two halves are added at the end. The
// bias gradient as in LayerAcc (output grp in element 0 of lane group grp).
template <int DIN>
struct OutAcc {
    static_assert(DIN == 32, "the tiles cover 32 input units");
    f4v w;
    f4v bs[1];
    __device__ __forceinline__ void zero() {
        w = f4v{0.f, 0.f, 0.f, 0.f};
        bs[0] = f4v{0.f, 0.f, 0.f, 0.f};
    }
    __device__ __forceinline__ void add_bias(const f4v (&d)[1]) { bs[0][0] += d[0][0]; }
    struct Operands {
        float av[8], bv[8];
    };
    __device__ __forceinline__ static void load(Operands& o, const float* __restrict__ in, const float* __restrict__ d, int lane) {
        const int x = lane & 3, t = (lane >> 2) & 7, half = lane >> 5;
#pragma unroll
        for (int k = 0; k < 8; ++k) {
            const int f = 8 * half + k;
            o.av[k] = d[f * (4 + kRowPad) + x];
            o.bv[k] = in[f * (DIN + kRowPad) + 4 * t + x];
        }
    }
    __device__ __forceinline__ void accumulate(const Operands& o) {
#pragma unroll
        for (int k = 0; k < 8; ++k) w = mfma4x4(o.av[k], o.bv[k], w);
    }
    __device__ __forceinline__ void store(float* __restrict__ row, int w_off, int b_off, int lane) const {
        // lanes 0..31 (the first half) add the second half's tiles
        f4v s;
#pragma unroll
        for (int i = 0; i < 4; ++i) s[i] = pair32f(w[i], w[i]);
        if (lane < 32) {
            const int pos = lane;   // tile lane / 4, column lane & 3
#pragma unroll
            for (int i = 0; i < 4; ++i) row[w_off + i * DIN + 16 * (pos >> 4) + unit_of(pos & 15)] = s[i];
        }
        f4v v = bs[0];
#pragma unroll
        for (int sh = 1; sh < 16; sh <<= 1) v[0] += __shfl_xor(v[0], sh, 64);
        if ((lane & 15) == 0) row[b_off + (lane >> 4)] = v[0];
    }
};

template <class S, bool OUT4 = (S::H == 32)>
struct OutAccOf {
    using type = LayerAcc<S::H, 4, true, true>;
};
template <class S>
struct OutAccOf<S, true> {
    using type = OutAcc<S::H>;
};

template <class S>
struct MlpGrad {
    LayerAcc<S::C, S::H, false> l0;
    LayerAcc<S::H, S::H, true> mid[S::NH > 1 ? S::NH - 1 : 1];
    typename OutAccOf<S>::type out;
};

// SHORT: the waves' ranges are equal in blocks of 16 fragments, the MLP's unit,
// and the last batch of a range leaves its empty blocks out. In whole batches,
// waves with three of them waited a quarter of the time for ones with four
// (one 800 x 800 view of 10,000 triangles: 116 -> 101 us); long lists keep the
// plain loop, in which a full batch takes 2 to 4% less.
template <class S, bool SHORT>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2))) void decode_bwd_kernel(DecodeArgs a) {
    constexpr int NW = 4;
    constexpr int SW = StageCfg<S>::kWidth;
    __shared__ __align__(16) float s_stage[NW][kStageRows * SW];
    __shared__ MfmaWeights<S> s_w;     // the MLP in the matrix cores' operand order
    // the batch's feature gradients, rows of C padded by kRowPad (not for C = 32: that
    // shape's LDS is full)
    constexpr int DXS = S::C + (S::C >= 32 ? 0 : kRowPad);
    __shared__ __align__(16) float s_dx[NW][64 * DXS];
    extern __shared__ __align__(16) float s_dyn[];   // [NW][G*G*C + kGridTail]: per-wave gradient grid of the current triangle

    const int tid = threadIdx.x, w = tid >> 6, lane = tid & 63;
    const int G = a.G;
    const int n_grid = G * G * S::C;
    gfloat* __restrict__ feats = as_global(uniform_ptr(a.feats));

    MlpGrad<S> acc;
    acc.l0.zero();
    if constexpr (S::NH == 2) acc.mid[0].zero();
    acc.out.zero();
    s_w.load(a.mlp, tid, blockDim.x);
    __syncthreads();
    const uint64_t n_waves = static_cast<uint64_t>(gridDim.x) * NW;
    const uint64_t wid = static_cast<uint64_t>(blockIdx.x) * NW + w;
    float* grid = s_dyn + static_cast<size_t>(w) * (n_grid + kGridTail);
    double* vgrid = reinterpret_cast<double*>(grid + n_grid);   // the nine vertex sums (n_grid is even)
    int cur = -1;                    // triangle held in grid (wave-uniform)
    // this wave's contiguous range of the sorted fragments
    const int64_t E = a.tri_off[a.T];
    const uint64_t nb = (static_cast<uint64_t>(E) + 63) / 64;
    const uint64_t per = (nb + n_waves - 1) / n_waves;
    const uint64_t b_begin = wid * per, b_end = b_begin + per < nb ? b_begin + per : nb;
    const uint64_t n16 = (static_cast<uint64_t>(E) + 15) / 16;
    const int64_t f0 = static_cast<int64_t>(SHORT ? n16 * wid / n_waves * 16 : b_begin * 64);
    const int64_t fe = static_cast<int64_t>(SHORT ? n16 * (wid + 1) / n_waves * 16 : b_end * 64);
    const int64_t f1 = fe < E ? fe : E;
    const int n_mine = SHORT ? static_cast<int>(f1 - f0) : 0;   // (a short list's share)
    for (int k = lane; k < n_grid + kGridTail; k += 64) grid[k] = 0.0f;
    SharedEnds ends;
    ends.load(a.sorted, f0, f1, E);
    // sorted list: the next batch's records, loaded one batch ahead, and the
    // per-pixel data of its winners (colour gradient, edge weights), loaded
    // once those records are in (after the current batch's MLP)
    uint4 na = make_uint4(0u, 0u, 0u, 0u);   // (pixel, triangle | winner, b1, b2)
    uint2 nx = make_uint2(0u, 0u);           // (score weight, view)
    float ng0 = 0.f, ng1 = 0.f, ng2 = 0.f, nex = 0.f, ney = 0.f;
    bool nvalid = false;
    auto prefetch = [&](uint64_t bi) __attribute__((always_inline)) {
        const int64_t fi = SHORT ? f0 + static_cast<int64_t>(bi) * 64 + lane : static_cast<int64_t>(bi) * 64 + lane;
        nvalid = SHORT ? fi < f1 : bi < b_end && fi < E;
        if (nvalid) {
            const uint2* fr = reinterpret_cast<const uint2*>(a.sorted + fi);
            const uint2 p0 = nt_load(fr), p1 = nt_load(fr + 1);
            na = make_uint4(p0.x, p0.y, p1.x, p1.y);
            nx = nt_load(fr + 2);
        }
    };
    auto pixfetch = [&]() __attribute__((always_inline)) {
        ng0 = ng1 = ng2 = nex = ney = 0.0f;
        if (nvalid && (na.y >> 31)) {
            const size_t p = na.x;
            ng0 = a.grad_color[3 * p];
            ng1 = a.grad_color[3 * p + 1];
            ng2 = a.grad_color[3 * p + 2];
            if (a.edge_w) {
                const float2 e = a.edge_w[p];
                nex = e.x;
                ney = e.y;
            }
        }
    };
    const uint64_t bi0 = SHORT ? 0 : b_begin, bi1 = SHORT ? (static_cast<uint64_t>(n_mine) + 63) / 64 : b_end;
    prefetch(bi0);
    pixfetch();
    // the grid of triangle t goes to HBM and is cleared (whole wave)
    auto flush = [&](int t) __attribute__((always_inline)) {
        wave_fence();
        const bool owned = ends.owned(t);
        float* gf = a.grad_feats + static_cast<size_t>(t) * n_grid;
        for (int k = lane; k < n_grid; k += 64) {
            const float v = grid[k];
            grid[k] = 0.0f;
            if (owned) __builtin_nontemporal_store(a.accumulate ? gf[k] + v : v, &gf[k]);
            else if (v != 0.0f) atomicAdd(&gf[k], v);
        }
        if (lane < 9) {
            const float v = static_cast<float>(vgrid[lane]);
            vgrid[lane] = 0.0;
            float* gv = a.grad_verts + static_cast<size_t>(t) * 9 + lane;
            if (owned) *gv = a.accumulate ? *gv + v : v;
            else if (v != 0.0f) atomicAdd(gv, v);
        }
        wave_fence();
    };
    for (uint64_t bi = bi0; bi < bi1; ++bi) {
        const bool on = SHORT ? static_cast<int>(bi) * 64 + lane < n_mine : static_cast<int64_t>(bi) * 64 + lane < E;
        uint4 fa = make_uint4(0u, 0u, 0u, 0u), fb4 = make_uint4(0u, 0u, 0u, 0u), fc4 = make_uint4(0u, 0u, 0u, 0u);
        if (on) {
            fa = na;
            fb4 = make_uint4(nx.x, __float_as_uint(ng0), __float_as_uint(ng1), __float_as_uint(ng2));
            fc4 = make_uint4(__float_as_uint(nex), __float_as_uint(ney), nx.y, 0u);
        }
        prefetch(bi + 1);
        const uint32_t pix = fa.x;
        const uint32_t tri = fa.y & 0x7FFFFFFFu;
        const bool win = on && (fa.y >> 31);
        const float b1 = __uint_as_float(fa.z), b2 = __uint_as_float(fa.w);
        const Cell c = cell_of(b1, b2, G);
        const uint64_t on_mask = __ballot(on);
        if (a.counter && lane == 0) atomicAdd(a.counter, static_cast<unsigned long long>(__popcll(on_mask)));
        float* st = s_stage[w];
        // Each fragment's data for the MLP goes to its row of s_dx, which its
        // feature gradient takes later: the lanes of its block read it back from
        // there (moving it between lanes took five instructions per value).
        // Triangle and winner bit are 0x7FFFFFFF for an empty lane (no triangle has
        // that index: T is below 2^31); an empty fragment has zero weights,
        // colour gradient and score weight, so that it adds nothing.
        {
            float* info = s_dx[w] + lane * DXS;
            *reinterpret_cast<float4*>(info) =
                make_float4(__uint_as_float(on ? fa.y : 0x7FFFFFFFu),
                            __uint_as_float(static_cast<uint32_t>(c.iy * G + c.ix)), c.fx, c.fy);
            *reinterpret_cast<float4*>(info + 4) = make_float4(__uint_as_float(fb4.x), __uint_as_float(fb4.y),
                                                               __uint_as_float(fb4.z), __uint_as_float(fb4.w));
        }
        wave_fence();
        float my_dfx = 0.0f, my_dfy = 0.0f;   // this lane's fragment: d loss / d (fx, fy), colour logits
        {   // ---- the batch's MLP on the matrix cores, 16-fragment block by block ----
            constexpr int CB = MfmaWeights<S>::CB, HB = MfmaWeights<S>::HB;
            const int col = lane & 15, grp = lane >> 4;
            const MfmaWeights<S>& Wt = s_w;
            const float inf = opaque_inf();
            // The four corners of the block's texels are loaded one block ahead:
            // they are in flight while the previous block runs on the matrix
            // cores. Lane (col, grp) takes channels 16 cb + 4 grp .. + 3 of
            // fragment 16 nb + col.
            float4 qv[CB][4];
            float qfx, qfy;        // the block fragment's position in its texture cell
            uint32_t qkey;         // its triangle and winner bit
            auto gather = [&](int nb) __attribute__((always_inline)) {
                const float4 q = *reinterpret_cast<const float4*>(s_dx[w] + (16 * nb + col) * DXS);
                qkey = __float_as_uint(q.x);
                qfx = q.z;
                qfy = q.w;
                // unconditional loads (an empty lane reads texel 0 of triangle
                // 0 and its input is zeroed), so that the wait before their use
                // can leave the next block's loads in flight
                const uint32_t tri_n = qkey & 0x7FFFFFFFu;
                const size_t t00 = tri_n != 0x7FFFFFFFu
                                       ? (static_cast<size_t>(tri_n) * G * G + __float_as_uint(q.y)) * S::C : 0;
                const size_t toff[4] = {0, S::C, static_cast<size_t>(G) * S::C, static_cast<size_t>(G + 1) * S::C};
#pragma unroll
                for (int cb = 0; cb < CB; ++cb) {
                    const int ch = 16 * cb + 4 * grp < S::C ? 16 * cb + 4 * grp : 0;
#pragma unroll
                    for (int q4 = 0; q4 < 4; ++q4) qv[cb][q4] = *reinterpret_cast<gfloat4*>(feats + t00 + toff[q4] + ch);
                }
            };
            gather(0);
            // While a wave runs its chains of products it issues ahead of the other
            // wave of its SIMD: priority 2 for the MLP, 1 for the grid adds, the
            // default for the vertex chain and the record loads (decode 2.95 -> 2.91 ms).
            __builtin_amdgcn_s_setprio(2);
            for (int nb = 0; nb < 4; ++nb) {   // fragments 16 nb + col
                if (SHORT && static_cast<int>(bi) * 64 + 16 * nb >= n_mine) break;
                const bool on_n = (qkey & 0x7FFFFFFFu) != 0x7FFFFFFFu, win_n = (qkey >> 31) != 0;
                // score weight, and lane group j < 3's channel j of the colour gradient
                const float4 g4 = *reinterpret_cast<const float4*>(s_dx[w] + (16 * nb + col) * DXS + 4);
                const float gl_n = g4.x, gcol = grp == 0 ? g4.y : grp == 1 ? g4.z : g4.w;
                // inputs, unit-major: channels 16 cb + 4 grp .. + 3 (an empty lane's
                // weights are zero; channels past C enter no step of layer 0)
                f4v xin[CB];
                // d feature / d fx and d feature / d fy at the fragment's texture
                // position (bilinear), the directions in which a winner's vertices
                // move its texture sample (an empty lane's are multiplied by a
                // zero feature gradient)
                f4v tgx[CB], tgy[CB];
                {
                    const float fx = qfx, fy = qfy, ax = 1.0f - fy, ay = 1.0f - fx;
                    const float qw[4] = {on_n ? ay * ax : 0.0f, on_n ? fx * ax : 0.0f, on_n ? ay * fy : 0.0f,
                                         on_n ? fx * fy : 0.0f};
#pragma unroll
                    for (int cb = 0; cb < CB; ++cb) {
                        const float4 q00 = qv[cb][0], q10 = qv[cb][1], q01 = qv[cb][2], q11 = qv[cb][3];
                        const float a00[4] = {q00.x, q00.y, q00.z, q00.w}, a10[4] = {q10.x, q10.y, q10.z, q10.w};
                        const float a01[4] = {q01.x, q01.y, q01.z, q01.w}, a11[4] = {q11.x, q11.y, q11.z, q11.w};
#pragma unroll
                        for (int i = 0; i < 4; ++i) {
                            xin[cb][i] = __builtin_fmaf(qw[3], a11[i], __builtin_fmaf(qw[2], a01[i],
                                                        __builtin_fmaf(qw[1], a10[i], qw[0] * a00[i])));
                            tgx[cb][i] = __builtin_fmaf(ax, a10[i] - a00[i], fy * (a11[i] - a01[i]));
                            tgy[cb][i] = __builtin_fmaf(ay, a01[i] - a00[i], fx * (a11[i] - a10[i]));
                        }
                        // channels in the order of the layer's steps
                        xin[cb] = transpose_rows(xin[cb]);
                    }
                }
                if (nb + 1 < 4) gather(nb + 1);
                // forward
                f4v h0[HB], h1[S::NH == 2 ? HB : 1];
                mfma_layer<HB, CB, S::C>(Wt.l0, Wt.b0, xin, h0, lane, inf);
                if constexpr (S::NH == 2) mfma_layer<HB, HB, S::H>(Wt.l1, Wt.b1, h0, h1, lane, inf);
                const f4v (&hl)[HB] = *reinterpret_cast<const f4v (*)[HB]>(S::NH == 2 ? h1 : h0);
                // output layer and the logit gradients (Eq. (9) through the sigmoid for the score term)
                float dO;   // lane group j: output j of the fragment
                {
                    // lane group g: outputs 0..3 summed over its own units 16 ib + 4 s + g
                    f4v pr = f4v{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                    for (int ib = 0; ib < HB; ++ib) {
                        const f4v wv = Wt.lo[ib][lane];
#pragma unroll
                        for (int s4 = 0; s4 < 4; ++s4) pr = mfma4x4(wv[s4], hl[ib][s4], pr);
                    }
                    // the four lane groups' parts summed, output g to lane group g
                    const float og = pair16f(pair32f(pr[0], pr[2]), pair32f(pr[1], pr[3])) + Wt.bo[lane];
                    const float sg = sigmoid_fast(og);
                    const float ds = win_n ? gl_n * (1.0f - sg) : -gl_n * sg;
                    const float dc = win_n ? gcol * sg * (1.0f - sg) : 0.0f;
                    dO = grp == 3 ? ds : dc;
                }
                // The backward of the block. Every weight gradient's stage is written
                // before, and its operands are read back behind, a data backward's
                // products, which do not wait for it.
                auto back = [&](auto with_split) __attribute__((always_inline)) {
                    constexpr bool kSplit = decltype(with_split)::value;
                    float* __restrict__ const st_h = st + kStageRows * (S::H + kRowPad);
                    float* __restrict__ const st_c = st + kStageRows * (S::C + kRowPad);
                    // output layer: its weight gradient's rows, and back through it: K =
                    // the four outputs, one step (with split, the colour logits' beside it)
                    stage_rows<HB>(st, S::H, hl, lane);
                    st_h[col * (4 + kRowPad) + grp] = dO;
                    f4v dl[HB], dlc[HB];
                    const float dOc = grp == 3 ? 0.0f : dO;
#pragma unroll
                    for (int ob = 0; ob < HB; ++ob) {
                        const float wl = Wt.loT[ob][lane];
                        f4v v = mfma4(wl, dO, f4v{0.f, 0.f, 0.f, 0.f}), vc = v;
                        if (kSplit) vc = mfma4(wl, dOc, f4v{0.f, 0.f, 0.f, 0.f});
#pragma unroll
                        for (int i = 0; i < 4; ++i) {
                            v[i] = hl[ob][i] > 0.0f ? v[i] : 0.0f;
                            vc[i] = hl[ob][i] > 0.0f ? vc[i] : 0.0f;
                        }
                        dl[ob] = v;
                        dlc[ob] = vc;
                    }
                    wave_fence();
                    typename OutAccOf<S>::type::Operands opo;
                    acc.out.load(opo, st, st_h, lane);
                    const f4v db[1] = {f4v{dO, 0.f, 0.f, 0.f}};
                    acc.out.add_bias(db);
                    wave_fence();
                    f4v dh0[HB], dh0c[HB];
                    if constexpr (S::NH == 2) {
                        // hidden layer 1
                        stage_rows<HB>(st, S::H, h0, lane);
                        stage_rows<HB>(st_h, S::H, dl, lane);
                        acc.out.accumulate(opo);
                        acc.mid[0].add_bias(dl);
                        wave_fence();
                        typename LayerAcc<S::H, S::H, true>::Operands op1;
                        acc.mid[0].load(op1, st, st_h, lane);
                        mfma_back<HB, HB, true, kSplit>(Wt.l1T, dl, dlc, h0, dh0, dh0c, lane);
                        acc.mid[0].accumulate(op1);
                        wave_fence();
                    } else {
                        acc.out.accumulate(opo);
#pragma unroll
                        for (int ob = 0; ob < HB; ++ob) {
                            dh0[ob] = dl[ob];
                            dh0c[ob] = dlc[ob];
                        }
                    }
                    // layer 0: its weight gradient, and the feature gradients into the
                    // fragments' rows of s_dx; the winners' vertices move with those of
                    // the colour logits alone
                    stage_channels<CB>(st, S::C, xin, lane);
                    stage_rows<HB>(st_c, S::H, dh0, lane);
                    acc.l0.add_bias(dh0);
                    wave_fence();
                    typename LayerAcc<S::C, S::H, false>::Operands op0;
                    acc.l0.load(op0, st, st_c, lane);
                    f4v dxv[CB], dxc[CB];
                    mfma_back<CB, HB, false, kSplit>(Wt.l0T, dh0, dh0c, nullptr, dxv, dxc, lane);
                    acc.l0.accumulate(op0);
                    wave_fence();
                    float pfx = 0.0f, pfy = 0.0f;   // this lane's channels of d logits / d (fx, fy)
#pragma unroll
                    for (int cb = 0; cb < CB; ++cb) {
                        const int ch = 16 * cb + 4 * grp;
                        if (ch < S::C)
                            *reinterpret_cast<float4*>(s_dx[w] + (16 * nb + col) * DXS + ch) =
                                make_float4(dxv[cb][0], dxv[cb][1], dxv[cb][2], dxv[cb][3]);
#pragma unroll
                        for (int i = 0; i < 4; ++i) {
                            pfx = __builtin_fmaf(dxc[cb][i], tgx[cb][i], pfx);
                            pfy = __builtin_fmaf(dxc[cb][i], tgy[cb][i], pfy);
                        }
                    }
                    // sum over the four lane groups' channels; lane 16 nb + col keeps
                    // the values of its own fragment
                    pfx = rows_sum(pfx);
                    pfy = rows_sum(pfy);
                    if (grp == nb) {
                        my_dfx = pfx;
                        my_dfy = pfy;
                    }
                };
                // A winner's vertices move with the feature gradient of its colour
                // logits only: the score logit reaches texture and MLP but no vertex
                // (Section 3.2). Where a winner of the block carries a score weight,
                // the colour logits get a data backward of their own; otherwise the
                // full one is the same thing.
                if (__ballot(win_n && gl_n != 0.0f)) back(std::true_type{});
                else back(std::false_type{});
            }
            wave_fence();
        }
        __builtin_amdgcn_s_setprio(0);
        pixfetch();   // the next batch's winners
        // --- the winner's world-space vertex gradient, in double precision ---
        // The chain is evaluated at the snapped vertex positions and the pixel
        // centre from exact integers, with the clip coordinates recomputed in
        // the setup's float32 order; its sums cancel, and float32 left errors
        // of about 1e-4 of a vertex's total.
        double gw[9] = {0., 0., 0., 0., 0., 0., 0., 0., 0.};
        if (win) {
            const ViewDesc& vd = a.views[fc4.z];
            const TriRec& tr = a.recs[vd.rec_base + tri];
            const int W = vd.W, H = vd.H;
            // the pixel within its view (below 2^32: a view has at most 16384^2 pixels)
            const uint32_t local = pix - static_cast<uint32_t>(vd.pix_base);
            const int py = static_cast<int>(local / static_cast<uint32_t>(W));
            const int px = static_cast<int>(local - static_cast<uint32_t>(py) * static_cast<uint32_t>(W));
            // texture position -> barycentrics -> vertex screen positions and 1/w
            const double gm1 = static_cast<double>(G - 1);
            double iwv[3];
            int32_t Xv[3], Yv[3];
#pragma unroll
            for (int i = 0; i < 3; ++i) {
                iwv[i] = tr.iw[i];
                Xv[i] = tr.X[i];
                Yv[i] = tr.Y[i];
            }
            const int32_t PX = kSnap * px + kSnap / 2, PY = kSnap * py + kSnap / 2;
            // screen barycentrics beta_i = E_i / A: E_i the orientation-normalised
            // integer edge function of edge i at the pixel centre, A their sum.
            // Every factor is an integer below 2^26 and every E_i below 2^52, so
            // the products and the fused sums are exact in double.
            double fb[3];
            {
                const double sgn = tr.rA < 0.0f ? -1.0 : 1.0;
                double Ei[3];
#pragma unroll
                for (int i = 0; i < 3; ++i) {
                    const int ea = i == 2 ? 0 : i + 1, eb = i == 0 ? 2 : (i == 1 ? 0 : 1);
                    const double ex = static_cast<double>(Xv[eb] - Xv[ea]), ey = static_cast<double>(Yv[eb] - Yv[ea]);
                    Ei[i] = sgn * __builtin_fma(ex, static_cast<double>(PY - Yv[ea]),
                                                -(ey * static_cast<double>(PX - Xv[ea])));
                }
                const double inv_a = rcp64((Ei[0] + Ei[1]) + Ei[2]);
#pragma unroll
                for (int i = 0; i < 3; ++i) fb[i] = Ei[i] * inv_a;
            }
            const double tt[3] = {fb[0] * iwv[0], fb[1] * iwv[1], fb[2] * iwv[2]};
            const double inv_s = rcp64((tt[0] + tt[1]) + tt[2]);
            const double bb[3] = {tt[0] * inv_s, tt[1] * inv_s, tt[2] * inv_s};
            const double db[3] = {0.0, static_cast<double>(my_dfx) * gm1, static_cast<double>(my_dfy) * gm1};
            const double dot = db[1] * bb[1] + db[2] * bb[2];
            double dbeta[3], diw[3];
#pragma unroll
            for (int i = 0; i < 3; ++i) {
                const double dt = (db[i] - dot) * inv_s;
                dbeta[i] = dt * iwv[i];
                diw[i] = dt * fb[i];
            }
            const double Ai = __builtin_fma(static_cast<double>(Xv[1] - Xv[0]), static_cast<double>(Yv[2] - Yv[0]),
                                            -(static_cast<double>(Yv[1] - Yv[0]) * static_cast<double>(Xv[2] - Xv[0])));
            const double inv_area = 65536.0 * rcp64(Ai);   // 1 / (signed 2 x area in px^2)
            const double inv256 = 1.0 / 256.0;
            // beta_i = e_i / area, e_i = edge(v_p(i), v_q(i), pixel centre) with edge i
            // joining vertices p(i) = i + 1 and q(i) = i + 2 (mod 3). Vertex jv moves
            // e_i only for the two edges it belongs to (i = jv + 2 as p, i = jv + 1 as
            // q), and the area as a whole; so d beta . dbeta / d(vertex jv) is
            // (sum over those two edges of dbeta_i de_i - d area . sb) / area with
            // sb = sum_i dbeta_i beta_i.
            double sb = 0.0;
#pragma unroll
            for (int i = 0; i < 3; ++i) sb = __builtin_fma(dbeta[i], fb[i], sb);
            double gsx[3], gsy[3];
#pragma unroll
            for (int jv = 0; jv < 3; ++jv) {
                const int jp = jv == 2 ? 0 : jv + 1, jq = jv == 0 ? 2 : (jv == 1 ? 0 : 1);
                const double dax = static_cast<double>(Yv[jp] - Yv[jq]) * inv256;
                const double day = static_cast<double>(Xv[jq] - Xv[jp]) * inv256;
                // edge ip has jv as its first vertex (its other one is jp), edge iq as its second (other: jq)
                const int ip = jv == 0 ? 2 : jv - 1, iq = jv == 2 ? 0 : jv + 1;
                const double ex_p = static_cast<double>(Yv[jp] - PY) * inv256, ey_p = static_cast<double>(PX - Xv[jp]) * inv256;
                const double ex_q = static_cast<double>(PY - Yv[jq]) * inv256, ey_q = static_cast<double>(Xv[jq] - PX) * inv256;
                gsx[jv] = (__builtin_fma(dbeta[ip], ex_p, dbeta[iq] * ex_q) - dax * sb) * inv_area;
                gsy[jv] = (__builtin_fma(dbeta[ip], ey_p, dbeta[iq] * ey_q) - day * sb) * inv_area;
            }
            // edge term (Section 3.2): the boundaries this pixel occludes move
            // with its surface point, w beta_i e on the screen position of vertex i
            const double ex = __uint_as_float(fc4.x), ey = __uint_as_float(fc4.y);
#pragma unroll
            for (int jv = 0; jv < 3; ++jv) {
                gsx[jv] += ex * fb[jv];
                gsy[jv] += ey * fb[jv];
            }
            // screen position (s = W/2 (c_x / c_w) + W/2, H/2 - H/2 (c_y / c_w)) and 1/w
            // -> clip -> world through the view-projection
            const double hw = 0.5 * W, hh = 0.5 * H;
            const float* vp = a.verts + static_cast<size_t>(tri) * 9;
#pragma unroll
            for (int jv = 0; jv < 3; ++jv) {
                const float x = vp[3 * jv], y = vp[3 * jv + 1], z = vp[3 * jv + 2];
                float cc[4];
#pragma unroll
                for (int j = 0; j < 4; ++j) {   // the setup's transform (row z unused)
                    float acc = vd.M[j * 4 + 3];
                    acc = __builtin_fmaf(vd.M[j * 4 + 0], x, acc);
                    acc = __builtin_fmaf(vd.M[j * 4 + 1], y, acc);
                    acc = __builtin_fmaf(vd.M[j * 4 + 2], z, acc);
                    cc[j] = acc;
                }
                const double cx = cc[0], cy = cc[1], iw = rcp64(static_cast<double>(cc[3]));
                const double gc0 = gsx[jv] * hw * iw;
                const double gc1 = -gsy[jv] * hh * iw;
                const double gc3 = (-gsx[jv] * hw * cx + gsy[jv] * hh * cy - diw[jv]) * (iw * iw);
#pragma unroll
                for (int k = 0; k < 3; ++k)
                    gw[3 * jv + k] = static_cast<double>(vd.M[k]) * gc0 + static_cast<double>(vd.M[4 + k]) * gc1 +
                                     static_cast<double>(vd.M[12 + k]) * gc3;
            }
        }
        __builtin_amdgcn_s_setprio(1);
        // --- sum into the wave's grid, one run of equal triangles at a time ---
        // The feature gradients are staged (row = fragment) and added one
        // fragment per step with the wave's lanes spread over (corner,
        // channel), so that no two lanes of an LDS add share an address;
        // the winners' vertex gradients are summed over the run by a wave
        // reduction.
        // One fragment per step also where it has 32 pairs only: two fragments may
        // share a texel, and an LDS float32 add of 64 lanes takes 194 cycles, one
        // lane after the other, where a read and a write take 26 (8-16-4, one 800 x 800
        // view of 20,000 triangles: step 2,304 -> 2,187 us; 500 triangles: 465 -> 384).
        constexpr int LPF = 4 * S::C;                  // (corner, channel) pairs of one fragment
        constexpr int PPF = LPF >= 64 ? LPF / 64 : 1;  // steps per fragment
        // Each lane's fragment leaves its four corner
        // weights (corner q = 2 dy + dx) in the stage, free once the MLP is
        // done, and keeps its cell's first texel; the steps then need no
        // per-fragment weight or address arithmetic beyond one add.
        const float x1 = c.fx, y1 = c.fy, x0 = 1.0f - c.fx, y0 = 1.0f - c.fy;
        *reinterpret_cast<float4*>(st + 4 * lane) = make_float4(x0 * y0, x1 * y0, x0 * y1, x1 * y1);
        const int cbase = (c.iy * G + c.ix) * S::C;
        wave_fence();
        const uint32_t tkey = on ? tri : 0xFFFFFFFFu;
        const uint32_t tprev = __shfl_up(tkey, 1, 64);
        uint64_t heads = __ballot(lane == 0 || tprev != tkey);
        while (heads) {
            const int h = __builtin_ctzll(heads);
            heads &= heads - 1;
            const int t = __builtin_amdgcn_readlane(static_cast<int>(tkey), h);
            if (t < 0) break;   // the sentinel run: empty lanes at the batch's end
            if (t != cur) {
                if (cur >= 0) flush(cur);
                cur = t;
            }
            const int end = heads ? __builtin_ctzll(heads) : 64;
            const bool in_run = lane >= h && lane < end;
            if (__ballot(in_run && win)) {   // the run's winners: vertex gradient summed over the wave
                double v[9], q[3];
#pragma unroll
                for (int k = 0; k < 9; ++k) v[k] = in_run ? gw[k] : 0.0;   // gw is zero for fragments in front
                wave_sum9(v, q);
                if ((lane & 15) == 0) {   // row g's first lane: components c, c + 2 (and 4 in row 0)
                    const int g = lane >> 4, c0 = (g & 1) + 5 * (g >> 1);
                    vgrid[c0] += q[0];
                    vgrid[c0 + 2] += q[1];
                    if (g == 0) vgrid[4] += q[2];
                }
            }
            constexpr int UF = 4;                          // steps in flight: their staged reads go first
            // lane (corner q, channel k) of step pp: weight st[4 f + q],
            // gradient s_dx[f][k], texel q of the fragment's cell
            float* gl[PPF];
            const float* wl[PPF];
            const float* dl[PPF];
#pragma unroll
            for (int pp = 0; pp < PPF; ++pp) {
                const int idx = pp * 64 + lane;
                const int q = idx / S::C, k = idx % S::C;
                gl[pp] = grid + ((q >> 1) * G + (q & 1)) * S::C + k;
                wl[pp] = st + q;
                dl[pp] = s_dx[w] + k;
            }
            // N fragments from f. The cells are read from their lanes while the whole
            // wave is active (a lane's register holds its value for certain only where
            // that lane takes part); lanes past a narrow shape's pairs leave after that.
            auto add = [&](auto n_steps, int f) __attribute__((always_inline)) {
                constexpr int N = decltype(n_steps)::value;
                int cb[N];
#pragma unroll
                for (int u = 0; u < N; ++u) cb[u] = __builtin_amdgcn_readlane(cbase, f + u);
                if (LPF < 64 && lane >= LPF) return;
                float wv[N][PPF], dv[N][PPF];
#pragma unroll
                for (int u = 0; u < N; ++u)
#pragma unroll
                    for (int pp = 0; pp < PPF; ++pp) {
                        wv[u][pp] = wl[pp][4 * (f + u)];
                        dv[u][pp] = dl[pp][(f + u) * DXS];
                    }
#pragma unroll
                for (int u = 0; u < N; ++u)
#pragma unroll
                    for (int pp = 0; pp < PPF; ++pp) {
                        float* gp = gl[pp] + cb[u];   // one fragment: distinct addresses
                        *gp = __builtin_fmaf(wv[u][pp], dv[u][pp], *gp);
                    }
            };
            int f = h;
            for (; f + UF <= end; f += UF) add(std::integral_constant<int, UF>{}, f);
            for (; f < end; ++f) add(std::integral_constant<int, 1>{}, f);
            wave_fence();
        }
    }
    if (cur >= 0) flush(cur);
    float* row = a.mlp_partial + (static_cast<size_t>(blockIdx.x) * NW + w) * S::kParams;
    acc.l0.store(row, S::w_off(0), S::b_off(0), lane);
    if constexpr (S::NH == 2) acc.mid[0].store(row, S::w_off(1), S::b_off(1), lane);
    acc.out.store(row, S::w_off(S::NH), S::b_off(S::NH), lane);
}

// Bytes of LDS one workgroup of the decode needs (static + dynamic), or 0 when
// the runtime cannot say.
template <class S>
static size_t decode_bwd_lds_s(int G) {
    hipFuncAttributes fa;
    if (hipFuncGetAttributes(&fa, reinterpret_cast<const void*>(decode_bwd_kernel<S, false>)) != hipSuccess) {
        (void)hipGetLastError();
        return 0;
    }
    return fa.sharedSizeBytes + static_cast<size_t>(4) * (static_cast<size_t>(G) * G * S::C + kGridTail) * sizeof(float);
}

template <class S>
static void launch_decode_bwd_s(const DecodeArgs& a, hipStream_t s) {
    const size_t lds = static_cast<size_t>(4) * (static_cast<size_t>(a.G) * a.G * S::C + kGridTail) * sizeof(float);
    if (a.short_list) hipLaunchKernelGGL((decode_bwd_kernel<S, true>), dim3(a.n_blocks), dim3(256), lds, s, a);
    else hipLaunchKernelGGL((decode_bwd_kernel<S, false>), dim3(a.n_blocks), dim3(256), lds, s, a);
}

}  // namespace soup
