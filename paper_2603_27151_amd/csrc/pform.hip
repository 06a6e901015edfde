// Paper form of the step (Section 3.3; Supplement B.3, B.6): kernels besides
// the forward raster (which takes the opacity-only policy PaperTex).
//
//  assemble      sigmoid(sum of the learnable levels sampled at the finest
//                grid's vertices), one workgroup per triangle, and its
//                gradient summed per triangle in LDS;
//  shade         the deferred colour of every pixel's winner: features of its
//                micro-triangle, harmonics of the view direction, the MLP on
//                the vector ALUs in the float32 contract, the RGBA blend;
//  frag          over a fragment list (the forward's log filtered, or a
//                replay): the score term of Eq. (9) on the opacity channel, or
//                log p(f*) of Eq. (6);
//  winner_bwd    per pixel: the colour path of the winner (the MLP's data
//                backward on the vector ALUs; its weight gradient, a
//                contraction over pixels, on the matrix cores), the features'
//                gradient onto the three grid vertices, and the vertex
//                gradient through the barycentrics and the edge term in
//                float64.
#include "decode_mfma.hpp"
#include "pform.hpp"

namespace soup {

// ---------------------------------------------------------------------------
// texture assembly
// ---------------------------------------------------------------------------

// (i, j) of the finest grid's vertex k (row-major storage): row j starts at
// j (n + 1) - j (j - 1) / 2; the float estimate of j is corrected exactly.
__device__ __forceinline__ void mc_ij(int n, int k, int& i, int& j) {
    const float b = static_cast<float>(2 * n + 3);
    int jj = static_cast<int>((b - __builtin_sqrtf(b * b - 8.0f * static_cast<float>(k))) * 0.5f);
    jj = jj < 0 ? 0 : (jj > n ? n : jj);
    while (jj > 0 && mc_index(n, 0, jj) > k) --jj;
    while (jj < n && mc_index(n, 0, jj + 1) <= k) ++jj;
    j = jj;
    i = k - mc_index(n, 0, jj);
}

// Fallback for levels too large to stage in LDS: one thread per (triangle,
// vertex of the finest grid), consecutive threads on consecutive vertices
// (32-byte records, written coalesced), the three grid vertices of every
// level gathered from global memory.
__global__ __launch_bounds__(256) void mc_assemble_kernel(AssembleArgs a) {
    const int nf = 1 << a.Rmax, Vf = mc_count(a.Rmax);
    const int64_t g = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
    if (g >= static_cast<int64_t>(a.T) * Vf) return;
    const int t = static_cast<int>(g / Vf);
    const int k = static_cast<int>(g - static_cast<int64_t>(t) * Vf);
    float* out = a.tex_out + static_cast<size_t>(t) * Vf * kPCh;
    {
        int i, j;
        mc_ij(nf, k, i, j);
        // i / n and j / n (n a power of two: the product by 1 / n is exact)
        const float b1 = static_cast<float>(i) * (1.0f / static_cast<float>(nf));
        const float b2 = static_cast<float>(j) * (1.0f / static_cast<float>(nf));
        float z[kPCh];
#pragma unroll
        for (int c = 0; c < kPCh; ++c) z[c] = 0.0f;
        for (int R = a.Rmin; R <= a.Rtop; ++R) {
            const Micro m = micro_of(1 << R, b1, b2);
            const float4* g = reinterpret_cast<const float4*>(a.raw[R - a.Rmin] + static_cast<size_t>(t) * mc_count(R) * kPCh);
            float4 v[3][2];
#pragma unroll
            for (int q = 0; q < 3; ++q) {
                v[q][0] = g[2 * m.idx[q]];
                v[q][1] = g[2 * m.idx[q] + 1];
            }
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                z[4 * h + 0] = z[4 * h + 0] + mc_mix(m, v[0][h].x, v[1][h].x, v[2][h].x);
                z[4 * h + 1] = z[4 * h + 1] + mc_mix(m, v[0][h].y, v[1][h].y, v[2][h].y);
                z[4 * h + 2] = z[4 * h + 2] + mc_mix(m, v[0][h].z, v[1][h].z, v[2][h].z);
                z[4 * h + 3] = z[4 * h + 3] + mc_mix(m, v[0][h].w, v[1][h].w, v[2][h].w);
            }
        }
        float4* o = reinterpret_cast<float4*>(out + static_cast<size_t>(k) * kPCh);
        o[0] = make_float4(sigmoid_c(z[0]), sigmoid_c(z[1]), sigmoid_c(z[2]), sigmoid_c(z[3]));
        o[1] = make_float4(sigmoid_c(z[4]), sigmoid_c(z[5]), sigmoid_c(z[6]), sigmoid_c(z[7]));
    }
}

// TPB consecutive triangles per workgroup: their learnable levels (contiguous
// per level in global memory) are staged in LDS with coalesced 16-byte loads;
// then each thread takes one (finest-grid vertex, half of the channels) for
// all TPB triangles, so the vertex's micro-triangle lookups, which do not
// depend on the triangle, are computed once. Same arithmetic, in the same
// order, as the fallback: the results are identical.
template <int TPB>
__global__ __launch_bounds__(256) void mc_assemble_lds_kernel(AssembleArgs a) {
    extern __shared__ float4 st4[];
    const int t0 = blockIdx.x * TPB;
    const int nt = a.T - t0 < TPB ? a.T - t0 : TPB;
    {
        int off = 0;   // float4 offset of level R's block of TPB triangles
        for (int R = a.Rmin; R <= a.Rtop; ++R) {
            const int v2 = mc_count(R) * 2;
            const float4* src = reinterpret_cast<const float4*>(a.raw[R - a.Rmin]) + static_cast<size_t>(t0) * v2;
            for (int e = threadIdx.x; e < nt * v2; e += blockDim.x) st4[off + e] = src[e];
            off += TPB * v2;
        }
    }
    __syncthreads();
    const int nf = 1 << a.Rmax, Vf = mc_count(a.Rmax);
    for (int e = threadIdx.x; e < 2 * Vf; e += blockDim.x) {
        const int k = e >> 1, h = e & 1;
        int i, j;
        mc_ij(nf, k, i, j);
        const float b1 = static_cast<float>(i) * (1.0f / static_cast<float>(nf));
        const float b2 = static_cast<float>(j) * (1.0f / static_cast<float>(nf));
        float4 z[TPB];
#pragma unroll
        for (int tt = 0; tt < TPB; ++tt) z[tt] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
        int off = 0;
        for (int R = a.Rmin; R <= a.Rtop; ++R) {
            const Micro m = micro_of(1 << R, b1, b2);
            const int v2 = mc_count(R) * 2;
#pragma unroll
            for (int tt = 0; tt < TPB; ++tt) {   // rows past nt hold stale LDS; their results are not stored
                const float4* g = st4 + off + tt * v2 + h;
                const float4 v0 = g[2 * m.idx[0]], v1 = g[2 * m.idx[1]], v2v = g[2 * m.idx[2]];
                z[tt].x = z[tt].x + mc_mix(m, v0.x, v1.x, v2v.x);
                z[tt].y = z[tt].y + mc_mix(m, v0.y, v1.y, v2v.y);
                z[tt].z = z[tt].z + mc_mix(m, v0.z, v1.z, v2v.z);
                z[tt].w = z[tt].w + mc_mix(m, v0.w, v1.w, v2v.w);
            }
            off += TPB * v2;
        }
#pragma unroll
        for (int tt = 0; tt < TPB; ++tt) {
            if (tt < nt) {
                float4* o = reinterpret_cast<float4*>(a.tex_out) + static_cast<size_t>(t0 + tt) * Vf * 2 + e;
                const f4v r = {sigmoid_c(z[tt].x), sigmoid_c(z[tt].y), sigmoid_c(z[tt].z), sigmoid_c(z[tt].w)};
                __builtin_nontemporal_store(r, reinterpret_cast<f4v*>(o));
            }
        }
    }
}

// Bytes of the learnable levels of one triangle.
static size_t mc_levels_bytes(int Rmin, int Rtop) {
    size_t b = 0;
    for (int R = Rmin; R <= Rtop; ++R) b += static_cast<size_t>(mc_count(R)) * kPCh * sizeof(float);
    return b;
}

// Gradient of the assembly. The lookup of level R at the vertices of level
// Rmax equals prolongation to level R + 1, then R + 2, ..., Rmax (the field of
// a level is linear on each of its micro-triangles, and every micro-triangle
// of the next level lies inside one of them; a vertex of level R + 1 is a
// vertex of level R, weight 1, or the midpoint of an edge, weights 1/2). Its
// transpose is the restriction chain: with dz = tex (1 - tex) d tex on level
// Rmax, g_R(I, J) = g_{R+1}(2I, 2J) + 1/2 sum over the six lattice neighbours
// (2I, 2J) + d, d in +-(1, 0), +-(0, 1), +-(1, -1), that exist. One workgroup
// per triangle keeps the chain in LDS (two buffers of the largest level) and
// writes every learnable level; without room for them the adds go to global
// memory directly, one lookup per level and vertex.
template <bool LDS_SUM>
__global__ __launch_bounds__(256) void mc_assemble_bwd_kernel(AssembleArgs a) {
    extern __shared__ float lds[];
    const int t = blockIdx.x;
    const int nf = 1 << a.Rmax, Vf = mc_count(a.Rmax);
    const float* tx = a.tex + static_cast<size_t>(t) * Vf * kPCh;
    const float* gt = a.grad_tex + static_cast<size_t>(t) * Vf * kPCh;
    if constexpr (LDS_SUM) {
        // level Rmax in the first buffer, the chain's levels then alternate
        // between a second buffer (levels Rmax - 1, Rmax - 3, ...) and the first
        float* cur = lds;
        float* nxt = lds + Vf * kPCh;
        const float4* tx4 = reinterpret_cast<const float4*>(tx);
        const float4* gt4 = reinterpret_cast<const float4*>(gt);
        float4* cur4 = reinterpret_cast<float4*>(cur);
        auto dz4 = [](float4 g, float4 s) {
            return make_float4(g.x * s.x * (1.0f - s.x), g.y * s.y * (1.0f - s.y), g.z * s.z * (1.0f - s.z),
                               g.w * s.w * (1.0f - s.w));
        };
        {   // four loads of each array in flight per thread
            const int n4 = Vf * 2;
            int e = threadIdx.x;
            const int nt = blockDim.x;
            for (; e + 3 * nt < n4; e += 4 * nt) {
                float4 sv[4], gv[4];
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    sv[u] = tx4[e + u * nt];
                    gv[u] = gt4[e + u * nt];
                }
#pragma unroll
                for (int u = 0; u < 4; ++u) cur4[e + u * nt] = dz4(gv[u], sv[u]);
            }
            for (; e < n4; e += nt) cur4[e] = dz4(gt4[e], tx4[e]);
        }
        __syncthreads();
        for (int R = a.Rmax;; --R) {
            if (R <= a.Rtop) {   // a learnable level: out (32 bytes per vertex, 16-byte aligned)
                const int n4 = mc_count(R) * 2;
                float4* g = reinterpret_cast<float4*>(a.graw[R - a.Rmin]) + static_cast<size_t>(t) * n4;
                const float4* c4 = reinterpret_cast<const float4*>(cur);
                for (int e = threadIdx.x; e < n4; e += blockDim.x) {
                    float4 v = c4[e];
                    if (a.accumulate) {
                        const float4 o = g[e];
                        v = make_float4(o.x + v.x, o.y + v.y, o.z + v.z, o.w + v.w);
                    }
                    g[e] = v;
                }
            }
            if (R == a.Rmin) break;
            // restrict level R (cur) onto level R - 1 (nxt): one thread per
            // (coarse vertex, four channels), the six neighbours in a fixed order
            const int nc = 1 << (R - 1), nfl = 1 << R, Vc = mc_count(R - 1);
            const float4* c4 = reinterpret_cast<const float4*>(cur);
            float4* n4 = reinterpret_cast<float4*>(nxt);
            for (int e = threadIdx.x; e < Vc * 2; e += blockDim.x) {
                const int q = e >> 1, h = e & 1;
                int I, J;
                mc_ij(nc, q, I, J);
                const int i = 2 * I, j = 2 * J;
                float4 side = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
                auto add = [&](int ii, int jj) __attribute__((always_inline)) {
                    const float4 v = c4[mc_index(nfl, ii, jj) * 2 + h];
                    side = make_float4(side.x + v.x, side.y + v.y, side.z + v.z, side.w + v.w);
                };
                if (i + 1 + j <= nfl) add(i + 1, j);
                if (i > 0) add(i - 1, j);
                if (i + j + 1 <= nfl) add(i, j + 1);
                if (j > 0) add(i, j - 1);
                if (j > 0) add(i + 1, j - 1);   // i + 1 + j - 1 <= n always
                if (i > 0) add(i - 1, j + 1);
                const float4 c = c4[mc_index(nfl, i, j) * 2 + h];
                n4[e] = make_float4(c.x + 0.5f * side.x, c.y + 0.5f * side.y, c.z + 0.5f * side.z, c.w + 0.5f * side.w);
            }
            __syncthreads();
            float* tmp = cur;
            cur = nxt;
            nxt = tmp;
        }
    } else {
        const int nl = a.Rtop - a.Rmin + 1;
        for (int k = threadIdx.x; k < Vf; k += blockDim.x) {
            int i, j;
            mc_ij(nf, k, i, j);
            const float b1 = static_cast<float>(i) * (1.0f / static_cast<float>(nf));
            const float b2 = static_cast<float>(j) * (1.0f / static_cast<float>(nf));
            float dz[kPCh];
#pragma unroll
            for (int c = 0; c < kPCh; ++c) {
                const float s = tx[k * kPCh + c];
                dz[c] = gt[k * kPCh + c] * s * (1.0f - s);
            }
            for (int l = 0; l < nl; ++l) {
                const int R = a.Rmin + l;
                const Micro m = micro_of(1 << R, b1, b2);
#pragma unroll
                for (int q = 0; q < 3; ++q) {
                    if (m.w[q] == 0.0f) continue;
#pragma unroll
                    for (int c = 0; c < kPCh; ++c) {
                        const float v = m.w[q] * dz[c];
                        if (v != 0.0f) atomicAdd(&a.graw[l][(static_cast<size_t>(t) * mc_count(R) + m.idx[q]) * kPCh + c], v);
                    }
                }
            }
        }
    }
}

// LDS one workgroup of the assembly gradient may take: half the CU's, at most 64 KiB.
size_t mc_assemble_bwd_lds_cap(size_t lds_limit) { return lds_limit / 2 < 65536 ? lds_limit / 2 : 65536; }

// The finest level's gradient and the next coarser one's (every later level fits the first).
size_t mc_assemble_bwd_lds(int Rmin, int Rmax) {
    const size_t next = Rmax > Rmin ? static_cast<size_t>(mc_count(Rmax - 1)) : 0;
    return (static_cast<size_t>(mc_count(Rmax)) + next) * kPCh * sizeof(float);
}

void launch_mc_assemble(const AssembleArgs& a, hipStream_t s) {
    if (a.T <= 0) return;
    // four triangles per workgroup while their levels take at most 32 KiB of
    // LDS, fewer up to 64 KiB, else the gathering fallback
    const size_t lb = mc_levels_bytes(a.Rmin, a.Rtop);
    const int tpb = 4 * lb <= 32768 ? 4 : (2 * lb <= 49152 ? 2 : (lb <= 65536 ? 1 : 0));
    const unsigned nb = static_cast<unsigned>((a.T + (tpb > 0 ? tpb : 1) - 1) / (tpb > 0 ? tpb : 1));
    if (tpb == 4) {
        hipLaunchKernelGGL(mc_assemble_lds_kernel<4>, dim3(nb), dim3(256), 4 * lb, s, a);
    } else if (tpb == 2) {
        hipLaunchKernelGGL(mc_assemble_lds_kernel<2>, dim3(nb), dim3(256), 2 * lb, s, a);
    } else if (tpb == 1) {
        hipLaunchKernelGGL(mc_assemble_lds_kernel<1>, dim3(nb), dim3(256), lb, s, a);
    } else {
        const int64_t n = static_cast<int64_t>(a.T) * mc_count(a.Rmax);
        hipLaunchKernelGGL(mc_assemble_kernel, dim3(static_cast<unsigned>((n + 255) / 256)), dim3(256), 0, s, a);
    }
}

void launch_mc_assemble_bwd(const AssembleArgs& a, size_t lds_limit, hipStream_t s) {
    if (a.T <= 0) return;
    const size_t lds = mc_assemble_bwd_lds(a.Rmin, a.Rmax);
    if (lds <= mc_assemble_bwd_lds_cap(lds_limit)) {
        hipLaunchKernelGGL(mc_assemble_bwd_kernel<true>, dim3(static_cast<unsigned>(a.T)), dim3(256), lds, s, a);
    } else {
        // outputs zeroed by the caller unless accumulating
        hipLaunchKernelGGL(mc_assemble_bwd_kernel<false>, dim3(static_cast<unsigned>(a.T)), dim3(256), 0, s, a);
    }
}

// ---------------------------------------------------------------------------
// per-pixel helpers
// ---------------------------------------------------------------------------

// View of global pixel p (views ordered by pix_base).
__device__ __forceinline__ int view_of_pixel(const ViewDesc* __restrict__ views, int V, int64_t p) {
    int lo = 0, hi = V - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (views[mid].pix_base <= p) lo = mid;
        else hi = mid - 1;
    }
    return lo;
}

// Workgroups are dealt to the eight XCDs in turn: workgroup b works on block
// (b % 8) * per + b / 8 of the grid's blocks (a bijection when the grid is a
// multiple of eight), so that each XCD takes one contiguous eighth of the
// pixels and a triangle's texture is read into one L2.
__device__ __forceinline__ uint32_t xcd_block() {
    const uint32_t per = gridDim.x / kXcds;
    return (blockIdx.x % kXcds) * per + blockIdx.x / kXcds;
}

// The forward's perspective-correct barycentrics of triangle record tr at the
// centre of pixel (x, y): the exact orientation-normalised edge functions,
// beta_i = (float)E_i |rA|, t_i = beta_i / w_i, then the contract's b1, b2.
__device__ __forceinline__ void frag_bary(const TriRec& tr, int x, int y, float& b1, float& b2, double (&E)[3]) {
    const int64_t PX = static_cast<int64_t>(kSnap) * x + kSnap / 2, PY = static_cast<int64_t>(kSnap) * y + kSnap / 2;
    const double sgn = tr.rA < 0.0f ? -1.0 : 1.0;
    const float ra = __builtin_fabsf(tr.rA);
    float t[3];
#pragma unroll
    for (int i = 0; i < 3; ++i) {
        const int ea = i == 2 ? 0 : i + 1, eb = i == 0 ? 2 : (i == 1 ? 0 : 1);
        const double ex = static_cast<double>(tr.X[eb] - tr.X[ea]), ey = static_cast<double>(tr.Y[eb] - tr.Y[ea]);
        // every factor is an integer below 2^26: the product and the fused sum are exact
        E[i] = sgn * __builtin_fma(ex, static_cast<double>(PY - tr.Y[ea]), -(ey * static_cast<double>(PX - tr.X[ea])));
        t[i] = (static_cast<float>(E[i]) * ra) * tr.iw[i];
    }
    persp_from_t(t[0], t[1], t[2], b1, b2);
}

// The winner's shading inputs: the eight channels of its micro-triangle's
// three grid vertices (v[q][0..1]) and their interpolation (feat).
__device__ __forceinline__ void fetch_texel(gfloat* __restrict__ tex, uint32_t tri, int V, const Micro& m,
                                            float4 (&v)[3][2], float (&feat)[kPCh]) {
    gfloat4* g = reinterpret_cast<gfloat4*>(tex + static_cast<size_t>(tri) * V * kPCh);
#pragma unroll
    for (int q = 0; q < 3; ++q) {
        v[q][0] = g[2 * m.idx[q]];
        v[q][1] = g[2 * m.idx[q] + 1];
    }
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        feat[4 * h + 0] = mc_mix(m, v[0][h].x, v[1][h].x, v[2][h].x);
        feat[4 * h + 1] = mc_mix(m, v[0][h].y, v[1][h].y, v[2][h].y);
        feat[4 * h + 2] = mc_mix(m, v[0][h].z, v[1][h].z, v[2][h].z);
        feat[4 * h + 3] = mc_mix(m, v[0][h].w, v[1][h].w, v[2][h].w);
    }
}

// ---------------------------------------------------------------------------
// deferred shading (forward)
// ---------------------------------------------------------------------------

__global__ __launch_bounds__(256) void pshade_kernel(PShadeArgs a) {
    const int64_t p = static_cast<int64_t>(xcd_block()) * blockDim.x + threadIdx.x;
    if (p >= a.P) return;
    const uint64_t key = a.vis[p];
    float* out = a.color + 3 * p;
    if (key == kBgKey) {
        out[0] = a.o.bg[0];
        out[1] = a.o.bg[1];
        out[2] = a.o.bg[2];
        return;
    }
    const int v = view_of_pixel(a.views, a.V, p);
    const ViewDesc& vd = a.views[v];
    const uint32_t local = static_cast<uint32_t>(p - vd.pix_base);
    const int y = static_cast<int>(local / static_cast<uint32_t>(vd.W));
    const int x = static_cast<int>(local - static_cast<uint32_t>(y) * static_cast<uint32_t>(vd.W));
    const uint32_t tri = static_cast<uint32_t>(key);
    const TriRec tr = a.recs[vd.rec_base + tri];
    float b1, b2;
    double E[3];
    frag_bary(tr, x, y, b1, b2, E);
    const Micro m = micro_of(1 << a.R, b1, b2);
    float4 tv[3][2];
    float feat[kPCh];
    fetch_texel(as_global(a.tex), tri, mc_count(a.R), m, tv, feat);
    float in[kPIn];
#pragma unroll
    for (int c = 0; c < kPFeat; ++c) in[c] = feat[c];
    float d[3];
    view_dir(vd.Mi, vd.W, vd.H, x, y, d);
    sh2(d, in + kPFeat);
    cfloat* mp = as_const(a.mlp);
    float h1[kPHid], h2[kPHid], o[kPOut];
    dense<kPIn, kPHid, true>(mp + kPW0, mp + kPB0, in, h1);
    dense<kPHid, kPHid, true>(mp + kPW1, mp + kPB1, h1, h2);
    dense<kPHid, kPOut, false>(mp + kPW2, mp + kPB2, h2, o);
    const float A = feat[3];
#pragma unroll
    for (int c = 0; c < 3; ++c) {
        const float mm = sigmoid_c(o[c]);
        out[c] = __builtin_fmaf(A, feat[c] - mm, mm);   // A RGB + (1 - A) MLP
    }
}

void launch_pshade(const PShadeArgs& a, hipStream_t s) {
    if (a.P <= 0) return;
    const int64_t nb = ((a.P + 255) / 256 + kXcds - 1) / kXcds * kXcds;
    hipLaunchKernelGGL(pshade_kernel, dim3(static_cast<unsigned>(nb)), dim3(256), 0, s, a);
}

// ---------------------------------------------------------------------------
// fragment list: score term (Eq. (9)) or log p(f*) (Eq. (6))
// ---------------------------------------------------------------------------

template <bool LOGP>
__global__ __launch_bounds__(256) void pfrag_kernel(PFragArgs a) {
    const int lane = threadIdx.x & 63;
    const int n = 1 << a.R, V = mc_count(a.R);
    gfloat* tex = as_global(a.tex);
    for_log_batches(a.log, [&](uint32_t r, uint32_t b, uint32_t cnt) {
        if (b + lane >= cnt) return;
        const uint64_t at = static_cast<uint64_t>(r) * a.log.region + b + lane;
        const uint4 e = a.log.frag[at];
        bool keep, win;
        a.sel.decide(e, keep, win);
        if (!keep) return;
        const uint32_t tri = e.y;
        const uint2 bc = a.log.bary[at];
        const Micro m = micro_of(n, __uint_as_float(bc.x), __uint_as_float(bc.y));
        gfloat* t = tex + static_cast<size_t>(tri) * V * kPCh + (kPCh - 1);
        const float alpha = mc_mix(m, t[m.idx[0] * kPCh], t[m.idx[1] * kPCh], t[m.idx[2] * kPCh]);
        if constexpr (LOGP) {
            atomicAdd(&a.logp[e.x], win ? logf(alpha) : log1pf(-alpha));
        } else {
            const float gl = a.sel.grad_logp[e.x];
            if (gl == 0.0f) return;
            // d log p / d alpha: 1 / alpha for the winner, -1 / (1 - alpha) in front of it
            const float da = win ? gl / alpha : -gl / (1.0f - alpha);
            float* g = a.grad_tex + static_cast<size_t>(tri) * V * kPCh + (kPCh - 1);
#pragma unroll
            for (int q = 0; q < 3; ++q)
                if (m.w[q] != 0.0f) atomicAdd(&g[m.idx[q] * kPCh], m.w[q] * da);
        }
    });
}

void launch_pfrag(const PFragArgs& a, bool logp, hipStream_t s) {
    const dim3 grid(log_blocks(a.log));
    if (logp) hipLaunchKernelGGL(pfrag_kernel<true>, grid, dim3(256), 0, s, a);
    else hipLaunchKernelGGL(pfrag_kernel<false>, grid, dim3(256), 0, s, a);
}

// ---------------------------------------------------------------------------
// winners (backward)
// ---------------------------------------------------------------------------

constexpr int kPStage = 64 + 4;   // staged row: 64 pixels, padded

// The world-space gradient of the vertices of the winner's triangle from the
// gradient of its perspective-correct barycentrics (db1, db2) and the edge
// weights (ex, ey), in float64 at the snapped positions (every edge function
// an exact integer), with the clip coordinates recomputed in the setup's
// float32 order.
__device__ __forceinline__ void vertex_grad(const ViewDesc& vd, const TriRec& tr, const float* __restrict__ vp,
                                            int px, int py, const double (&E)[3], double db1, double db2, double ex,
                                            double ey, double (&gw)[9]) {
    const double inv_a = 1.0 / ((E[0] + E[1]) + E[2]);
    double fb[3], iwv[3];
#pragma unroll
    for (int i = 0; i < 3; ++i) {
        fb[i] = E[i] * inv_a;
        iwv[i] = tr.iw[i];
    }
    const double tt[3] = {fb[0] * iwv[0], fb[1] * iwv[1], fb[2] * iwv[2]};
    const double inv_s = 1.0 / ((tt[0] + tt[1]) + tt[2]);
    const double bb[3] = {tt[0] * inv_s, tt[1] * inv_s, tt[2] * inv_s};
    const double db[3] = {0.0, db1, db2};
    const double dot = db[1] * bb[1] + db[2] * bb[2];
    double dbeta[3], diw[3];
#pragma unroll
    for (int i = 0; i < 3; ++i) {
        const double dt = (db[i] - dot) * inv_s;
        dbeta[i] = dt * iwv[i];
        diw[i] = dt * fb[i];
    }
    const int32_t PX = kSnap * px + kSnap / 2, PY = kSnap * py + kSnap / 2;
    const double Ai = __builtin_fma(static_cast<double>(tr.X[1] - tr.X[0]), static_cast<double>(tr.Y[2] - tr.Y[0]),
                                    -(static_cast<double>(tr.Y[1] - tr.Y[0]) * static_cast<double>(tr.X[2] - tr.X[0])));
    const double inv_area = 65536.0 / Ai;   // 1 / (signed 2 x area in px^2)
    const double inv256 = 1.0 / 256.0;
    double gsx[3] = {0., 0., 0.}, gsy[3] = {0., 0., 0.};
#pragma unroll
    for (int i = 0; i < 3; ++i) {
        // beta_i = e_i / area with e_i = edge(v_p, v_q, pixel centre)
        const int p = i == 2 ? 0 : i + 1, q = i == 0 ? 2 : (i == 1 ? 0 : 1);
#pragma unroll
        for (int jv = 0; jv < 3; ++jv) {
            const int jp = jv == 2 ? 0 : jv + 1, jq = jv == 0 ? 2 : (jv == 1 ? 0 : 1);
            const double dax = static_cast<double>(tr.Y[jp] - tr.Y[jq]) * inv256;
            const double day = static_cast<double>(tr.X[jq] - tr.X[jp]) * inv256;
            double dex = 0., dey = 0.;
            if (jv == p) {
                dex = static_cast<double>(tr.Y[q] - PY) * inv256;
                dey = static_cast<double>(PX - tr.X[q]) * inv256;
            } else if (jv == q) {
                dex = static_cast<double>(PY - tr.Y[p]) * inv256;
                dey = static_cast<double>(tr.X[p] - PX) * inv256;
            }
            gsx[jv] += dbeta[i] * (dex - fb[i] * dax) * inv_area;
            gsy[jv] += dbeta[i] * (dey - fb[i] * day) * inv_area;
        }
    }
    // edge term (Section 3.2): the boundaries this pixel occludes move with its
    // surface point, w beta_i e on the screen position of vertex i
#pragma unroll
    for (int jv = 0; jv < 3; ++jv) {
        gsx[jv] += ex * fb[jv];
        gsy[jv] += ey * fb[jv];
    }
    // screen position (W/2 (c_x / c_w) + W/2, H/2 - H/2 (c_y / c_w)) and 1/w -> clip -> world
    const double hw = 0.5 * vd.W, hh = 0.5 * vd.H;
#pragma unroll
    for (int jv = 0; jv < 3; ++jv) {
        const float x = vp[3 * jv], y = vp[3 * jv + 1], z = vp[3 * jv + 2];
        float cc[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) {   // the setup's transform
            float acc = vd.M[j * 4 + 3];
            acc = __builtin_fmaf(vd.M[j * 4 + 0], x, acc);
            acc = __builtin_fmaf(vd.M[j * 4 + 1], y, acc);
            acc = __builtin_fmaf(vd.M[j * 4 + 2], z, acc);
            cc[j] = acc;
        }
        const double cx = cc[0], cy = cc[1], iw = 1.0 / static_cast<double>(cc[3]);
        const double gc0 = gsx[jv] * hw * iw;
        const double gc1 = -gsy[jv] * hh * iw;
        const double gc3 = (-gsx[jv] * hw * cx + gsy[jv] * hh * cy - diw[jv]) * (iw * iw);
#pragma unroll
        for (int k = 0; k < 3; ++k)
            gw[3 * jv + k] = static_cast<double>(vd.M[k]) * gc0 + static_cast<double>(vd.M[4 + k]) * gc1 +
                             static_cast<double>(vd.M[12 + k]) * gc3;
    }
}

// One weight-gradient block of the wave's 64 pixels on the matrix cores:
// D[j][c] += sum over pixels of delta[p][j] act[p][c] (v_mfma_f32_16x16x4f32,
// K = pixels: step s of lane group grp takes pixel 16 grp + s, so that lane
// (grp, col) reads 16 consecutive pixels of unit col from the stage: act in
// st[0], delta in st[1]), and bsum += the lane's 16 values of delta unit col (the bias gradient).
__device__ __forceinline__ void wgrad_staged(const float (*st)[kPIn][kPStage], int lane, f4v& acc, float& bsum) {
    const int col = lane & 15, grp = lane >> 4;
    wave_fence();
    float4 A4[4], B4[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        A4[q] = *reinterpret_cast<const float4*>(&st[1][col][16 * grp + 4 * q]);
        B4[q] = *reinterpret_cast<const float4*>(&st[0][col][16 * grp + 4 * q]);
    }
    wave_fence();
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        acc = mfma4(A4[q].x, B4[q].x, acc);
        acc = mfma4(A4[q].y, B4[q].y, acc);
        acc = mfma4(A4[q].z, B4[q].z, acc);
        acc = mfma4(A4[q].w, B4[q].w, acc);
        bsum += (A4[q].x + A4[q].y) + (A4[q].z + A4[q].w);
    }
}

__device__ __forceinline__ void wgrad_block(float (*st)[kPIn][kPStage], const float (&act)[kPIn], const float* delta,
                                            int nd, int lane, f4v& acc, float& bsum) {
#pragma unroll
    for (int u = 0; u < kPIn; ++u) {
        st[0][u][lane] = act[u];
        st[1][u][lane] = u < nd ? delta[u] : 0.0f;
    }
    wgrad_staged(st, lane, acc, bsum);
}

__global__ __launch_bounds__(256) void pwinner_bwd_kernel(PWinArgs a) {
    __shared__ __align__(16) float stage[4][2][kPIn][kPStage];
    const int tid = threadIdx.x, w = tid >> 6, lane = tid & 63, col = lane & 15, grp = lane >> 4;
    float (*st)[kPIn][kPStage] = stage[w];
    // contiguous runs of 64-pixel batches per wave, the waves of one XCD on adjacent runs
    const int64_t nbat = (a.P + 63) / 64;
    const int64_t nw = static_cast<int64_t>(gridDim.x) * 4;
    const int64_t wid = static_cast<int64_t>(xcd_block()) * 4 + w;
    const int64_t bbeg = nbat * wid / nw, bend = nbat * (wid + 1) / nw;
    const int R = a.R, n = 1 << R, V = mc_count(R);
    cfloat* mp = as_const(a.mlp);
    gfloat* tex = as_global(a.tex);
    f4v acc0 = {0.f, 0.f, 0.f, 0.f}, acc1 = {0.f, 0.f, 0.f, 0.f}, acc2 = {0.f, 0.f, 0.f, 0.f};
    float ab0 = 0.f, ab1 = 0.f, ab2 = 0.f;
    for (int64_t b = bbeg; b < bend; ++b) {
        const int64_t p = b * 64 + lane;
        uint64_t key = kBgKey;
        if (p < a.P) key = a.vis[p];
        const bool on = key != kBgKey;
        float gc[3] = {0.f, 0.f, 0.f};
        float ex = 0.f, ey = 0.f;
        if (on) {
            gc[0] = a.grad_color[3 * p];
            gc[1] = a.grad_color[3 * p + 1];
            gc[2] = a.grad_color[3 * p + 2];
            if (a.edge_w) {
                const float2 e = a.edge_w[p];
                ex = e.x;
                ey = e.y;
            }
        }
        const bool cpath = on && (gc[0] != 0.f || gc[1] != 0.f || gc[2] != 0.f);
        const bool active = cpath || (on && (ex != 0.f || ey != 0.f));
        int x = 0, y = 0, v = 0;
        uint32_t tri = 0;
        TriRec tr{};
        float b1 = 0.f, b2 = 0.f;
        double E[3] = {1.0, 0.0, 0.0};
        Micro m{};
        float4 tv[3][2];
        float feat[kPCh];
        if (active) {
            v = view_of_pixel(a.views, a.V, p);
            const ViewDesc& vd = a.views[v];
            const uint32_t local = static_cast<uint32_t>(p - vd.pix_base);
            y = static_cast<int>(local / static_cast<uint32_t>(vd.W));
            x = static_cast<int>(local - static_cast<uint32_t>(y) * static_cast<uint32_t>(vd.W));
            tri = static_cast<uint32_t>(key);
            tr = a.recs[vd.rec_base + tri];
            frag_bary(tr, x, y, b1, b2, E);
            m = micro_of(n, b1, b2);
        }
        // --- colour path: recompute in the forward's arithmetic, then the data backward ---
        float in[kPIn], h1[kPHid], h2[kPHid], d1[kPHid], d2[kPHid], d3[kPOut];
        float dfeat[kPFeat];
#pragma unroll
        for (int u = 0; u < kPHid; ++u) {
            in[u] = 0.f;
            h1[u] = 0.f;
            h2[u] = 0.f;
            d1[u] = 0.f;
            d2[u] = 0.f;
        }
#pragma unroll
        for (int c = 0; c < kPOut; ++c) d3[c] = 0.f;
#pragma unroll
        for (int c = 0; c < kPFeat; ++c) dfeat[c] = 0.f;
        if (cpath) {
            const ViewDesc& vd = a.views[v];
            fetch_texel(tex, tri, V, m, tv, feat);
#pragma unroll
            for (int c = 0; c < kPFeat; ++c) in[c] = feat[c];
            float d[3];
            view_dir(vd.Mi, vd.W, vd.H, x, y, d);
            sh2(d, in + kPFeat);
            float o[kPOut];
            dense<kPIn, kPHid, true>(mp + kPW0, mp + kPB0, in, h1);
            dense<kPHid, kPHid, true>(mp + kPW1, mp + kPB1, h1, h2);
            dense<kPHid, kPOut, false>(mp + kPW2, mp + kPB2, h2, o);
            const float A = feat[3];
            float dA = 0.f;
#pragma unroll
            for (int c = 0; c < kPOut; ++c) {
                const float mm = sigmoid_c(o[c]);
                dfeat[c] = A * gc[c];
                dA = __builtin_fmaf(gc[c], feat[c] - mm, dA);
                d3[c] = (1.0f - A) * gc[c] * (mm * (1.0f - mm));
            }
            dfeat[3] = dA;
            // through the output layer and the ReLU gates of the recompute (the forward's own)
#pragma unroll
            for (int u = 0; u < kPHid; ++u) {
                float s = 0.f;
#pragma unroll
                for (int c = 0; c < kPOut; ++c) s = __builtin_fmaf(mp[kPW2 + c * kPHid + u], d3[c], s);
                d2[u] = h2[u] > 0.f ? s : 0.f;
            }
#pragma unroll
            for (int u = 0; u < kPHid; ++u) {
                float s = 0.f;
#pragma unroll
                for (int j = 0; j < kPHid; ++j) s = __builtin_fmaf(mp[kPW1 + j * kPHid + u], d2[j], s);
                d1[u] = h1[u] > 0.f ? s : 0.f;
            }
#pragma unroll
            for (int c = 0; c < kPFeat; ++c) {
                float s = 0.f;
#pragma unroll
                for (int j = 0; j < kPHid; ++j) s = __builtin_fmaf(mp[kPW0 + j * kPIn + c], d1[j], s);
                dfeat[c] += s;   // the harmonics have no parameters
            }
        }
        // --- MLP weight gradients over the wave's pixels (lanes without a colour path add zeros) ---
        if (__ballot(cpath)) {
            wgrad_block(st, in, d1, kPHid, lane, acc0, ab0);
            wgrad_block(st, h1, d2, kPHid, lane, acc1, ab1);
            wgrad_block(st, h2, d3, kPOut, lane, acc2, ab2);
        }
        // --- features -> the micro-triangle's grid vertices; along (b1, b2) -> the triangle ---
        double gw[9] = {0., 0., 0., 0., 0., 0., 0., 0., 0.};
        if (active) {
            float dfu = 0.f, dfv = 0.f;
            if (cpath) {
                float* gt = a.grad_tex + static_cast<size_t>(tri) * V * kPCh;
#pragma unroll
                for (int q = 0; q < 3; ++q) {
                    if (m.w[q] == 0.0f) continue;
#pragma unroll
                    for (int c = 0; c < kPFeat; ++c)
                        if (dfeat[c] != 0.0f) atomicAdd(&gt[m.idx[q] * kPCh + c], m.w[q] * dfeat[c]);
                }
                // upright: w = (1 - fu - fv, fu, fv); inverted: w = (fu + fv - 1, 1 - fv, 1 - fu)
#pragma unroll
                for (int c = 0; c < kPFeat; ++c) {
                    const float t0 = c < 4 ? (&tv[0][0].x)[c] : (&tv[0][1].x)[c - 4];
                    const float t1 = c < 4 ? (&tv[1][0].x)[c] : (&tv[1][1].x)[c - 4];
                    const float t2 = c < 4 ? (&tv[2][0].x)[c] : (&tv[2][1].x)[c - 4];
                    dfu = __builtin_fmaf(dfeat[c], m.inv ? t0 - t2 : t1 - t0, dfu);
                    dfv = __builtin_fmaf(dfeat[c], m.inv ? t0 - t1 : t2 - t0, dfv);
                }
            }
            vertex_grad(a.views[v], tr, a.verts + static_cast<size_t>(tri) * 9, x, y, E,
                        static_cast<double>(dfu) * n, static_cast<double>(dfv) * n, ex, ey, gw);
        }
        // --- the vertex gradient summed over each run of equal triangles among the
        // wave's lanes (neighbouring pixels of a row mostly share their winner), one
        // set of float64 atomics per run ---
        if (__ballot(active)) {
            const uint32_t tk = active ? tri : 0xFFFFFFFFu;
            const uint32_t tp = static_cast<uint32_t>(__shfl_up(static_cast<int>(tk), 1, 64));
            const bool head = lane == 0 || tp != tk;
            const uint64_t heads = __ballot(head);
            double* sd = reinterpret_cast<double*>(&st[0][0][0]);   // [9][64], within the stage
#pragma unroll
            for (int k = 0; k < 9; ++k) sd[k * 64 + lane] = gw[k];
            wave_fence();
            if (head && active) {
                const uint64_t above = lane == 63 ? 0ull : (heads & (~0ull << (lane + 1)));
                const int end = above ? __builtin_ctzll(above) : 64;
                double acc[9] = {0., 0., 0., 0., 0., 0., 0., 0., 0.};
                for (int l = lane; l < end; ++l)
#pragma unroll
                    for (int k = 0; k < 9; ++k) acc[k] += sd[k * 64 + l];
                double* gv = a.gvert + static_cast<size_t>(tri) * 9;
#pragma unroll
                for (int k = 0; k < 9; ++k)
                    if (acc[k] != 0.0) atomicAdd(&gv[k], acc[k]);
            }
            wave_fence();
        }
    }
    // the wave's partial row of the MLP gradient (D[4 grp + i][col] of each block)
    float* row = a.mlp_partial + static_cast<size_t>(blockIdx.x * 4 + w) * kPParams;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        row[kPW0 + (4 * grp + i) * kPIn + col] = acc0[i];
        row[kPW1 + (4 * grp + i) * kPHid + col] = acc1[i];
        if (grp == 0 && i < kPOut) row[kPW2 + i * kPHid + col] = acc2[i];
    }
    ab0 += __shfl_xor(ab0, 16, 64);
    ab0 += __shfl_xor(ab0, 32, 64);
    ab1 += __shfl_xor(ab1, 16, 64);
    ab1 += __shfl_xor(ab1, 32, 64);
    ab2 += __shfl_xor(ab2, 16, 64);
    ab2 += __shfl_xor(ab2, 32, 64);
    if (grp == 0) {
        row[kPB0 + col] = ab0;
        row[kPB1 + col] = ab1;
        if (col < kPOut) row[kPB2 + col] = ab2;
    }
}

int pwinner_blocks(int num_cus) { return ((num_cus * 2 + kXcds - 1) / kXcds) * kXcds; }

void launch_pwinner_bwd(const PWinArgs& a, hipStream_t s) {
    if (a.n_blocks <= 0) return;
    hipLaunchKernelGGL(pwinner_bwd_kernel, dim3(static_cast<unsigned>(a.n_blocks)), dim3(256), 0, s, a);
}

// ---------------------------------------------------------------------------
// backward over the triangle-sorted fragment list
// ---------------------------------------------------------------------------

// The 16-16-16-3 MLP on the matrix cores, in a wave's registers: every operand
// is one value per lane and step. Layout of the activations as in the grid
// form's backward (element i of an f4v: unit 4 i + grp of the fragment 16 nb +
// col), the contractions in ascending unit order, so that the hidden layers,
// the logits and the data gradients are bit for bit those of the scalar
// chains (dense, and sums over j ascending from 0).
struct PMlp {
    f4v l0, l1, lo, l1T, l0T, b0, b1;
    float loT, bo;
    __device__ __forceinline__ void load(const float* __restrict__ m, int lane) {
        const int col = lane & 15, grp = lane >> 4, u = unit_of(col);
        const bool out = (col & 3) == 0 && (col >> 2) < kPOut;   // output g is element 0 of lane group g
#pragma unroll
        for (int s = 0; s < 4; ++s) {
            const int k = 4 * s + grp;
            l0[s] = m[kPW0 + u * kPIn + k];
            l1[s] = m[kPW1 + u * kPHid + k];
            lo[s] = out ? m[kPW2 + (col >> 2) * kPHid + k] : 0.0f;
            l1T[s] = m[kPW1 + k * kPHid + u];
            l0T[s] = u < kPFeat ? m[kPW0 + k * kPIn + u] : 0.0f;   // the harmonics take no gradient
            b0[s] = m[kPB0 + k];
            b1[s] = m[kPB1 + k];
        }
        loT = grp < kPOut ? m[kPW2 + grp * kPHid + u] : 0.0f;
        bo = grp < kPOut ? m[kPB2 + grp] : 0.0f;
    }
};
__device__ __forceinline__ f4v pmlp_dot(const f4v& w, const f4v& x, f4v acc) {
#pragma unroll
    for (int s = 0; s < 4; ++s) acc = mfma4(w[s], x[s], acc);
    return acc;
}
// Element i of block nb to row 4 i + grp of a stage, the fragment's column.
__device__ __forceinline__ void stage_units(float (*st)[kPStage], const f4v (&v)[4], int lane) {
    const int col = lane & 15, grp = lane >> 4;
#pragma unroll
    for (int nb = 0; nb < 4; ++nb)
#pragma unroll
        for (int i = 0; i < 4; ++i) st[4 * i + grp][16 * nb + col] = v[nb][i];
}

// One wave per workgroup walks a contiguous range of the fragment list sorted
// by triangle (every winner, and the fragments in front of it where the pixel
// carries a score weight), 64 fragments per batch, and keeps the gradient of
// the current triangle's texture (V x 8) and its nine vertex sums in its LDS.
// Per fragment: its opacity lookup and the score term; per winner also the
// colour path of pwinner_bwd_kernel (recompute, blend, the MLP and its data and
// weight gradients on the matrix cores, features onto the three grid vertices,
// the float64 vertex chain with the edge term). Adds into the row are LDS
// atomics (two fragments of a run may share a grid vertex): of float64 where
// that fits (ptri_row64), because an LDS add of 64 float32 takes 194 cycles
// here, one lane after the other, and one of 64 float64 takes 10. When the
// triangle changes, the row goes to HBM: plain stores when the wave holds all
// of the triangle's fragments, float atomics when the triangle straddles two
// waves' ranges.
//
// LEVELS: the gradient of the learnable levels instead of the assembled
// texture's (the assembly's backward folded in). Every add is multiplied by
// tex (1 - tex) at its grid vertex (the sigmoid's derivative; the texels are
// the ones the fragment's lookups already read), which gives the gradient of
// the level-R sum. The rest is the restriction chain, the transpose of the
// lookups at the level-R vertices: the coincident coarse vertex takes weight
// 1, the two ends of the coarse edge that a vertex halves 1/2 each. Where level R
// itself is not learnable (it is not in the training's levels) its step is
// taken before the add: a fragment's three vertices lie in one coarse
// triangle, so its three corners take three sums each (corner_code), and the
// row is level R - 1 (153 vertices instead of 561 at R = 5: 9.9 KB of LDS, two
// waves per SIMD). When the triangle changes, the remaining steps run
// in LDS, gathering: level L - 1 in the stage buffer (free between batches),
// level L - 2 behind it, and so on, and each learnable level goes out. The
// restriction is linear, so a triangle split between two waves restricts
// each part and adds them. The seven fine-grid indices of every coarse
// vertex are tabulated once per workgroup (a neighbour outside the grid
// points at a zero vertex one past the level's last), so a restriction step
// is one table read and seven reads per (vertex, four channels).
//
// What bounds it: latency at two waves per SIMD, and the waves' uneven shares (a
// triangle costs a flush besides its fragments; with counters in the kernel the
// longest wave took 515 us, the average one 311). Runs from four places of
// the list per wave left the spread and cost the flushes of the triangles that
// they cut (432 us). Four 800 x 800 views of 50,000 triangles, levels 2..4 onto
// 5: 606 us with float32 rows of level 5 and the MLP on the vector ALUs, 381
// now.
constexpr int kPCoarse = 153 + 45 + 15 + 6 + 3 + 5;   // vertices of levels 4..0, each with its zero vertex
static_assert(kPCoarse * kPCh <= 2 * kPIn * kPStage, "the coarse levels fit the stage buffer");

// The level of ptri_bwd_kernel's row, and its LDS: the row (planes of one channel,
// each with the zero vertex), then the tables of the coarser learnable levels.
__host__ __device__ constexpr int ptri_row_level(bool levels, int R, int Rtop) { return levels && Rtop < R ? R - 1 : R; }
// Rows of level 5 are float32: 36 KB of float64 leave three waves per CU, 18 KB
// six (a step with the separate backward, four 800 x 800 views of 50,000 triangles:
// 2,369 us in float64, 2,036 in float32); smaller ones do not bound the waves.
constexpr bool ptri_row64(int Rr) { return Rr < 5; }
static size_t ptri_lds(bool levels, int R, int Rmin, int Rtop) {
    const int Rr = ptri_row_level(levels, R, Rtop);
    size_t n = static_cast<size_t>(mc_count(Rr) + 1) * kPCh * (ptri_row64(Rr) ? sizeof(double) : sizeof(float));
    if (levels)
        for (int L = Rr - 1; L >= Rmin; --L) n += static_cast<size_t>(mc_count(L)) * sizeof(uint4);
    return n;
}

// Weights of a micro-triangle's vertices at the corners of the level below's
// triangle that holds it, in halves: bits 2 (3 q + k) for vertex q and corner
// k. Corners: 0 = (I, J), or (I + 1, J + 1) in an inverted triangle, 1 =
// (I + 1, J), 2 = (I, J + 1) with I = i / 2, J = j / 2; (pi, pj) = (i, j) & 1.
constexpr uint32_t corner_code_of(int inv, int pi, int pj) {
    const int vx[2][3] = {{0, 1, 0}, {1, 1, 0}}, vy[2][3] = {{0, 0, 1}, {1, 0, 1}};
    uint32_t code = 0;
    for (int q = 0; q < 3; ++q) {
        const int x = pi + vx[inv][q], y = pj + vy[inv][q];   // from (2 I, 2 J)
        const int dx = x & 1, dd = dx && (y & 1) ? 1 : 0, dy = (y & 1) && !dx ? 1 : 0;
        for (int e = 0; e < 2; ++e) {   // the two ends (twice the same one where coincident)
            const int I = (e ? x + dx : x - dx) / 2, J = (e ? y + dy - dd : y - dy + dd) / 2;
            const int k = I == 1 && J == 0 ? 1 : I == 0 && J == 1 ? 2 : 0;
            code += 1u << (2 * (3 * q + k));
        }
    }
    return code;
}
__device__ __forceinline__ uint32_t corner_code(bool inv, int pi, int pj) {
    const uint32_t u0 = pi ? corner_code_of(0, 1, 0) : corner_code_of(0, 0, 0);
    const uint32_t u1 = pi ? corner_code_of(0, 1, 1) : corner_code_of(0, 0, 1);
    const uint32_t v0 = pi ? corner_code_of(1, 1, 0) : corner_code_of(1, 0, 0);
    const uint32_t v1 = pi ? corner_code_of(1, 1, 1) : corner_code_of(1, 0, 1);
    return inv ? (pj ? v1 : v0) : (pj ? u1 : u0);
}
// the inverted coarse triangles: those of upright micro-triangles with both indices odd and of
// inverted ones with one or both odd
__device__ __forceinline__ bool corner_inverted(bool inv, int pi, int pj) { return inv ? (pi | pj) != 0 : (pi & pj) != 0; }

template <bool LEVELS, typename Row>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(2))) void ptri_bwd_kernel(PTriArgs a) {
    __shared__ __align__(16) float stage[2][kPIn][kPStage];
    __shared__ double vsum[9];
    extern __shared__ __align__(16) char s_row[];   // [8][Vr + 1] of Row, then the tables
    Row* const row = reinterpret_cast<Row*>(s_row);
    const int lane = threadIdx.x, col = lane & 15, grp = lane >> 4;
    float (*st)[kPIn][kPStage] = stage;
    const int R = a.R, n = 1 << R, NR = mc_count(R) * kPCh;
    const int Rr = ptri_row_level(LEVELS, R, a.Rtop), Vr = mc_count(Rr), Vp = Vr + 1;
    uint4* const s_tab = reinterpret_cast<uint4*>(row + kPCh * Vp);   // per coarse vertex: centre, six neighbours (16-bit)
    if constexpr (LEVELS) {   // the restriction tables of levels Rr - 1 down to Rmin, in that order
        int off = 0;
        for (int L = Rr; L > a.Rmin; --L) {
            const int nc = 1 << (L - 1), nfl = 1 << L, Vc = mc_count(L - 1), Vfl = mc_count(L);
            for (int q = lane; q < Vc; q += 64) {
                int I, J;
                mc_ij(nc, q, I, J);
                const int i = 2 * I, j = 2 * J;
                const uint32_t z = static_cast<uint32_t>(Vfl);   // the zero vertex
                const uint32_t c = mc_index(nfl, i, j);
                const uint32_t n1 = i + 1 + j <= nfl ? mc_index(nfl, i + 1, j) : z;
                const uint32_t n2 = i > 0 ? mc_index(nfl, i - 1, j) : z;
                const uint32_t n3 = i + j + 1 <= nfl ? mc_index(nfl, i, j + 1) : z;
                const uint32_t n4 = j > 0 ? mc_index(nfl, i, j - 1) : z;
                const uint32_t n5 = j > 0 ? mc_index(nfl, i + 1, j - 1) : z;   // i + 1 + j - 1 <= n always
                const uint32_t n6 = i > 0 ? mc_index(nfl, i - 1, j + 1) : z;
                s_tab[off + q] = make_uint4(c | (n1 << 16), n2 | (n3 << 16), n4 | (n5 << 16), n6);
            }
            off += Vc;
        }
    }
    PMlp mlp;
    mlp.load(a.mlp, lane);
    const float inf = opaque_inf();
    gfloat* tex = as_global(a.tex);
    const int64_t E = a.tri_off[a.T];
    const int64_t nb = (E + 63) / 64;
    const int64_t nw = gridDim.x;
    const int64_t wid = xcd_block();
    const int64_t bbeg = nb * wid / nw, bend = nb * (wid + 1) / nw;
    const int64_t f0 = bbeg * 64, f1 = bend * 64 < E ? bend * 64 : E;
    for (int k = lane; k < kPCh * Vp; k += 64) row[k] = Row(0);
    if (lane < 9) vsum[lane] = 0.0;
    f4v acc0 = {0.f, 0.f, 0.f, 0.f}, acc1 = {0.f, 0.f, 0.f, 0.f}, acc2 = {0.f, 0.f, 0.f, 0.f};
    float ab0 = 0.f, ab1 = 0.f, ab2 = 0.f;
    int cur = -1;   // triangle held in the row (wave-uniform)
    SharedEnds ends;
    ends.load(a.sorted, f0, f1, E);
    // four channels of a vertex's gradient out to its grid row: a plain store when
    // the wave owns the triangle, else atomics of the nonzero entries
    auto put = [&](float* __restrict__ g, float4 v, bool owned) __attribute__((always_inline)) {
        if (owned) {
            if (a.accumulate) {   // the outputs were zero-filled unless accumulating
                const float4 o = *reinterpret_cast<const float4*>(g);
                v = make_float4(o.x + v.x, o.y + v.y, o.z + v.z, o.w + v.w);
            }
            *reinterpret_cast<float4*>(g) = v;
        } else {
            if (v.x != 0.0f) atomicAdd(g, v.x);
            if (v.y != 0.0f) atomicAdd(g + 1, v.y);
            if (v.z != 0.0f) atomicAdd(g + 2, v.z);
            if (v.w != 0.0f) atomicAdd(g + 3, v.w);
        }
    };
    // the row goes out and is cleared
    auto flush = [&](int t) __attribute__((always_inline)) {
        wave_fence();
        int l = lane;   // opaque: no address of the flush is held in a register across batches
        asm volatile("" : "+v"(l));
        const bool owned = ends.owned(t);
        if (!LEVELS || Rr <= a.Rtop) {
            float* g = (LEVELS ? a.graw[Rr - a.Rmin] : a.grad_tex) + static_cast<size_t>(t) * Vr * kPCh;
#pragma unroll 1
            for (int e = l; e < 2 * Vr; e += 64) {
                const Row* s = row + (e & 1) * 4 * Vp + (e >> 1);
                const float4 v = make_float4(static_cast<float>(s[0]), static_cast<float>(s[Vp]),
                                             static_cast<float>(s[2 * Vp]), static_cast<float>(s[3 * Vp]));
                if (v.x != 0.0f || v.y != 0.0f || v.z != 0.0f || v.w != 0.0f) put(g + 4 * e, v, owned);
            }
        }
        if constexpr (LEVELS) {
            // a level onto the next: l per (coarse vertex, four channels), the neighbours
            // in a fixed order, an absent one read as the zero vertex
            const float4* src = nullptr;   // level L (null: the row)
            float4* dst = reinterpret_cast<float4*>(&st[0][0][0]);
            int off = 0;
            for (int L = Rr; L > a.Rmin; --L) {
                const int Vc = mc_count(L - 1);
                float* const g = L - 1 <= a.Rtop ? a.graw[L - 1 - a.Rmin] + static_cast<size_t>(t) * Vc * kPCh : nullptr;
#pragma unroll 1
                for (int e = l; e < 2 * Vc; e += 64) {
                    const uint4 ix = s_tab[off + (e >> 1)];
                    const int h = e & 1;
                    const uint32_t id[7] = {ix.x & 0xFFFFu, ix.x >> 16, ix.y & 0xFFFFu, ix.y >> 16,
                                            ix.z & 0xFFFFu, ix.z >> 16, ix.w};
                    float4 v;
                    if (src == nullptr) {
                        float o[4];
#pragma unroll
                        for (int c = 0; c < 4; ++c) {
                            const Row* s = row + (4 * h + c) * Vp;
                            const Row sd = ((((s[id[1]] + s[id[2]]) + s[id[3]]) + s[id[4]]) + s[id[5]]) + s[id[6]];
                            o[c] = static_cast<float>(s[id[0]] + Row(0.5) * sd);
                        }
                        v = make_float4(o[0], o[1], o[2], o[3]);
                    } else {
                        float4 s[7];
#pragma unroll
                        for (int k = 0; k < 7; ++k) s[k] = src[2 * id[k] + h];
                        v.x = s[0].x + 0.5f * (((((s[1].x + s[2].x) + s[3].x) + s[4].x) + s[5].x) + s[6].x);
                        v.y = s[0].y + 0.5f * (((((s[1].y + s[2].y) + s[3].y) + s[4].y) + s[5].y) + s[6].y);
                        v.z = s[0].z + 0.5f * (((((s[1].z + s[2].z) + s[3].z) + s[4].z) + s[5].z) + s[6].z);
                        v.w = s[0].w + 0.5f * (((((s[1].w + s[2].w) + s[3].w) + s[4].w) + s[5].w) + s[6].w);
                    }
                    dst[e] = v;
                    if (g && (v.x != 0.0f || v.y != 0.0f || v.z != 0.0f || v.w != 0.0f)) put(g + 4 * e, v, owned);
                }
                if (l < 2) dst[Vc * 2 + l] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);   // the level's zero vertex
                off += Vc;
                wave_fence();
                src = dst;
                dst += (Vc + 1) * 2;
            }
        }
#pragma unroll 1
        for (int k = l; k < kPCh * Vp * static_cast<int>(sizeof(Row)) / 16; k += 64)
            reinterpret_cast<float4*>(s_row)[k] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
        if (l < 9) {
            const double v = vsum[l];
            vsum[l] = 0.0;
            if (v != 0.0) atomicAdd(&a.gvert[static_cast<size_t>(t) * 9 + l], v);
        }
        wave_fence();
    };
    // Memory is pipelined across batches: a batch's records are loaded two
    // batches ahead, and its per-fragment loads (the opacity texels; for a
    // winner its eight-channel texels, colour gradient and edge weights) are
    // issued before the previous batch's adds into the row and its flush, so
    // that their latency falls behind that work.
    struct Pre {
        FragRec fr;
        bool on;
        Micro m;
        float s7[3];        // the opacity texels of the micro-triangle's vertices
        float gc[3];        // the winner's colour gradient
        float ex, ey;       // ... and its pixel's edge weights
        float4 tv[3][2];    // ... and its eight-channel texels
    };
    auto load_rec = [&](int64_t b, FragRec& fr) __attribute__((always_inline)) {
        const int64_t fi = b * 64 + lane;
        fr = {make_uint2(0u, 0u), make_uint2(0u, 0u), make_uint2(0u, 0u)};
        if (b < bend && fi < E) fr = a.sorted[fi];
    };
    auto issue = [&](const FragRec& fr, int64_t b, Pre& P) __attribute__((always_inline)) {
        P.fr = fr;
        P.on = b < bend && b * 64 + lane < E;
        P.m = Micro{};
        P.ex = P.ey = 0.f;
#pragma unroll
        for (int q = 0; q < 3; ++q) {
            P.s7[q] = 0.f;
            P.gc[q] = 0.f;
        }
        if (P.on) {
            const uint32_t tri = fr.p0.y & 0x7FFFFFFFu;
            P.m = micro_of(n, __uint_as_float(fr.p1.x), __uint_as_float(fr.p1.y));
            gfloat* t7 = tex + static_cast<size_t>(tri) * NR + (kPCh - 1);
#pragma unroll
            for (int q = 0; q < 3; ++q) P.s7[q] = t7[P.m.idx[q] * kPCh];
            if (fr.p0.y >> 31) {   // a winner
                const uint32_t p = fr.p0.x;
#pragma unroll
                for (int c = 0; c < 3; ++c) P.gc[c] = a.grad_color[3 * static_cast<size_t>(p) + c];
                if (a.edge_w) {
                    const float2 e = a.edge_w[p];
                    P.ex = e.x;
                    P.ey = e.y;
                }
                gfloat4* g = reinterpret_cast<gfloat4*>(tex + static_cast<size_t>(tri) * NR);
#pragma unroll
                for (int q = 0; q < 3; ++q) {
                    P.tv[q][0] = g[2 * P.m.idx[q]];
                    P.tv[q][1] = g[2 * P.m.idx[q] + 1];
                }
            }
        }
    };
    Pre nx;
    FragRec rec1;
    {
        FragRec rec0;
        load_rec(bbeg, rec0);
        issue(rec0, bbeg, nx);
        load_rec(bbeg + 1, rec1);
    }
    for (int64_t b = bbeg; b < bend; ++b) {
        const Pre P = nx;       // this batch's records and loads
        FragRec rec2;           // the records two batches ahead
        load_rec(b + 2, rec2);
        const FragRec& fr = P.fr;
        const bool on = P.on;
        const uint32_t tri = on ? (fr.p0.y & 0x7FFFFFFFu) : 0xFFFFFFFFu;
        const bool win = on && (fr.p0.y >> 31) != 0u;
        const float gl = a.score ? __uint_as_float(fr.x.x) : 0.0f;
        const Micro& m = P.m;
        const float(&s7)[3] = P.s7;
        const float alpha = on ? mc_mix(m, s7[0], s7[1], s7[2]) : 1.0f;
        // d log p / d alpha: 1 / alpha for the winner, -1 / (1 - alpha) in front of it
        const float da = gl == 0.0f ? 0.0f : (win ? gl / alpha : -gl / (1.0f - alpha));
        // --- the winner's colour path ---
        const float(&gc)[3] = P.gc;
        const float ex = P.ex, ey = P.ey;
        int x = 0, y = 0, v = 0;
        if (win) {
            const uint32_t p = fr.p0.x;
            v = static_cast<int>(fr.x.y);
            const ViewDesc& vd = a.views[v];
            const uint32_t local = p - static_cast<uint32_t>(vd.pix_base);
            y = static_cast<int>(local / static_cast<uint32_t>(vd.W));
            x = static_cast<int>(local - static_cast<uint32_t>(y) * static_cast<uint32_t>(vd.W));
        }
        const bool cpath = win && (gc[0] != 0.f || gc[1] != 0.f || gc[2] != 0.f);
        const bool vpath = cpath || (win && (ex != 0.f || ey != 0.f));
        // the winner's setup record and vertices, for its vertex chain after the MLP:
        // loaded before the MLP's last layer, whose products cover their latency
        TriRec tr{};
        float vx[9];
#pragma unroll
        for (int k = 0; k < 9; ++k) vx[k] = 0.f;
        auto load_tri = [&]() __attribute__((always_inline)) {
            if (vpath) {
                tr = a.recs[a.views[v].rec_base + tri];
#pragma unroll
                for (int k = 0; k < 9; ++k) vx[k] = a.verts[static_cast<size_t>(tri) * 9 + k];
            }
        };
        const float4(&tv)[3][2] = P.tv;
        float dfeat[kPFeat];
#pragma unroll
        for (int c = 0; c < kPFeat; ++c) dfeat[c] = 0.f;
        const uint64_t cp_mask = __ballot(cpath);
        if (cp_mask) {
            // The batch's MLP on the matrix cores, 16 fragments per block, the four
            // blocks' chains side by side (fragments without a colour path: zeros).
            // Between a fragment's own lane and its block's lanes the values go
            // through the stage.
            float feat[kPCh], in[kPIn];
#pragma unroll
            for (int u = 0; u < kPIn; ++u) in[u] = 0.f;
#pragma unroll
            for (int h = 0; h < 2; ++h) {   // the texels' interpolation, as fetch_texel
                feat[4 * h + 0] = mc_mix(m, tv[0][h].x, tv[1][h].x, tv[2][h].x);
                feat[4 * h + 1] = mc_mix(m, tv[0][h].y, tv[1][h].y, tv[2][h].y);
                feat[4 * h + 2] = mc_mix(m, tv[0][h].z, tv[1][h].z, tv[2][h].z);
                feat[4 * h + 3] = mc_mix(m, tv[0][h].w, tv[1][h].w, tv[2][h].w);
            }
            if (cpath) {
                const ViewDesc& vd = a.views[v];
#pragma unroll
                for (int c = 0; c < kPFeat; ++c) in[c] = feat[c];
                float d[3];
                view_dir(vd.Mi, vd.W, vd.H, x, y, d);
                sh2(d, in + kPFeat);
            }
#pragma unroll
            for (int u = 0; u < kPIn; ++u) st[0][u][lane] = in[u];
            wave_fence();
            f4v xin[4], h1[4], h2[4];
#pragma unroll
            for (int nb = 0; nb < 4; ++nb)
#pragma unroll
                for (int s = 0; s < 4; ++s) xin[nb][s] = st[0][4 * s + grp][16 * nb + col];
#pragma unroll
            for (int nb = 0; nb < 4; ++nb) {
                h1[nb] = pmlp_dot(mlp.l0, xin[nb], mlp.b0);
#pragma unroll
                for (int i = 0; i < 4; ++i) h1[nb][i] = relu(h1[nb][i], inf);
            }
#pragma unroll
            for (int nb = 0; nb < 4; ++nb) {
                h2[nb] = pmlp_dot(mlp.l1, h1[nb], mlp.b1);
#pragma unroll
                for (int i = 0; i < 4; ++i) h2[nb][i] = relu(h2[nb][i], inf);
            }
            // the sigmoid of output g in lane group g, to the fragment's lane
#pragma unroll
            for (int nb = 0; nb < 4; ++nb) {
                const f4v o = pmlp_dot(mlp.lo, h2[nb], f4v{mlp.bo, 0.f, 0.f, 0.f});
                st[1][grp][16 * nb + col] = sigmoid_c(o[0]);
                // zeros where the fragment has no colour path: they take no part below
                const bool cp = (cp_mask >> (16 * nb + col)) & 1u;
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    h1[nb][i] = cp ? h1[nb][i] : 0.0f;
                    h2[nb][i] = cp ? h2[nb][i] : 0.0f;
                }
            }
            wave_fence();
            float d3[kPOut];
            {
                const float A = feat[3];
                float dA = 0.f;
#pragma unroll
                for (int c = 0; c < kPOut; ++c) {
                    const float mm = st[1][c][lane];
                    dfeat[c] = cpath ? A * gc[c] : 0.0f;
                    dA = __builtin_fmaf(gc[c], feat[c] - mm, dA);
                    d3[c] = cpath ? (1.0f - A) * gc[c] * (mm * (1.0f - mm)) : 0.0f;
                }
                dfeat[3] = cpath ? dA : 0.0f;
            }
            wave_fence();
            // layer 2: the deltas' rows past kPOut hold what was there, and so do rows
            // of the product that nothing reads
#pragma unroll
            for (int c = 0; c < kPOut; ++c) st[1][c][lane] = d3[c];
            stage_units(st[0], h2, lane);
            wave_fence();
            f4v dl[4];
#pragma unroll
            for (int nb = 0; nb < 4; ++nb) {
                const float dO = grp < kPOut ? st[1][grp][16 * nb + col] : 0.0f;
                dl[nb] = mfma4(mlp.loT, dO, f4v{0.f, 0.f, 0.f, 0.f});
#pragma unroll
                for (int i = 0; i < 4; ++i) dl[nb][i] = h2[nb][i] > 0.0f ? dl[nb][i] : 0.0f;
            }
            wgrad_staged(st, lane, acc2, ab2);
            // layer 1
            stage_units(st[0], h1, lane);
            stage_units(st[1], dl, lane);
#pragma unroll
            for (int nb = 0; nb < 4; ++nb) {
                f4v d = pmlp_dot(mlp.l1T, dl[nb], f4v{0.f, 0.f, 0.f, 0.f});
#pragma unroll
                for (int i = 0; i < 4; ++i) d[i] = h1[nb][i] > 0.0f ? d[i] : 0.0f;
                dl[nb] = d;
            }
            wgrad_staged(st, lane, acc1, ab1);
            // layer 0
            stage_units(st[0], xin, lane);
            stage_units(st[1], dl, lane);
            f4v dx[4];
#pragma unroll
            for (int nb = 0; nb < 4; ++nb) dx[nb] = pmlp_dot(mlp.l0T, dl[nb], f4v{0.f, 0.f, 0.f, 0.f});
            wgrad_staged(st, lane, acc0, ab0);
#pragma unroll
            for (int nb = 0; nb < 4; ++nb) {
                st[0][grp][16 * nb + col] = dx[nb][0];
                st[0][4 + grp][16 * nb + col] = dx[nb][1];
            }
            wave_fence();
#pragma unroll
            for (int c = 0; c < kPFeat; ++c) dfeat[c] += cpath ? st[0][c][lane] : 0.0f;
            wave_fence();
        }
        load_tri();
        // along (b1, b2)
        float dfu = 0.f, dfv = 0.f;
        if (cpath) {
#pragma unroll
            for (int c = 0; c < kPFeat; ++c) {
                const float t0 = c < 4 ? (&tv[0][0].x)[c] : (&tv[0][1].x)[c - 4];
                const float t1 = c < 4 ? (&tv[1][0].x)[c] : (&tv[1][1].x)[c - 4];
                const float t2 = c < 4 ? (&tv[2][0].x)[c] : (&tv[2][1].x)[c - 4];
                dfu = __builtin_fmaf(dfeat[c], m.inv ? t0 - t2 : t1 - t0, dfu);
                dfv = __builtin_fmaf(dfeat[c], m.inv ? t0 - t1 : t2 - t0, dfv);
            }
        }
        // What the fragment adds to its three grid vertices, zero where it has no
        // weight or no gradient (LEVELS: times the sigmoid's derivative at the
        // grid vertex). Branches, products and float32 adds in the runs' loop took
        // 3,900 cycles per run of 23 fragments, the float64 adds alone 1,850.
        float add[3][kPCh];
#pragma unroll
        for (int q = 0; q < 3; ++q) {
            const bool wq = m.w[q] != 0.0f;
#pragma unroll
            for (int c = 0; c < kPCh; ++c) {
                const float tq = c == kPCh - 1 ? s7[q] : c < 4 ? (&tv[q][0].x)[c] : (&tv[q][1].x)[c - 4];
                const float wc = LEVELS ? m.w[q] * (tq * (1.0f - tq)) : m.w[q];
                const float g = c == kPCh - 1 ? da : dfeat[c];
                add[q][c] = wq && g != 0.0f ? wc * g : 0.0f;
            }
        }
        int vtx[3];
        if (LEVELS && Rr < R) {   // onto the corners of the coarse triangle
            const int pi = m.i & 1, pj = m.j & 1, I = m.i >> 1, J = m.j >> 1;
            const uint32_t code = corner_code(m.inv, pi, pj);
            const int r0 = mc_index(n >> 1, I, J), r1 = mc_index(n >> 1, I, J + 1);
            vtx[0] = corner_inverted(m.inv, pi, pj) ? r1 + 1 : r0;
            vtx[1] = r0 + 1;
            vtx[2] = r1;
            // 0, 1/2 or 1 (zero also times an infinity)
            float f[3][3];
#pragma unroll
            for (int q = 0; q < 3; ++q)
#pragma unroll
                for (int k = 0; k < 3; ++k) f[q][k] = 0.5f * static_cast<float>((code >> (2 * (3 * q + k))) & 3u);
#pragma unroll
            for (int c = 0; c < kPCh; ++c) {
                float o[3];
#pragma unroll
                for (int k = 0; k < 3; ++k)
                    o[k] = ((f[0][k] != 0.0f ? f[0][k] * add[0][c] : 0.0f) + (f[1][k] != 0.0f ? f[1][k] * add[1][c] : 0.0f)) +
                           (f[2][k] != 0.0f ? f[2][k] * add[2][c] : 0.0f);
#pragma unroll
                for (int k = 0; k < 3; ++k) add[k][c] = o[k];
            }
        } else {
#pragma unroll
            for (int q = 0; q < 3; ++q) vtx[q] = m.idx[q];
        }
        // --- the winner's vertex gradient (colour path and edge term), float64 ---
        double gw[9] = {0., 0., 0., 0., 0., 0., 0., 0., 0.};
        if (vpath) {
            const ViewDesc& vd = a.views[v];
            float pb1, pb2;
            double E3[3];
            frag_bary(tr, x, y, pb1, pb2, E3);
            vertex_grad(vd, tr, vx, x, y, E3, static_cast<double>(dfu) * n, static_cast<double>(dfv) * n, ex, ey, gw);
        }
        // the next batch's loads go out before this batch's adds and flush
        issue(rec1, b + 1, nx);
        rec1 = rec2;
        // --- into the wave's row, one run of equal triangles at a time ---
        const uint32_t tp = static_cast<uint32_t>(__shfl_up(static_cast<int>(tri), 1, 64));
        uint64_t heads = __ballot(lane == 0 || tp != tri);
        while (heads) {
            const int h = __builtin_ctzll(heads);
            heads &= heads - 1;
            const int t = __builtin_amdgcn_readlane(static_cast<int>(tri), h);
            if (t < 0) break;   // the sentinel run: empty lanes at the list's end
            if (t != cur) {
                if (cur >= 0) flush(cur);
                cur = t;
            }
            const int end = heads ? __builtin_ctzll(heads) : 64;
            const bool in_run = lane >= h && lane < end;
            if (in_run && da != 0.0f) {
#pragma unroll
                for (int q = 0; q < 3; ++q) atomicAdd(row + (kPCh - 1) * Vp + vtx[q], static_cast<Row>(add[q][kPCh - 1]));
            }
            if (in_run && cpath) {
#pragma unroll
                for (int q = 0; q < 3; ++q)
#pragma unroll
                    for (int c = 0; c < kPFeat; ++c) atomicAdd(row + c * Vp + vtx[q], static_cast<Row>(add[q][c]));
            }
            if (__ballot(in_run && vpath)) {   // the run's winners: vertex sums over the wave
                double vv[9], q[3];
#pragma unroll
                for (int k = 0; k < 9; ++k) vv[k] = in_run ? gw[k] : 0.0;
                wave_sum9(vv, q);
                if ((lane & 15) == 0) {   // row g's first lane: components c, c + 2 (and 4 in row 0)
                    const int g = lane >> 4, c0 = (g & 1) + 5 * (g >> 1);
                    vsum[c0] += q[0];
                    vsum[c0 + 2] += q[1];
                    if (g == 0) vsum[4] += q[2];
                }
            }
            wave_fence();
        }
    }
    if (cur >= 0) flush(cur);
    // the wave's partial row of the MLP gradient
    float* prow = a.mlp_partial + static_cast<size_t>(blockIdx.x) * kPParams;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        prow[kPW0 + (4 * grp + i) * kPIn + col] = acc0[i];
        prow[kPW1 + (4 * grp + i) * kPHid + col] = acc1[i];
        if (grp == 0 && i < kPOut) prow[kPW2 + i * kPHid + col] = acc2[i];
    }
    ab0 += __shfl_xor(ab0, 16, 64);
    ab0 += __shfl_xor(ab0, 32, 64);
    ab1 += __shfl_xor(ab1, 16, 64);
    ab1 += __shfl_xor(ab1, 32, 64);
    ab2 += __shfl_xor(ab2, 16, 64);
    ab2 += __shfl_xor(ab2, 32, 64);
    if (grp == 0) {
        prow[kPB0 + col] = ab0;
        prow[kPB1 + col] = ab1;
        if (col < kPOut) prow[kPB2 + col] = ab2;
    }
}

// The sorted path's grids (a finer one's texture gradient takes the per-pixel path).
bool ptri_sorted(int R) { return R <= 5; }

static size_t ptri_lds(const PTriArgs& a) { return ptri_lds(a.levels, a.R, a.Rmin, a.Rtop); }

// As many single-wave workgroups as are resident at once (the LDS row bounds them), a
// multiple of eight: the wave ranges are static, so a second round of workgroups
// would double the time.
using PTriKernel = void (*)(PTriArgs);
static PTriKernel ptri_kernel(bool levels, int R, int Rtop) {
    const bool wide = ptri_row64(ptri_row_level(levels, R, Rtop));
    if (levels) return wide ? ptri_bwd_kernel<true, double> : ptri_bwd_kernel<true, float>;
    return wide ? ptri_bwd_kernel<false, double> : ptri_bwd_kernel<false, float>;
}

int ptri_blocks(int num_cus, bool levels, int R, int Rmin, int Rtop) {
    int per_cu = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, ptri_kernel(levels, R, Rtop), 64,
                                                     ptri_lds(levels, R, Rmin, Rtop)) != hipSuccess ||
        per_cu < 1) {
        (void)hipGetLastError();
        per_cu = 1;
    }
    return (num_cus * per_cu / kXcds) * kXcds > 0 ? (num_cus * per_cu / kXcds) * kXcds : kXcds;
}

void launch_ptri_bwd(const PTriArgs& a, hipStream_t s) {
    if (a.n_blocks <= 0) return;
    hipLaunchKernelGGL(ptri_kernel(a.levels, a.R, a.Rtop), dim3(static_cast<unsigned>(a.n_blocks)), dim3(64), ptri_lds(a),
                       s, a);
}

__global__ __launch_bounds__(256) void pvert_finish_kernel(const double* __restrict__ g, float* __restrict__ out,
                                                           int64_t n, int accumulate) {
    const int64_t i = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
    if (i >= n) return;
    out[i] = static_cast<float>((accumulate ? static_cast<double>(out[i]) : 0.0) + g[i]);
}

void launch_pvert_finish(const double* g, float* out, int64_t n, bool accumulate, hipStream_t s) {
    if (n <= 0) return;
    hipLaunchKernelGGL(pvert_finish_kernel, dim3(static_cast<unsigned>((n + 255) / 256)), dim3(256), 0, s, g, out, n,
                       accumulate ? 1 : 0);
}

}  // namespace soup
