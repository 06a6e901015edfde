// The training step around the rasterizer (Section 3.4 "Loss function";
// Supplement "Hyperparameters").
//
//  * ssim_stats_kernel: per pixel and channel, the local statistics of the
//    SSIM map under an 11 x 11 Gaussian window (zero outside the image):
//    the three factors through which S depends on the window sums,
//        G1 = dS/dmu_x - 2 mu_x dS/dsigma_x^2 - mu_y dS/dsigma_xy,
//        G2 = dS/dsigma_x^2,   G3 = dS/dsigma_xy,
//    so that dS(q)/dx_p = w(p - q) (G1(q) + 2 x_p G2(q) + y_p G3(q)). It also
//    writes each pixel's share of the loss (the score term's weight), and each
//    workgroup the sum of its shares, in double.
//  * loss_sum_kernel: the loss from the workgroups' sums.
//  * ssim_grad_kernel: dL/dC = lambda sign(C - T) / (3P) minus
//    (1 - lambda) / (3P) times the window sums of G1, G2, G3 around p.
//    One thread per pixel of a 32 x 8 tile; the window is applied as two
//    11-tap passes over an LDS copy of the tile and its halo, columns first
//    (the halo's 42 columns for the tile's 8 rows, two rows per thread from
//    their 12 shared input rows), then rows (the tile's 32 columns).
//  * adam_kernel: Adam (vec = 1) or VectorAdam (vec = 3: one second moment
//    per 3-vector from its squared norm), one thread per vector.
#include <hip/hip_runtime.h>

#include "internal.hpp"

namespace soup {

namespace {

constexpr float kC1 = 0.0001f;  // 0.01^2
constexpr float kC2 = 0.0009f;  // 0.03^2
// The window statistics are formed from values shifted by this constant
// (colours and targets live in [0, 1]): variances and covariances do not
// change under a shift, and sigma^2 = E[x^2] - mu^2 then cancels far fewer
// digits in float32 (E[(x - 1/2)^2] <= 1/4 against E[x^2] <= 1). Padding
// outside the image is the shifted zero, -1/2; the means are shifted back.
constexpr float kShift = 0.5f;

// Both SSIM passes work on 32 x 8 pixel tiles, one thread per pixel. The
// tile plus its 5-pixel halo is staged in LDS (zeros outside the image: the
// zero padding of the definition) and filtered along columns for the tile's
// rows over the halo's columns (a thread takes two output rows of one
// column, whose windows share 10 of their 12 input rows), then along rows:
// 22 taps per map instead of 121. Columns first: for a tile wider than
// tall the first pass covers 42 x 8 positions instead of 18 x 32.
constexpr int kTW = 32, kTH = 8;
constexpr int kHW = kTW + 2 * kSsimR, kHH = kTH + 2 * kSsimR;
static_assert(kTH % 2 == 0, "the column pass takes output rows in pairs");

// The views of one launch: view i owns tiles [tile[i], tile[i + 1]), pixels from pix[i] in the
// caller's arrays and from stat[i] in the record array.
struct SsimView {
    int W, H, tx;
    const float* color;
    const float* target;
    float* gc;
    float* gl;
    float* stats;
};
__device__ __forceinline__ SsimView ssim_view(const SsimBatch& b, int tile, int& x0, int& y0) {
    int i = 0;
    while (i + 1 < b.n && b.tile[i + 1] <= tile) ++i;   // uniform
    SsimView v;
    v.W = b.w[i];
    v.H = b.h[i];
    v.tx = (v.W + kTW - 1) / kTW;
    const int t = tile - b.tile[i];
    x0 = (t % v.tx) * kTW;
    y0 = (t / v.tx) * kTH;
    v.color = b.color + 3 * b.pix[i];
    v.target = b.target + 3 * b.pix[i];
    v.gc = b.grad_color + 3 * b.pix[i];
    v.gl = b.grad_logp + b.pix[i];
    v.stats = b.stats + 12 * (b.pix[i] - b.pix[0]);
    return v;
}

// All views of a batch in one launch, tiles dealt by stride to at most kSumParts
// workgroups, two rounds of the four per CU that the LDS (39 KB) admits: a launch
// per view left the GPU part empty for small views, and one
// float atomic per 32 x 8 tile on the loss queued behind each other. The two
// passes' sums are fused multiply-adds: VALU work bounds both kernels, and a
// separate multiply and add was twice the instructions (four views, 1.96 Mpixel:
// statistics 153 -> 83 us, gradient 69 -> 50).
__global__ void __launch_bounds__(256) ssim_stats_kernel(SsimBatch b, float lam, float inv_n, SsimWindow win,
                                                         double* __restrict__ parts) {
    __shared__ float in[kHH][kHW][6];   // colour rgb, target rgb
    __shared__ float vs[kTH][15][kHW];  // column sums: x, y, x^2, y^2, xy per channel
    __shared__ double part[4];
    double total = 0.0;
    for (int tile = blockIdx.x; tile < b.tile[b.n]; tile += gridDim.x) {
        int tx0, ty0;
        const SsimView v = ssim_view(b, tile, tx0, ty0);
        const int W = v.W, H = v.H;
        for (int i = threadIdx.x; i < kHH * kHW; i += 256) {
            const int r = i / kHW, cc = i % kHW;
            const int gx = tx0 + cc - kSsimR, gy = ty0 + r - kSsimR;
            const bool ok = gx >= 0 && gx < W && gy >= 0 && gy < H;
            const int64_t q = ok ? static_cast<int64_t>(gy) * W + gx : 0;
#pragma unroll
            for (int c = 0; c < 3; ++c) {
                in[r][cc][c] = (ok ? v.color[q * 3 + c] : 0.0f) - kShift;
                in[r][cc][3 + c] = (ok ? v.target[q * 3 + c] : 0.0f) - kShift;
            }
        }
        __syncthreads();
        // columns: output rows 2 pr and 2 pr + 1 of halo column cc, from input
        // rows 2 pr .. 2 pr + 11 (row 2 pr + k is tap k of the first, k - 1 of the second)
        for (int i = threadIdx.x; i < kHW * (kTH / 2); i += 256) {
            const int cc = i % kHW, pr = i / kHW;
            float a0[15], a1[15];
#pragma unroll
            for (int j = 0; j < 15; ++j) {
                a0[j] = 0.0f;
                a1[j] = 0.0f;
            }
#pragma unroll
            for (int k = 0; k <= 2 * kSsimR + 1; ++k) {
                const float* px = in[2 * pr + k][cc];
                float v15[15];
#pragma unroll
                for (int c = 0; c < 3; ++c) {
                    const float x = px[c], y = px[3 + c];
                    v15[c] = x;
                    v15[3 + c] = y;
                    v15[6 + c] = x * x;
                    v15[9 + c] = y * y;
                    v15[12 + c] = x * y;
                }
                if (k <= 2 * kSsimR) {
                    const float w = win.g[k];
#pragma unroll
                    for (int j = 0; j < 15; ++j) a0[j] = __builtin_fmaf(w, v15[j], a0[j]);
                }
                if (k >= 1) {
                    const float w = win.g[k - 1];
#pragma unroll
                    for (int j = 0; j < 15; ++j) a1[j] = __builtin_fmaf(w, v15[j], a1[j]);
                }
            }
#pragma unroll
            for (int j = 0; j < 15; ++j) {
                vs[2 * pr][j][cc] = a0[j];
                vs[2 * pr + 1][j][cc] = a1[j];
            }
        }
        __syncthreads();
        const int lx = threadIdx.x % kTW, ly = threadIdx.x / kTW;
        const int x = tx0 + lx, y = ty0 + ly;
        if (x < W && y < H) {
            float sm[15];
#pragma unroll
            for (int j = 0; j < 15; ++j) sm[j] = 0.0f;
#pragma unroll
            for (int k = 0; k <= 2 * kSsimR; ++k) {
                const float w = win.g[k];
#pragma unroll
                for (int j = 0; j < 15; ++j) sm[j] = __builtin_fmaf(w, vs[ly][j][lx + k], sm[j]);
            }
            const int64_t p = static_cast<int64_t>(y) * W + x;
            float4* st = reinterpret_cast<float4*>(v.stats + p * 12);
            float rec[12];
            float share = 0.0f;
#pragma unroll
            for (int c = 0; c < 3; ++c) {
                const float sx = sm[c], sy = sm[3 + c];   // shifted means
                const float vx = sm[6 + c] - sx * sx, vy = sm[9 + c] - sy * sy, cxy = sm[12 + c] - sx * sy;
                const float mx = sx + kShift, my = sy + kShift;
                const float A1 = 2.0f * mx * my + kC1, A2 = 2.0f * cxy + kC2;
                const float B1 = mx * mx + my * my + kC1, B2 = vx + vy + kC2;
                const float S = (A1 * A2) / (B1 * B2);
                const float dS_dmx = 2.0f * my * A2 / (B1 * B2) - S * 2.0f * mx / B1;
                const float dS_dvx = -S / B2;
                const float dS_dcxy = 2.0f * A1 / (B1 * B2);
                // G1 in shifted coordinates: the gradient pass pairs it with shifted values
                rec[c] = dS_dmx - 2.0f * sx * dS_dvx - sy * dS_dcxy;
                rec[3 + c] = dS_dvx;
                rec[6 + c] = dS_dcxy;
                rec[9 + c] = 0.0f;
                const float d = v.color[p * 3 + c] - v.target[p * 3 + c];
                share += lam * fabsf(d) + (1.0f - lam) * (1.0f - S);
            }
            st[0] = make_float4(rec[0], rec[1], rec[2], rec[3]);
            st[1] = make_float4(rec[4], rec[5], rec[6], rec[7]);
            st[2] = make_float4(rec[8], rec[9], rec[10], rec[11]);
            share *= inv_n;
            v.gl[p] = share;
            total += static_cast<double>(share);
        }
        // (the next tile's loads write `in`, which every thread has left behind at the last barrier,
        // and its column pass writes vs after another barrier)
    }
    if (!parts) return;
    for (int o = 32; o > 0; o >>= 1) total += __shfl_xor(total, o, 64);
    if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = total;
    __syncthreads();
    if (threadIdx.x == 0) parts[blockIdx.x] = (part[0] + part[1]) + (part[2] + part[3]);
}

// The loss from a batch's n parts, added in a fixed order; the total of the batches so far is a double
// behind them until the last one. One workgroup.
__global__ void __launch_bounds__(256) loss_sum_kernel(double* __restrict__ parts, int n, int add, int last,
                                                       float* __restrict__ out) {
    __shared__ double s_sum[4];
    double v = 0.0;
#pragma unroll
    for (int i = 0; i < kSumParts / 256; ++i) {
        const int k = i * 256 + threadIdx.x;
        v += k < n ? parts[k] : 0.0;
    }
#pragma unroll
    for (int d = 32; d > 0; d >>= 1) v += __shfl_xor(v, d, 64);
    if ((threadIdx.x & 63) == 0) s_sum[threadIdx.x >> 6] = v;
    __syncthreads();
    if (threadIdx.x == 0) {
        const double total = (add ? parts[kSumParts] : 0.0) + ((s_sum[0] + s_sum[1]) + (s_sum[2] + s_sum[3]));
        if (last) *out = static_cast<float>(total);
        else parts[kSumParts] = total;
    }
}

__global__ void __launch_bounds__(256) ssim_grad_kernel(SsimBatch b, float lam, float inv_n, SsimWindow win) {
    __shared__ float in[kHH][kHW][9];   // G1, G2, G3 per channel (zero outside the image)
    __shared__ float vs[kTH][9][kHW];   // their column sums
    for (int tile = blockIdx.x; tile < b.tile[b.n]; tile += gridDim.x) {
        int tx0, ty0;
        const SsimView v = ssim_view(b, tile, tx0, ty0);
        const int W = v.W, H = v.H;
        for (int i = threadIdx.x; i < kHH * kHW; i += 256) {
            const int r = i / kHW, cc = i % kHW;
            const int gx = tx0 + cc - kSsimR, gy = ty0 + r - kSsimR;
            if (gx >= 0 && gx < W && gy >= 0 && gy < H) {
                // a record is G1[3] G2[3] G3[3] and three unused floats: three 16-byte loads
                const float4* st = reinterpret_cast<const float4*>(v.stats + (static_cast<int64_t>(gy) * W + gx) * 12);
                const float4 r0 = st[0], r1 = st[1], r2 = st[2];
                in[r][cc][0] = r0.x;
                in[r][cc][1] = r0.y;
                in[r][cc][2] = r0.z;
                in[r][cc][3] = r0.w;
                in[r][cc][4] = r1.x;
                in[r][cc][5] = r1.y;
                in[r][cc][6] = r1.z;
                in[r][cc][7] = r1.w;
                in[r][cc][8] = r2.x;
            } else {
#pragma unroll
                for (int j = 0; j < 9; ++j) in[r][cc][j] = 0.0f;
            }
        }
        __syncthreads();
        for (int i = threadIdx.x; i < kHW * (kTH / 2); i += 256) {   // columns, two output rows each
            const int cc = i % kHW, pr = i / kHW;
            float a0[9], a1[9];
#pragma unroll
            for (int j = 0; j < 9; ++j) {
                a0[j] = 0.0f;
                a1[j] = 0.0f;
            }
#pragma unroll
            for (int k = 0; k <= 2 * kSsimR + 1; ++k) {
                const float* px = in[2 * pr + k][cc];
                if (k <= 2 * kSsimR) {
                    const float w = win.g[k];
#pragma unroll
                    for (int j = 0; j < 9; ++j) a0[j] = __builtin_fmaf(w, px[j], a0[j]);
                }
                if (k >= 1) {
                    const float w = win.g[k - 1];
#pragma unroll
                    for (int j = 0; j < 9; ++j) a1[j] = __builtin_fmaf(w, px[j], a1[j]);
                }
            }
#pragma unroll
            for (int j = 0; j < 9; ++j) {
                vs[2 * pr][j][cc] = a0[j];
                vs[2 * pr + 1][j][cc] = a1[j];
            }
        }
        __syncthreads();
        const int lx = threadIdx.x % kTW, ly = threadIdx.x / kTW;
        const int x = tx0 + lx, y = ty0 + ly;
        if (x >= W || y >= H) continue;   // (no barrier follows in this round)
        float sm[9];
#pragma unroll
        for (int j = 0; j < 9; ++j) sm[j] = 0.0f;
#pragma unroll
        for (int k = 0; k <= 2 * kSsimR; ++k) {
            const float w = win.g[k];
#pragma unroll
            for (int j = 0; j < 9; ++j) sm[j] = __builtin_fmaf(w, vs[ly][j][lx + k], sm[j]);
        }
        const int64_t p = static_cast<int64_t>(y) * W + x;
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            const float a = v.color[p * 3 + c], t = v.target[p * 3 + c];
            const float d = a - t;
            const float sgn = d > 0.0f ? 1.0f : (d < 0.0f ? -1.0f : 0.0f);
            const float dssim = sm[c] + 2.0f * (a - kShift) * sm[3 + c] + (t - kShift) * sm[6 + c];
            v.gc[p * 3 + c] = inv_n * (lam * sgn - (1.0f - lam) * dssim);
        }
    }
}

__global__ void __launch_bounds__(256) adam_kernel(float* __restrict__ p, const float* __restrict__ g,
                                                   float* __restrict__ m, float* __restrict__ v, int64_t nvec, int vec,
                                                   float lr, float b1, float omb1, float b2, float omb2, float eps,
                                                   float bc1, float bc2) {
    for (int64_t i = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x; i < nvec;
         i += static_cast<int64_t>(gridDim.x) * blockDim.x) {
        float g2 = 0.0f;
        for (int k = 0; k < vec; ++k) {
            const float gk = g[i * vec + k];
            g2 += gk * gk;
        }
        const float vi = b2 * v[i] + omb2 * g2;
        v[i] = vi;
        const float den = sqrtf(vi / bc2) + eps;
        for (int k = 0; k < vec; ++k) {
            const int64_t j = i * vec + k;
            const float mj = b1 * m[j] + omb1 * g[j];
            m[j] = mj;
            p[j] -= lr * (mj / bc1) / den;
        }
    }
}

// Adam on 16-byte groups of four parameters (vec = 1, n a multiple of 4,
// every array 16-byte aligned): the same arithmetic per element, with
// 16-byte loads and stores.
__global__ void __launch_bounds__(256) adam4_kernel(float4* __restrict__ p, const float4* __restrict__ g,
                                                    float4* __restrict__ m, float4* __restrict__ v, int64_t n4,
                                                    float lr, float b1, float omb1, float b2, float omb2, float eps,
                                                    float bc1, float bc2) {
    for (int64_t i = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x; i < n4;
         i += static_cast<int64_t>(gridDim.x) * blockDim.x) {
        const float4 gi = nt_load(g + i);
        float4 mi = nt_load(m + i), vi = nt_load(v + i), pi = nt_load(p + i);
        float* pm = &mi.x;
        float* pv = &vi.x;
        float* pp = &pi.x;
        const float* pg = &gi.x;
        for (int k = 0; k < 4; ++k) {
            pv[k] = b2 * pv[k] + omb2 * (pg[k] * pg[k]);
            pm[k] = b1 * pm[k] + omb1 * pg[k];
            pp[k] -= lr * (pm[k] / bc1) / (sqrtf(pv[k] / bc2) + eps);
        }
        nt_store(mi, m + i);
        nt_store(vi, v + i);
        nt_store(pi, p + i);
    }
}

}  // namespace

int ssim_tiles(int W, int H) { return ((W + kTW - 1) / kTW) * ((H + kTH - 1) / kTH); }

void launch_loss_l1_ssim(const SsimBatch& b, float lam, float inv_n, const SsimWindow& win, float* loss,
                         double* parts, hipStream_t s) {
    const int tiles = b.tile[b.n];
    if (tiles <= 0) return;
    const dim3 g(static_cast<unsigned>(tiles < kSumParts ? tiles : kSumParts));
    hipLaunchKernelGGL(ssim_stats_kernel, g, dim3(kTW * kTH), 0, s, b, lam, inv_n, win,
                       loss ? parts : nullptr);
    if (loss)
        hipLaunchKernelGGL(loss_sum_kernel, dim3(1), dim3(256), 0, s, parts, static_cast<int>(g.x), b.add, b.last, loss);
    hipLaunchKernelGGL(ssim_grad_kernel, g, dim3(kTW * kTH), 0, s, b, lam, inv_n, win);
}

void launch_adam(float* p, const float* g, float* m, float* v, int64_t nvec, int vec, float lr, float b1, float omb1,
                 float b2, float omb2, float eps, float bc1, float bc2, hipStream_t s) {
    if (nvec <= 0) return;
    const uintptr_t align = reinterpret_cast<uintptr_t>(p) | reinterpret_cast<uintptr_t>(g) |
                            reinterpret_cast<uintptr_t>(m) | reinterpret_cast<uintptr_t>(v);
    if (vec == 1 && nvec % 4 == 0 && (align & 15) == 0) {
        const int64_t n4 = nvec / 4;
        int64_t blocks = (n4 + 255) / 256;
        if (blocks > 16384) blocks = 16384;
        hipLaunchKernelGGL(adam4_kernel, dim3(static_cast<unsigned>(blocks)), dim3(256), 0, s,
                           reinterpret_cast<float4*>(p), reinterpret_cast<const float4*>(g),
                           reinterpret_cast<float4*>(m), reinterpret_cast<float4*>(v), n4, lr, b1, omb1, b2, omb2,
                           eps, bc1, bc2);
        return;
    }
    int64_t blocks = (nvec + 255) / 256;
    if (blocks > 16384) blocks = 16384;
    hipLaunchKernelGGL(adam_kernel, dim3(static_cast<unsigned>(blocks)), dim3(256), 0, s, p, g, m, v, nvec, vec, lr,
                       b1, omb1, b2, omb2, eps, bc1, bc2);
}

}  // namespace soup
