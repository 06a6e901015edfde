// Host-side declarations of the kernel launchers (internal to the library).
#pragma once

#include "common.hpp"

namespace soup {

void launch_fill_i32(int32_t* p, int64_t n, int32_t v, hipStream_t s);
// Ranges of 4-byte words that one launch clears.
struct ZeroList {
    int32_t* p[12];
    int64_t n[12];
    int k = 0;
    void add(void* q, int64_t words) {
        p[k] = static_cast<int32_t*>(q);
        n[k++] = words;
    }
};
void launch_zero(const ZeroList& z, hipStream_t s);
void launch_fill_f32(float* p, int64_t n, float v, hipStream_t s);
// Binning works on chunks of triangles per view. Large chunks (kBinChunk) of
// a view with at most kHistBins tiles are counted in an LDS histogram, and
// chunk_base ([chunks][tiles] int32) receives each chunk's first slot in every
// tile list it touches; when large chunks would leave the GPU idle (few views,
// few triangles) the chunks are small, their (tile, triangle) pairs spread over
// a workgroup and counted with global atomics.
constexpr int kBinChunk = 2048;
constexpr int kHistBins = 8192;
int bin_chunk_size(int V, int maxT, int num_cus);
inline int bin_chunks(int maxT, int chunk) { return maxT <= 0 ? 0 : (maxT + chunk - 1) / chunk; }
void launch_setup(const ViewDesc* views, int V, int maxT, int chunk, const SceneDesc* scenes, const Opts& o,
                  int tile, TriRec* recs, int32_t* tile_count, int32_t* chunk_base, int64_t n_tiles,
                  unsigned long long* visible, hipStream_t s);
// Distance of two tiles' counters in the count and fill arrays.
int bin_stride(int chunk, int64_t n_tiles);
// host_total: pinned memory that receives the sum of all values, or null.
void launch_scan(const int32_t* in, int64_t n, int stride, int64_t* bsum, int64_t* out, int64_t* host_total,
                 hipStream_t s);
void launch_scatter(const ViewDesc* views, int V, int maxT, int chunk, int tile, const TriRec* recs,
                    const int64_t* tile_start, int64_t n_tiles, const int32_t* chunk_base, int32_t* tile_fill,
                    uint64_t* entries, int64_t cap, hipStream_t s);
// entries holds cap entries: a scatter of more writes no further, and the sort of more does nothing.
void launch_sort(const int64_t* tile_start, int64_t n_tiles, uint64_t* entries, int64_t cap, hipStream_t s);
void launch_clip(int64_t* tile_start, int64_t n_tiles, int64_t cap, unsigned int* local, unsigned int* sticky,
                 hipStream_t s);

// Sticky overflow bits of the static-capacity mode.
constexpr unsigned kOverflowBins = 1u;
constexpr unsigned kOverflowFragments = 2u;

// MLP shapes compiled in: (C, H, NH); kPaper is the paper form's raster (opacity
// texture only, the shading MLP deferred), kReplay the walk with the winners known
enum class MlpKind { k8_16_1, k16_32_2, k32_64_2, kPaper, kReplay, kNone };
MlpKind mlp_kind(int n_layers, const int32_t* dims);
int mlp_params(int n_layers, const int32_t* dims);

// Work counters of the forward, each in a 256-byte line of its own.
constexpr uint32_t kWorkCounters = 8, kWorkStride = 64;

struct RasterArgs {
    const ViewDesc* views;
    int V;
    const SceneDesc* scenes;
    Opts o;
    int G;
    const TriRec* recs;
    const int64_t* tile_start;
    const uint64_t* entries;
    int64_t n_tiles;
    uint64_t* vis;                 // concatenated outputs (may be null when views carry their own)
    float* color;
    unsigned long long* counter;   // counters or null: [0] decodes, [8] pixels that some fragment covers
    unsigned int* work;            // persistent-kernel work counters (zeroed by the launcher's caller)
    uint32_t fixed;                // forward: regions below it are dealt by stride (a multiple of n_blocks)
    const float* weights;          // forward: every scene's weights as matrix operands (launch_begin), or null
    int n_blocks;                  // persistent grid of the forward (single-wave workgroups)
    int region;                    // side of a forward wave's region: 16 (tiles of 16, 32) or 8
    // optional log of the decoded fragments, one region per wave (= workgroup)
    uint4* log_frag;               // (pixel, triangle, depth bits, view)
    uint2* log_bary;               // (b1, b2)
    uint32_t log_region;
    uint32_t* log_counts;
    // the walk with the winners known (MlpKind::kReplay, else unused): the saved winners, and the
    // pixels' gradients, which decide whether a winner without a score weight is needed
    const uint64_t* replay_vis;
    const float* replay_color;     // [P,3] or null (every pixel is needed)
    const float* replay_logp;      // [P] score weights or null
    const float2* replay_edge;     // [P] edge weights or null
    int replay_all;                // 1: every pixel needs its whole front set (log p)
};

// The first launch of a binning: clears z and, for the MLP shapes decoded on the matrix cores, lays
// out the weights of each scene in their operand order (fwd_weights_bytes per scene; 0: none).
size_t fwd_weights_bytes(MlpKind k);
void launch_begin(const ZeroList& z, const SceneDesc* scenes, int n_scenes, MlpKind k, float* weights, hipStream_t s);
void launch_raster_fwd(const RasterArgs& a, int tile, MlpKind k, hipStream_t s);
// Resident single-wave workgroups per CU of the forward kernel for a tile side, MLP shape and
// region side (16: 16x16 pixels of a tile of 16 or 32; 8: one 8x8 block).
int raster_fwd_blocks_per_cu(int tile, MlpKind k, int region);
// The forward's unit of work: a region of `region` x `region` pixels of a tile.
inline int fwd_regions_per_tile(int tile, int region) { return (tile / region) * (tile / region); }

// One fragment the backward needs (24 bytes): p0 = (pixel, triangle | winner
// << 31), p1 = the perspective-correct barycentrics (b1, b2) as bits, x =
// (the pixel's score weight as bits, view). A winner's colour gradient and
// edge weights are read from the per-pixel arrays by the decode.
struct FragRec {
    uint2 p0;
    uint2 p1;
    uint2 x;
};

// A log of fragments, one region of `region` entries per wave of the raster
// that wrote it (so that no two waves share a counter). counts[w] is the number
// of fragments wave w found (it may exceed `region`: the log is then not used,
// or, in static-capacity mode, cut there and flagged).
constexpr int kMaxRegions = 4096;
struct FragLogView {
    const uint4* frag;             // (pixel, triangle, depth bits, view)
    const uint2* bary;             // (b1, b2)
    const uint32_t* counts;        // [n_regions]
    uint32_t region;
    int n_regions;
    int split;                     // waves that share a region's batches of 64
};
// 64-entry batches of one region.
__host__ __device__ constexpr uint32_t log_slots(uint32_t region) { return (region + 63) / 64; }
// Workgroups of four waves for the kernels that read a log: one wave per share of a
// region, at most 2,048 workgroups, eight for each of the MI355X's 256 CUs (four views of
// 50,000 triangles: placing 39 us with four per CU, 32 with eight; 64 views the same).
inline unsigned log_blocks(const FragLogView& L) {
    const int64_t waves = static_cast<int64_t>(L.n_regions) * L.split;
    return static_cast<unsigned>(waves < 4 ? 1 : waves > 8192 ? 2048 : (waves + 3) / 4);
}

// Which fragments of a log are kept: the pixel's winner, and every fragment in
// front of it where the pixel carries a score weight (or everywhere).
struct FragSelect {
    const uint64_t* vis;
    const float* grad_logp;        // [P] or null
    int all_front;                 // log p: every fragment in front
    __device__ __forceinline__ void decide(const uint4& e, bool& keep, bool& win) const {
        const uint64_t key = (static_cast<uint64_t>(e.z) << 32) | e.y;
        const uint64_t kstar = vis[e.x];
        win = key == kstar;
        keep = win || (key < kstar && (all_front || (grad_logp && grad_logp[e.x] != 0.0f)));
    }
};

#if defined(__HIPCC__)
// f(region, first entry, entries of the region) for every batch of this wave
// (workgroups of four waves; wave-uniform arguments).
template <class F>
__device__ __forceinline__ void for_log_batches(const FragLogView& L, F&& f) {
    const uint32_t n_items = static_cast<uint32_t>(L.n_regions) * static_cast<uint32_t>(L.split);
    const uint32_t w = static_cast<uint32_t>(__builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x >> 6)));
    for (uint32_t it = blockIdx.x * 4 + w; it < n_items; it += gridDim.x * 4) {
        const uint32_t r = it / static_cast<uint32_t>(L.split), q = it % static_cast<uint32_t>(L.split);
        const uint32_t c = L.counts[r], n = c < L.region ? c : L.region;
        for (uint32_t b = 64 * q; b < n; b += 64 * static_cast<uint32_t>(L.split)) f(r, b, n);
    }
}
// Lanes 0..l, and the lanes of the run that starts at head lane l (heads: the first lanes of all runs).
__device__ __forceinline__ uint64_t upto_mask(int l) { return ~0ull >> (63 - l); }
__device__ __forceinline__ uint64_t run_of(uint64_t heads, int l) {
    const uint64_t above = heads & ~upto_mask(l);
    return (above ? (1ull << __builtin_ctzll(above)) - 1 : ~0ull) & (~0ull << l);
}
#endif

// Total and largest count of a log's regions; an overflow sets kOverflowFragments in *sticky (when not null).
// summary: pinned memory that receives (total, largest), or null.
void launch_log_summary(const uint32_t* counts, int n, uint32_t region, unsigned long long* summary,
                        unsigned int* sticky, hipStream_t s);
// What is kept of a log, per 64 entries the masks (kept, winners), log_slots(region) per region,
// and the kept fragments per triangle (added to tri_count [T]).
void launch_count(const FragLogView& L, const FragSelect& sel, ulonglong2* masks, int32_t* tri_count, hipStream_t s);
// Counting-sort placement by triangle: within triangle t's range [tri_off[t], tri_off[t + 1])
// (the scanned counts) its winners come first (filled upwards) and the fragments in front of
// winners last (filled downwards). tri_fill [T] zeroed: winners placed (low 32 bits), others (high).
void launch_place(const FragLogView& L, const float* grad_logp, const ulonglong2* masks, const int64_t* tri_off,
                  unsigned long long* tri_fill, FragRec* sorted, hipStream_t s);

struct LogpArgs {
    FragLogView log;
    FragSelect sel;
    const float* feats;
    const float* mlp;
    const float* weights;          // the scene's weights as the forward's matrix operands
    int G;
    float* logp;                   // [P], zeroed by the caller
};
void launch_logp(const LogpArgs& a, MlpKind k, hipStream_t s);

struct DecodeArgs {
    const ViewDesc* views;
    int V;
    const TriRec* recs;
    const float* feats;
    const float* mlp;
    int G;
    int T;
    // the list sorted by triangle
    const FragRec* sorted;         // [tri_off[T]]
    const int64_t* tri_off;        // [T + 1]
    const float* verts;            // [T, 3, 3]: the winners' clip coordinates are recomputed
    const float* grad_color;       // [P, 3]: the winners' colour gradients
    const float2* edge_w;          // [P] the winners' edge weights, or null (none)
    float* grad_feats;             // [T, G, G, C]: zeroed by the caller unless accumulate
    float* grad_verts;             // [T, 9]: zeroed by the caller unless accumulate
    int accumulate;
    float* mlp_partial;            // [n_blocks * 4, n_params]
    int short_list;                  // 1: fewer than eight batches of 64 fragments per wave (known on the host)
    unsigned long long* counter;   // decode counter or null
    int n_blocks;
};

void launch_decode_bwd(const DecodeArgs& a, MlpKind k, hipStream_t s);
// LDS bytes one workgroup of the decode needs for a grid side G (0: unknown).
size_t decode_bwd_lds(MlpKind k, int G);
// ew[p] = (x, y) edge weights of the pairs pixel p occludes (Section 3.2),
// written for covered pixels only (a background pixel occludes nothing)
void launch_edge_weights(const ViewDesc* views, int V, int64_t P, const Opts& o, const uint64_t* vis,
                         const float* color, const float* grad_color, float2* ew, hipStream_t s);
void launch_mlp_reduce(const float* partial, int n_rows, int n_params, float* out, bool accumulate, hipStream_t s);
void launch_loss_l2(const float* color, const float* target, int64_t P, float* gc, float* gl, float* loss,
                    hipStream_t s);
void launch_selftest_sigmoid(const float* x, float* y, int64_t n, hipStream_t s);
void launch_selftest_uniform(uint64_t seed, const uint32_t* pixel, const uint32_t* tri, uint32_t view_id,
                             uint32_t step, float* u, int64_t n, hipStream_t s);


// Paper form (Section 3.3; Supplement B.3, B.6): mesh-colour texture assembly,
// deferred shading, the score term and log p over a fragment list, the
// winners' backward.
constexpr int kPMaxLevels = 8;
struct AssembleArgs {
    const float* raw[kPMaxLevels];   // learnable level Rmin + l: [T][V(level)][8]
    float* graw[kPMaxLevels];        // backward: their gradients
    int Rmin, Rtop, Rmax, T;
    float* tex_out;                  // forward: [T][V(Rmax)][8]
    const float* tex;                // backward: the assembled texture and its gradient
    const float* grad_tex;
    int accumulate;
};
void launch_mc_assemble(const AssembleArgs& a, hipStream_t s);
size_t mc_assemble_bwd_lds(int Rmin, int Rmax);
size_t mc_assemble_bwd_lds_cap(size_t lds_limit);
void launch_mc_assemble_bwd(const AssembleArgs& a, size_t lds_limit, hipStream_t s);

struct PShadeArgs {
    const ViewDesc* views;
    int V;
    int64_t P;
    const TriRec* recs;
    const float* tex;
    const float* mlp;
    int R;
    const uint64_t* vis;
    float* color;
    Opts o;
};
void launch_pshade(const PShadeArgs& a, hipStream_t s);

struct PFragArgs {
    FragLogView log;
    FragSelect sel;
    const float* tex;
    int R;
    float* grad_tex;                 // score pass: d / d opacity channel (added to)
    float* logp;                     // logp pass (zeroed by the caller)
};
void launch_pfrag(const PFragArgs& a, bool logp, hipStream_t s);

struct PWinArgs {
    const ViewDesc* views;
    int V;
    int64_t P;
    const TriRec* recs;
    const float* verts;
    const float* tex;
    const float* mlp;
    int R;
    const uint64_t* vis;
    const float* grad_color;
    const float2* edge_w;            // or null
    float* grad_tex;                 // added to
    double* gvert;                   // [T, 9] float64 sums (zeroed by the caller)
    float* mlp_partial;              // [n_blocks * 4, 595]
    int n_blocks;
};
struct PTriArgs {
    const ViewDesc* views;
    const TriRec* recs;
    const float* verts;
    const float* tex;
    const float* mlp;
    int R;
    int T;
    const FragRec* sorted;           // [tri_off[T]] the fragment list sorted by triangle
    const int64_t* tri_off;          // [T + 1]
    const float* grad_color;
    const float2* edge_w;            // or null
    int score;                       // 1: the score term (mode 0 with score weights)
    int accumulate;                  // 1: add into grad_tex rows (else they were zero-filled)
    float* grad_tex;
    double* gvert;                   // [T, 9] float64 sums (zeroed by the caller)
    float* mlp_partial;              // [n_blocks, 595]
    int n_blocks;                    // single-wave workgroups, a multiple of 8
    // levels = 1: the learnable levels' gradients instead of grad_tex (tex is
    // their assembly onto level R); graw[l] = level Rmin + l, zero-filled by
    // the caller unless accumulating
    int levels;
    int Rmin, Rtop;
    float* graw[kPMaxLevels];
};
bool ptri_sorted(int R);

// measured ceilings (probe.hip)
void launch_probe_copy(const float4* src, float4* dst, int64_t n, int num_cus, hipStream_t s);
void launch_probe_read(const float4* src, int64_t n, float* partial, int64_t n_partial, hipStream_t s);
void launch_probe_atomic(float* slots, int64_t n_slots, int64_t n_ops, int num_cus, hipStream_t s);
void launch_probe_fma(float* out, int64_t n_threads, int iters, hipStream_t s);
void launch_probe_mfma(float* out, int64_t n_threads, int iters, hipStream_t s);
int ptri_blocks(int num_cus, bool levels, int R, int Rmin, int Rtop);
void launch_ptri_bwd(const PTriArgs& a, hipStream_t s);
int pwinner_blocks(int num_cus);
void launch_pwinner_bwd(const PWinArgs& a, hipStream_t s);
void launch_pvert_finish(const double* g, float* out, int64_t n, bool accumulate, hipStream_t s);

// Adaptive control of primitives.
constexpr int kEdgeViews = 32;  // views per edge-length launch (kernel argument)
struct EdgeViews {
    float m[kEdgeViews][16];    // row-major view-projection matrices
    float w[kEdgeViews], h[kEdgeViews];
    int n;
};
constexpr int kActRemove = 0, kActKeep = 1, kActSplit0 = 2;
void launch_coverage(const uint64_t* vis, int64_t n, int32_t T, uint32_t* counts, int num_cus, hipStream_t s);
void launch_edge_lengths(const float* verts, int32_t T, const EdgeViews& ev, float near_w, bool first, float* rel,
                         hipStream_t s);
void launch_apply(const float* verts, const float* feats, const int32_t* actions, const int32_t* offsets, int32_t T,
                  int32_t G, int32_t C, int32_t n_new, float* vout, float* fout, hipStream_t s);
int32_t plan_host(const uint32_t* counts, const float* rel, int32_t T, float split_frac, int32_t target,
                  bool prune_zero, bool fill, int32_t* actions, int32_t* offsets);

// Training step: L1 + SSIM loss, Adam / VectorAdam.
constexpr int kSsimR = 5;  // 11 x 11 window
struct SsimWindow {
    float g[2 * kSsimR + 1];   // normalised 1-D Gaussian, sigma 1.5; the window is its outer product
};
// Views whose loss one pair of launches evaluates (consecutive views of a call).
constexpr int kSsimViews = 32;
struct SsimBatch {
    const float* color;
    const float* target;
    float* grad_color;
    float* grad_logp;
    float* stats;                    // 12 floats per pixel of the batch
    int64_t pix[kSsimViews];         // first pixel of each view in the caller's arrays
    int w[kSsimViews], h[kSsimViews];
    int tile[kSsimViews + 1];        // first tile of each view, and their number
    int n;
    int add;                         // 1: the loss of earlier batches is added to
    int last;                        // 1: no batch follows, the loss goes out
};
int ssim_tiles(int W, int H);
// parts: kSumParts sums and the running total
void launch_loss_l1_ssim(const SsimBatch& b, float lam, float inv_n, const SsimWindow& win, float* loss,
                         double* parts, hipStream_t s);
void launch_adam(float* p, const float* g, float* m, float* v, int64_t nvec, int vec, float lr, float b1, float omb1,
                 float b2, float omb2, float eps, float bc1, float bc2, hipStream_t s);

}  // namespace soup
