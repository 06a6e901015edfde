// C ABI of the gfx950 soup rasterizer: context, argument validation,
// workspace management and the launch sequence of each entry point.
#include <algorithm>
#include <cmath>
#include <cstdarg>
#include <cstdio>
#include <cstring>
#include <mutex>
#include <new>
#include <string>
#include <vector>

#include "../../include/diffsoup.h"
#include "internal.hpp"
#include "pform.hpp"

namespace {

using namespace soup;

struct DevBuf {
    void* p = nullptr;
    size_t bytes = 0;
};

}  // namespace

struct soup_ctx {
    int device = 0;
    int num_cus = 256;
    size_t lds_limit = 163840;   // LDS bytes one workgroup may use (the CU's whole LDS on this GPU)
    int tile = 16;
    bool counting = false;
    bool fixed = false;              // static-capacity mode: no synchronisation, no allocation
    bool flags_ready = false;        // sticky overflow flags cleared after allocation
    // a fragment log: its buffers, region size and count, and the largest count of the
    // last call (0: none yet), which sizes the next
    struct FragLog {
        DevBuf frag, bary, counts;
        uint64_t region = 0, hint = 0;
        uint64_t total = 0;          // fragments of the last eager call
        int regions = 0;
        bool pending = false;        // the counts of the last eager raster have not been read yet
        bool fits = false;           // ... and whether they fitted the regions
    };
    FragLog flog, rlog;              // the forward's, and that of the walk with the winners known
    DevBuf masks;                    // what is kept of a log
    // pinned: the tile lists' length, then (total, largest) of either log, written by kernels
    // and read after the event behind them
    int64_t* host_res = nullptr;
    hipEvent_t ev_total = nullptr, ev_log = nullptr;
    bool staging_busy = false;       // an upload from host_stage may be in flight
    // the draws the forward's log was made with (valid only with bins_valid)
    bool log_valid = false;
    uint64_t log_seed = 0;
    uint32_t log_step = 0;
    int log_mode = 0;
    // the setup records and tile lists in place: built for desc_cache, this tile size and near_w
    bool bins_valid = false;
    int bins_tile = 0;
    float bins_near_w = 0.0f;
    std::vector<char> desc_cache;    // descriptors of the last upload (static mode reuses them)
    std::string err;
    soup_stats stats{};
    DevBuf views;        // view descriptors, then scene descriptors
    DevBuf recs, tile_count, tile_fill, tile_start, bsum, entries, edge_w, partial, counters;
    DevBuf fwd_weights;  // every scene's MLP weights as the forward's matrix operands
    DevBuf chunk_base;   // [binning chunks][tiles] first slot of a chunk in each tile list
    DevBuf tri_count, tri_fill, tri_off, tri_bsum, sorted, flags;
    DevBuf ssim;                                      // the training loss's parts and running total, then its SSIM statistics
    DevBuf gvert;                                     // the paper form's float64 vertex gradient sums
    DevBuf gtex;                                      // its texture gradient when levels are asked for and the sorted path cannot fold them in
    void* host_stage = nullptr;      // pinned: descriptors up, totals down
    float* scratch = nullptr;        // this device's address of the allocation-free loss's static scratch
    size_t host_stage_bytes = 0;
    // optional per-kernel timing: recorded event pairs and a pool of free events
    bool timing = false;
    struct Mark {
        int kind;
        hipEvent_t a, b;
    };
    std::vector<Mark> marks;
    std::vector<hipEvent_t> pool;
};

namespace {

soup_status fail(soup_ctx* c, soup_status s, const char* fmt, ...) {
    char buf[512];
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(buf, sizeof(buf), fmt, ap);
    va_end(ap);
    if (c) c->err = buf;
    return s;
}

#define HIP_TRY(ctx, expr)                                                                              \
    do {                                                                                                \
        hipError_t e_ = (expr);                                                                         \
        if (e_ != hipSuccess) return fail(ctx, SOUP_ERR_HIP, "%s failed: %s", #expr, hipGetErrorString(e_)); \
    } while (0)

soup_status ensure(soup_ctx* c, DevBuf& b, size_t bytes) {
    if (bytes == 0) bytes = 256;
    if (b.bytes >= bytes) return SOUP_OK;
    if (c->fixed)
        return fail(c, SOUP_ERR_CAPACITY, "static mode: a workspace of %zu bytes is needed (have %zu); run the "
                    "call once outside static mode to size it", bytes, b.bytes);
    if (b.p) {
        hipError_t e = hipFree(b.p);
        b.p = nullptr;
        b.bytes = 0;
        if (e != hipSuccess) return fail(c, SOUP_ERR_HIP, "hipFree failed: %s", hipGetErrorString(e));
    }
    size_t want = bytes + bytes / 4;
    hipError_t e = hipMalloc(&b.p, want);
    if (e != hipSuccess) {
        (void)hipGetLastError();
        b.p = nullptr;
        return fail(c, SOUP_ERR_OOM, "device allocation of %zu bytes failed", want);
    }
    b.bytes = want;
    return SOUP_OK;
}

soup_status ensure_host(soup_ctx* c, size_t bytes) {
    if (c->host_stage_bytes >= bytes) return SOUP_OK;
    if (c->host_stage) (void)hipHostFree(c->host_stage);
    c->host_stage = nullptr;
    c->host_stage_bytes = 0;
    size_t want = std::max<size_t>(bytes + bytes / 4, 4096);
    if (hipHostMalloc(&c->host_stage, want, hipHostMallocDefault) != hipSuccess) {
        (void)hipGetLastError();
        return fail(c, SOUP_ERR_OOM, "pinned host allocation of %zu bytes failed", want);
    }
    c->host_stage_bytes = want;
    return SOUP_OK;
}

}  // namespace

namespace {

hipEvent_t take_event(soup_ctx* c) {
    if (!c->pool.empty()) {
        hipEvent_t e = c->pool.back();
        c->pool.pop_back();
        return e;
    }
    hipEvent_t e = nullptr;
    if (hipEventCreate(&e) != hipSuccess) {
        (void)hipGetLastError();
        return nullptr;
    }
    return e;
}

// Brackets the launches made during its lifetime with two events (timing on).
struct Timed {
    soup_ctx* c;
    int kind;
    hipStream_t s;
    hipEvent_t a = nullptr;
    Timed(soup_ctx* c_, int k, hipStream_t s_) : c(c_), kind(k), s(s_) {
        if (c->timing && !c->fixed && (a = take_event(c))) (void)hipEventRecord(a, s);
    }
    ~Timed() {
        if (!a) return;
        hipEvent_t b = take_event(c);
        if (!b) {
            c->pool.push_back(a);
            return;
        }
        (void)hipEventRecord(b, s);
        c->marks.push_back({kind, a, b});
    }
};

}  // namespace

namespace soup {

MlpKind mlp_kind(int n_layers, const int32_t* dims) {
    if (n_layers == 2 && dims[0] == 8 && dims[1] == 16 && dims[2] == 4) return MlpKind::k8_16_1;
    if (n_layers == 3 && dims[0] == 16 && dims[1] == 32 && dims[2] == 32 && dims[3] == 4) return MlpKind::k16_32_2;
    if (n_layers == 3 && dims[0] == 32 && dims[1] == 64 && dims[2] == 64 && dims[3] == 4) return MlpKind::k32_64_2;
    return MlpKind::kNone;
}

int mlp_params(int n_layers, const int32_t* dims) {
    int n = 0;
    for (int l = 0; l < n_layers; ++l) n += dims[l + 1] * dims[l] + dims[l + 1];
    return n;
}

}  // namespace soup

namespace {

soup_status check_scene(soup_ctx* c, const soup_scene* s, MlpKind* kind) {
    if (!s) return fail(c, SOUP_ERR_INVALID, "scene is NULL");
    if (s->T < 0) return fail(c, SOUP_ERR_INVALID, "scene.T = %d < 0", s->T);
    if (s->G < 2 || s->G > 256) return fail(c, SOUP_ERR_INVALID, "scene.G = %d outside [2, 256]", s->G);
    if (s->n_layers < 1 || s->n_layers > 16 || !s->dims)
        return fail(c, SOUP_ERR_INVALID, "scene.n_layers = %d or dims missing", s->n_layers);
    if (s->dims[0] != s->C) return fail(c, SOUP_ERR_INVALID, "dims[0] = %d != C = %d", s->dims[0], s->C);
    if (s->dims[s->n_layers] != 4) return fail(c, SOUP_ERR_INVALID, "dims[last] = %d != 4", s->dims[s->n_layers]);
    if (static_cast<int64_t>(s->G) * s->G * s->C > 4096)
        return fail(c, SOUP_ERR_UNSUPPORTED, "G*G*C = %d exceeds the per-wave LDS gradient grid (4096 floats)",
                    s->G * s->G * s->C);
    if (s->T > 0 && (!s->verts || !s->feats || !s->mlp))
        return fail(c, SOUP_ERR_INVALID, "scene device pointers are NULL");
    *kind = soup::mlp_kind(s->n_layers, s->dims);
    if (*kind == MlpKind::kNone) {
        std::string d;
        for (int i = 0; i <= s->n_layers; ++i) d += (i ? "->" : "") + std::to_string(s->dims[i]);
        return fail(c, SOUP_ERR_UNSUPPORTED, "MLP shape %s is not compiled in (8->16->4, 16->32->32->4, 32->64->64->4)",
                    d.c_str());
    }
    return SOUP_OK;
}

// The backward decode keeps one triangle's gradient grid per wave in LDS: refuse a
// grid that would not fit one workgroup's LDS rather than launch it.
soup_status check_decode_lds(soup_ctx* c, MlpKind kind, int G) {
    const size_t need = decode_bwd_lds(kind, G);
    if (need > c->lds_limit)
        return fail(c, SOUP_ERR_UNSUPPORTED, "the backward decode needs %zu bytes of LDS per workgroup for G = %d "
                    "(the device has %zu): use a smaller texture grid", need, G, c->lds_limit);
    return SOUP_OK;
}

soup_status check_views(soup_ctx* c, const soup_views* v) {
    if (!v) return fail(c, SOUP_ERR_INVALID, "views is NULL");
    if (v->V < 1 || v->V > soup::kMaxViews) return fail(c, SOUP_ERR_INVALID, "views.V = %d outside [1, 65536]", v->V);
    if (!v->width || !v->height || !v->view_id || !v->view_proj)
        return fail(c, SOUP_ERR_INVALID, "views host arrays are NULL");
    for (int i = 0; i < v->V; ++i)
        if (v->width[i] < 1 || v->width[i] > 16384 || v->height[i] < 1 || v->height[i] > 16384)
            return fail(c, SOUP_ERR_INVALID, "view %d size %dx%d outside [1, 16384]", i, v->width[i], v->height[i]);
    return SOUP_OK;
}

soup_status check_opts(soup_ctx* c, const soup_opts* o) {
    if (!o) return fail(c, SOUP_ERR_INVALID, "opts is NULL");
    if (o->mode != 0 && o->mode != 1) return fail(c, SOUP_ERR_INVALID, "opts.mode = %d (0 or 1)", o->mode);
    if (o->accumulate != 0 && o->accumulate != 1)
        return fail(c, SOUP_ERR_INVALID, "opts.accumulate = %d (0 or 1)", o->accumulate);
    if (o->edge_pairs < 0 || o->edge_pairs > 2)
        return fail(c, SOUP_ERR_INVALID, "opts.edge_pairs = %d (0, 1 or 2)", o->edge_pairs);
    if (o->reuse_bins != 0 && o->reuse_bins != 1)
        return fail(c, SOUP_ERR_INVALID, "opts.reuse_bins = %d (0 or 1)", o->reuse_bins);
    if (!(o->near_w > 0.0f)) return fail(c, SOUP_ERR_INVALID, "opts.near_w must be > 0");
    return SOUP_OK;
}

// A fragment log holds a pixel's index in 32 bits.
constexpr int64_t kMaxLogPixels = int64_t(1) << 32;

soup_status check_log_pixels(soup_ctx* c, const char* what, int64_t n_pix) {
    if (n_pix >= kMaxLogPixels) return fail(c, SOUP_ERR_CAPACITY, "%s needs fewer than 2^32 pixels per call", what);
    return SOUP_OK;
}

// An eager call reads on the host what its kernels found, which a stream that captures does not run:
// refused before anything is enqueued or kept.
soup_status check_capture(soup_ctx* c, hipStream_t s) {
    if (c->fixed || !s) return SOUP_OK;   // (the null stream cannot capture)
    hipStreamCaptureStatus capture = hipStreamCaptureStatusNone;
    HIP_TRY(c, hipStreamIsCapturing(s, &capture));
    if (capture == hipStreamCaptureStatusNone) return SOUP_OK;
    return fail(c, SOUP_ERR_HIP, "the stream is capturing: only static-mode calls can be captured");
}

Opts to_opts(const soup_opts* o) {
    Opts r{};
    r.seed = o->seed;
    r.step = o->step;
    r.mode = o->mode;
    r.bg[0] = o->background[0];
    r.bg[1] = o->background[1];
    r.bg[2] = o->background[2];
    r.edge_pairs = o->edge_pairs;
    r.near_w = o->near_w;
    r.accumulate = o->accumulate;
    r.reuse_bins = o->reuse_bins;
    return r;
}

// The counters buffer: 128 bytes of counts, totals and flags, then the work counters.
constexpr size_t kCountersBytes = 128;

// Per-call plan: descriptors and sizes.
struct Plan {
    std::vector<ViewDesc> views;
    std::vector<SceneDesc> scenes;
    int64_t n_tiles = 0, n_pix = 0, n_recs = 0;
    int maxT = 0;
    int G = 0;
    MlpKind kind = MlpKind::kNone;
    int n_params = 0;
};

void plan_views(Plan& p, const soup_views* v, int tile, const std::vector<int>& scene_of_view,
                const std::vector<int64_t>& rec_base) {
    p.views.resize(v->V);
    int64_t tb = 0, pb = 0;
    for (int i = 0; i < v->V; ++i) {
        ViewDesc& d = p.views[i];
        memset(&d, 0, sizeof(d));
        memcpy(d.M, v->view_proj + 16 * i, sizeof(d.M));
        d.W = v->width[i];
        d.H = v->height[i];
        d.view_id = v->view_id[i];
        d.scene = scene_of_view[i];
        d.tiles_x = (d.W + tile - 1) / tile;
        d.tiles_y = (d.H + tile - 1) / tile;
        d.T = p.scenes[d.scene].T;
        d.tile_base = tb;
        d.pix_base = pb;
        d.rec_base = rec_base[i];
        tb += static_cast<int64_t>(d.tiles_x) * d.tiles_y;
        pb += static_cast<int64_t>(d.W) * d.H;
        p.maxT = std::max(p.maxT, d.T);
    }
    p.n_tiles = tb;
    p.n_pix = pb;
}

bool same_descriptors(const soup_ctx* c, const Plan& p) {
    const size_t vbytes = p.views.size() * sizeof(ViewDesc), sbytes = p.scenes.size() * sizeof(SceneDesc);
    return c->desc_cache.size() == vbytes + sbytes && memcmp(c->desc_cache.data(), p.views.data(), vbytes) == 0 &&
           memcmp(c->desc_cache.data() + vbytes, p.scenes.data(), sbytes) == 0;
}

// Upload descriptors, run setup + scan, scatter + sort. An eager call scatters and sorts into the
// entries buffer in place while the host waits for the lists' length (an event behind the scan); lists
// that need a larger buffer are made again. forward: the raster's work counters and weight operands are
// made ready by the first launch.
soup_status bin(soup_ctx* c, Plan& p, const Opts& o, bool forward, hipStream_t s) {
    const size_t vbytes = p.views.size() * sizeof(ViewDesc), sbytes = p.scenes.size() * sizeof(SceneDesc);
    const int chunk = bin_chunk_size(static_cast<int>(p.views.size()), p.maxT, c->num_cus);
    const int stride = bin_stride(chunk, p.n_tiles);
    soup_status st;
    if ((st = check_capture(c, s))) return st;
    // the forward counts its regions in 32 bits, a wave adds its grid to an index, and every wave fetches
    // one index past the last
    if (p.n_tiles * fwd_regions_per_tile(c->tile, 8) >=
        (int64_t(1) << 32) - kMaxRegions - 2 * static_cast<int64_t>(kWorkCounters))
        return fail(c, SOUP_ERR_CAPACITY, "too many pixels in one call (2^32 forward regions)");
    if ((st = ensure(c, c->views, vbytes + sbytes)) ||
        (st = ensure(c, c->recs, static_cast<size_t>(p.n_recs) * sizeof(TriRec))) ||
        (st = ensure(c, c->tile_count, static_cast<size_t>(p.n_tiles) * stride * 4)) ||
        (st = ensure(c, c->tile_fill, static_cast<size_t>(p.n_tiles) * stride * 4)) ||
        // per-chunk tile slots exist only for the LDS-histogram chunks (small chunks count with
        // global atomics and need none)
        (st = ensure(c, c->chunk_base,
                     chunk >= kBinChunk ? static_cast<size_t>(bin_chunks(p.maxT, chunk)) * p.n_tiles * 4 : 0)) ||
        (st = ensure(c, c->tile_start, static_cast<size_t>(p.n_tiles + 1) * 8)) ||
        (st = ensure(c, c->bsum, static_cast<size_t>((p.n_tiles + 1023) / 1024 + 1) * 8)) ||
        (st = ensure(c, c->counters, kCountersBytes + kWorkCounters * kWorkStride * 4)) ||
        (st = ensure(c, c->flags, 256)) || (st = ensure_host(c, vbytes + sbytes)) ||
        // (a backward's binning sizes it too: a static-mode forward may follow)
        (st = ensure(c, c->fwd_weights, fwd_weights_bytes(p.kind) * p.scenes.size())))
        return st;
    if (!c->flags_ready) {   // first allocation (never in static mode): clear the sticky flags
        launch_fill_i32(static_cast<int32_t*>(c->flags.p), 64, 0, s);
        c->flags_ready = true;
    }
    const bool same = same_descriptors(c, p);
    c->bins_valid = false;
    c->log_valid = false;
    ViewDesc* const views = static_cast<ViewDesc*>(c->views.p);
    SceneDesc* const scenes = reinterpret_cast<SceneDesc*>(static_cast<char*>(c->views.p) + vbytes);
    if (c->fixed) {
        // a captured call must not depend on host memory at replay time
        if (!same) return fail(c, SOUP_ERR_INVALID, "static mode needs the views and scenes of the previous call");
    } else {
        // every call that uploads waits below for an event behind the upload, so that the staging
        // buffer is free, unless that call failed in between
        if (c->staging_busy) HIP_TRY(c, hipDeviceSynchronize());
        char* hs = static_cast<char*>(c->host_stage);
        memcpy(hs, p.views.data(), vbytes);
        memcpy(hs + vbytes, p.scenes.data(), sbytes);
        c->desc_cache.assign(hs, hs + vbytes + sbytes);
        c->staging_busy = true;
        HIP_TRY(c, hipMemcpyAsync(c->views.p, hs, vbytes + sbytes, hipMemcpyHostToDevice, s));
    }
    unsigned long long* cnt = static_cast<unsigned long long*>(c->counters.p);
    int32_t* const count = static_cast<int32_t*>(c->tile_count.p);
    int32_t* const fill = static_cast<int32_t*>(c->tile_fill.p);
    int64_t* const start = static_cast<int64_t*>(c->tile_start.p);
    {
        Timed t(c, SOUP_T_FILL, s);
        ZeroList z;
        z.add(cnt, (kCountersBytes + kWorkCounters * kWorkStride * 4) / 4);
        z.add(count, p.n_tiles * stride);
        z.add(fill, p.n_tiles * stride);
        launch_begin(z, scenes, static_cast<int>(p.scenes.size()), forward ? p.kind : MlpKind::kNone,
                     static_cast<float*>(c->fwd_weights.p), s);
    }
    {
        Timed t_setup(c, SOUP_T_SETUP, s);
        launch_setup(views, static_cast<int>(p.views.size()), p.maxT, chunk, scenes, o, c->tile,
                     static_cast<TriRec*>(c->recs.p), count, static_cast<int32_t*>(c->chunk_base.p), p.n_tiles,
                     c->counting ? cnt + 1 : nullptr, s);
    }
    {
        Timed t(c, SOUP_T_SCAN, s);
        launch_scan(count, p.n_tiles, stride, static_cast<int64_t*>(c->bsum.p), start, c->fixed ? nullptr : c->host_res, s);
    }
    auto lists = [&]() {
        const int64_t cap = static_cast<int64_t>(c->entries.bytes / 8);
        uint64_t* const entries = static_cast<uint64_t*>(c->entries.p);
        {
            Timed t(c, SOUP_T_SCATTER, s);
            launch_scatter(views, static_cast<int>(p.views.size()), p.maxT, chunk, c->tile,
                           static_cast<TriRec*>(c->recs.p), start, p.n_tiles, static_cast<int32_t*>(c->chunk_base.p),
                           fill, entries, cap, s);
        }
        Timed t(c, SOUP_T_SORT, s);
        launch_sort(start, p.n_tiles, entries, cap, s);
    };
    int64_t total = -1;
    if (c->fixed) {
        // the capacity in place bounds the lists; an overflow empties them and is flagged
        launch_clip(start, p.n_tiles, static_cast<int64_t>(c->entries.bytes / 8),
                    reinterpret_cast<unsigned int*>(cnt + 7), static_cast<unsigned int*>(c->flags.p), s);
        lists();
    } else {
        HIP_TRY(c, hipEventRecord(c->ev_total, s));
        const bool ahead = c->entries.p != nullptr;
        if (ahead) lists();
        HIP_TRY(c, hipGetLastError());
        HIP_TRY(c, hipEventSynchronize(c->ev_total));
        c->staging_busy = false;
        total = *static_cast<volatile int64_t*>(c->host_res);
        if (!ahead || total > static_cast<int64_t>(c->entries.bytes / 8)) {
            if ((st = ensure(c, c->entries, static_cast<size_t>(total) * 8))) return st;
            if (ahead) launch_fill_i32(fill, p.n_tiles * stride, 0, s);
            lists();
        }
    }
    HIP_TRY(c, hipGetLastError());
    c->stats.pixels = p.n_pix;
    c->stats.tiles = p.n_tiles;
    c->stats.bin_entries = total;
    c->bins_valid = true;
    c->bins_tile = c->tile;
    c->bins_near_w = o.near_w;
    return SOUP_OK;
}

RasterArgs raster_args(soup_ctx* c, const Plan& p, const Opts& o, MlpKind kind) {
    RasterArgs a{};
    a.views = static_cast<ViewDesc*>(c->views.p);
    a.V = static_cast<int>(p.views.size());
    a.scenes = reinterpret_cast<SceneDesc*>(static_cast<char*>(c->views.p) + p.views.size() * sizeof(ViewDesc));
    a.weights = static_cast<float*>(c->fwd_weights.p);
    a.o = o;
    a.G = p.G;
    a.recs = static_cast<TriRec*>(c->recs.p);
    a.tile_start = static_cast<int64_t*>(c->tile_start.p);
    a.entries = static_cast<uint64_t*>(c->entries.p);
    a.n_tiles = p.n_tiles;
    unsigned long long* cnt = static_cast<unsigned long long*>(c->counters.p);
    a.counter = c->counting ? cnt : nullptr;
    a.work = reinterpret_cast<unsigned int*>(cnt) + kCountersBytes / 4;
    // the forward's workgroups are single waves, one region of a tile at a time: 16x16 pixels, or a
    // single 8x8 block for 8-pixel tiles and for calls with fewer 16x16 regions than two per resident
    // wave (a small render); as many waves as are resident
    int region = 8;
    if (c->tile >= 16) {
        const int64_t r16 = p.n_tiles * fwd_regions_per_tile(c->tile, 16);
        const int64_t res16 = static_cast<int64_t>(c->num_cus) * raster_fwd_blocks_per_cu(c->tile, kind, 16);
        region = r16 >= 2 * res16 ? 16 : 8;
    }
    a.region = region;
    const int64_t items = p.n_tiles * fwd_regions_per_tile(c->tile, region);
    const int64_t resident = static_cast<int64_t>(c->num_cus) * raster_fwd_blocks_per_cu(c->tile, kind, region);
    a.n_blocks = static_cast<int>(std::max<int64_t>(1, std::min<int64_t>(std::min<int64_t>(resident, kMaxRegions), items)));
    // few single-block regions per wave are all dealt by stride, else only the first round
    a.fixed = static_cast<uint32_t>(region == 8 && items <= int64_t(16) * a.n_blocks
                                        ? (items + a.n_blocks - 1) / a.n_blocks * a.n_blocks : a.n_blocks);
    return a;
}

soup_status finish_stats(soup_ctx* c, hipStream_t s, bool raster = true) {
    if (!c->counting || c->fixed) {
        c->stats.visible_tris = -1;
        c->stats.decodes = -1;
        c->stats.covered_pixels = -1;
        return SOUP_OK;
    }
    unsigned long long h[9];
    HIP_TRY(c, hipMemcpyAsync(h, c->counters.p, sizeof(h), hipMemcpyDeviceToHost, s));
    HIP_TRY(c, hipStreamSynchronize(s));
    c->stats.decodes = static_cast<int64_t>(h[0]);
    c->stats.visible_tris = static_cast<int64_t>(h[1]);
    c->stats.covered_pixels = raster ? static_cast<int64_t>(h[8]) : -1;
    return SOUP_OK;
}

soup_status plan_single(soup_ctx* c, Plan& p, const soup_scene* scene, const soup_views* views) {
    soup_status st = check_scene(c, scene, &p.kind);
    if (st) return st;
    if ((st = check_views(c, views))) return st;
    SceneDesc sd{};
    sd.verts = scene->verts;
    sd.feats = scene->feats;
    sd.mlp = scene->mlp;
    sd.T = scene->T;
    p.scenes = {sd};
    p.G = scene->G;
    p.n_params = mlp_params(scene->n_layers, scene->dims);
    std::vector<int> sov(views->V, 0);
    std::vector<int64_t> rb(views->V);
    for (int i = 0; i < views->V; ++i) rb[i] = static_cast<int64_t>(i) * scene->T;
    p.n_recs = static_cast<int64_t>(views->V) * scene->T;
    plan_views(p, views, c->tile, sov, rb);
    return SOUP_OK;
}

soup_status check_pscene(soup_ctx* c, const soup_pscene* s) {
    if (!s) return fail(c, SOUP_ERR_INVALID, "scene is NULL");
    if (s->T < 0) return fail(c, SOUP_ERR_INVALID, "scene.T = %d < 0", s->T);
    if (s->R < 0 || s->R > kPMaxR) return fail(c, SOUP_ERR_INVALID, "scene.R = %d outside [0, %d]", s->R, kPMaxR);
    if (s->T > 0 && (!s->verts || !s->tex || !s->mlp)) return fail(c, SOUP_ERR_INVALID, "scene device pointers are NULL");
    return SOUP_OK;
}

soup_status plan_paper(soup_ctx* c, Plan& p, const soup_pscene* scene, const soup_views* views,
                       const float* inv_view_proj) {
    soup_status st;
    if ((st = check_pscene(c, scene)) || (st = check_views(c, views))) return st;
    if (!inv_view_proj) return fail(c, SOUP_ERR_INVALID, "inv_view_proj is NULL");
    SceneDesc sd{};
    sd.verts = scene->verts;
    sd.feats = scene->tex;   // the raster reads the opacity channel through the feature pointer
    sd.mlp = scene->mlp;
    sd.T = scene->T;
    p.scenes = {sd};
    p.G = scene->R;          // ... and the texture level through the grid side
    p.kind = MlpKind::kPaper;
    p.n_params = kPParams;
    std::vector<int> sov(views->V, 0);
    std::vector<int64_t> rb(views->V);
    for (int i = 0; i < views->V; ++i) rb[i] = static_cast<int64_t>(i) * scene->T;
    p.n_recs = static_cast<int64_t>(views->V) * scene->T;
    plan_views(p, views, c->tile, sov, rb);
    for (int i = 0; i < views->V; ++i) memcpy(p.views[i].Mi, inv_view_proj + 16 * i, sizeof(p.views[i].Mi));
    return SOUP_OK;
}

}  // namespace

namespace {

// Scratch of soup_loss_l1_ssim_noalloc: the SSIM statistics record (12
// floats per pixel) of one view at a time. Every GPU the library runs on
// holds its own copy of this array until the process ends. Host code never
// passes the array's name to a kernel (on the host it is a stand-in, not a
// device address): it uses the address hipGetSymbolAddress gives on each
// device, kept in noalloc_scratch_ptr.
constexpr size_t kNoAllocScratchBytes = size_t(64) << 20;
constexpr int kNoAllocMaxDevices = 64;
// ... and behind it the loss's parts and running total
static __device__ __align__(256) float scratch[kNoAllocScratchBytes / sizeof(float) + 2 * (kSumParts + 1)];

std::mutex noalloc_scratch_mu;
float* noalloc_scratch_ptr[kNoAllocMaxDevices] = {};

// Once per device, with that device current: the device address of scratch.
soup_status noalloc_scratch_setup(soup_ctx* c) {
    std::lock_guard<std::mutex> lock(noalloc_scratch_mu);
    if (c->device >= kNoAllocMaxDevices)
        return fail(c, SOUP_ERR_UNSUPPORTED, "device %d: the allocation-free entry point supports devices 0..%d",
                    c->device, kNoAllocMaxDevices - 1);
    if (!noalloc_scratch_ptr[c->device]) {
        void* p = nullptr;
        const hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess || !p) {
            (void)hipGetLastError();
            return fail(c, SOUP_ERR_HIP, "hipGetSymbolAddress of the static scratch failed: %s", hipGetErrorString(e));
        }
        noalloc_scratch_ptr[c->device] = static_cast<float*>(p);
    }
    c->scratch = noalloc_scratch_ptr[c->device];
    return SOUP_OK;
}

soup_status log_read(soup_ctx* c, soup_ctx::FragLog& g);

}  // namespace

extern "C" {

soup_status soup_ctx_create(soup_ctx** out, int device) {
    if (!out) return SOUP_ERR_INVALID;
    *out = nullptr;
    int n = 0;
    if (hipGetDeviceCount(&n) != hipSuccess || device < 0 || device >= n) {
        (void)hipGetLastError();
        return SOUP_ERR_HIP;
    }
    if (hipSetDevice(device) != hipSuccess) return SOUP_ERR_HIP;
    soup_ctx* c = new soup_ctx();
    c->device = device;
    hipDeviceProp_t prop;
    if (hipGetDeviceProperties(&prop, device) == hipSuccess && prop.multiProcessorCount > 0)
        c->num_cus = prop.multiProcessorCount;
    int lds = 0;
    if (hipDeviceGetAttribute(&lds, hipDeviceAttributeMaxSharedMemoryPerMultiprocessor, device) == hipSuccess && lds > 0)
        c->lds_limit = static_cast<size_t>(lds);
    else
        (void)hipGetLastError();
    // error messages are formatted into a 512-byte buffer: with this capacity in
    // place, reporting one allocates no memory
    c->err.reserve(512);
    if (noalloc_scratch_setup(c) != SOUP_OK ||
        hipHostMalloc(reinterpret_cast<void**>(&c->host_res), 64, hipHostMallocCoherent) != hipSuccess ||
        hipEventCreateWithFlags(&c->ev_total, hipEventDisableTiming) != hipSuccess ||
        hipEventCreateWithFlags(&c->ev_log, hipEventDisableTiming) != hipSuccess) {
        (void)hipGetLastError();
        soup_ctx_destroy(c);
        return SOUP_ERR_HIP;
    }
    *out = c;
    return SOUP_OK;
}

void soup_ctx_destroy(soup_ctx* c) {
    if (!c) return;
    (void)hipSetDevice(c->device);
    (void)hipDeviceSynchronize();
    DevBuf* bufs[] = {&c->views,      &c->recs,      &c->tile_count, &c->tile_fill,   &c->tile_start,
                      &c->bsum,       &c->entries,     &c->edge_w,    &c->partial,    &c->counters,    &c->tri_count,
                      &c->tri_fill,   &c->tri_off,     &c->tri_bsum,     &c->sorted,      &c->flags,
                      &c->flog.frag,  &c->flog.bary,   &c->flog.counts, &c->rlog.frag, &c->rlog.bary,  &c->rlog.counts,
                      &c->masks,      &c->ssim,        &c->chunk_base, &c->fwd_weights, &c->gvert,     &c->gtex};
    for (DevBuf* b : bufs)
        if (b->p) (void)hipFree(b->p);
    if (c->host_stage) (void)hipHostFree(c->host_stage);
    if (c->host_res) (void)hipHostFree(c->host_res);
    if (c->ev_total) (void)hipEventDestroy(c->ev_total);
    if (c->ev_log) (void)hipEventDestroy(c->ev_log);
    for (auto& m : c->marks) {
        (void)hipEventDestroy(m.a);
        (void)hipEventDestroy(m.b);
    }
    for (hipEvent_t e : c->pool) (void)hipEventDestroy(e);
    delete c;
}

const char* soup_last_error(const soup_ctx* c) { return c ? c->err.c_str() : "context is NULL"; }

soup_status soup_ctx_set_tile(soup_ctx* c, int32_t tile) {
    if (!c) return SOUP_ERR_INVALID;
    if (tile != 8 && tile != 16 && tile != 32) return fail(c, SOUP_ERR_INVALID, "tile = %d (8, 16 or 32)", tile);
    c->tile = tile;
    return SOUP_OK;
}

int32_t soup_ctx_get_tile(const soup_ctx* c) { return c ? c->tile : 0; }

soup_status soup_ctx_set_timing(soup_ctx* c, int32_t on) {
    if (!c) return SOUP_ERR_INVALID;
    c->timing = on != 0;
    return SOUP_OK;
}

soup_status soup_read_timings(soup_ctx* c, double* ms, int64_t* count) {
    if (!c || !ms || !count) return SOUP_ERR_INVALID;
    HIP_TRY(c, hipSetDevice(c->device));
    for (auto& m : c->marks) {
        HIP_TRY(c, hipEventSynchronize(m.b));
        float t = 0.0f;
        HIP_TRY(c, hipEventElapsedTime(&t, m.a, m.b));
        if (m.kind >= 0 && m.kind < SOUP_TIMING_KINDS) {
            ms[m.kind] += t;
            count[m.kind] += 1;
        }
        c->pool.push_back(m.a);
        c->pool.push_back(m.b);
    }
    c->marks.clear();
    return SOUP_OK;
}

soup_status soup_ctx_set_static(soup_ctx* c, int32_t on) {
    if (!c) return SOUP_ERR_INVALID;
    if (on && (c->counting || c->timing))
        return fail(c, SOUP_ERR_INVALID, "static mode excludes counting and timing (both synchronise)");
    // counts that an eager call left to be read size the log's views; none is read in static mode
    soup_status st;
    if ((st = log_read(c, c->flog)) || (st = log_read(c, c->rlog))) return st;
    c->fixed = on != 0;
    return SOUP_OK;
}

soup_status soup_ctx_check(soup_ctx* c) {
    if (!c) return SOUP_ERR_INVALID;
    c->err.clear();
    if (!c->flags.p) return SOUP_OK;
    HIP_TRY(c, hipSetDevice(c->device));
    HIP_TRY(c, hipDeviceSynchronize());
    unsigned int h[2] = {0, 0};
    HIP_TRY(c, hipMemcpy(h, c->flags.p, sizeof(h), hipMemcpyDeviceToHost));
    h[0] &= kOverflowBins | kOverflowFragments;
    if (!h[0]) return SOUP_OK;
    const unsigned int zero[2] = {0, 0};
    HIP_TRY(c, hipMemcpy(c->flags.p, zero, sizeof(zero), hipMemcpyHostToDevice));
    return fail(c, SOUP_ERR_CAPACITY, "a static-mode call overflowed its %s%s%s; rerun outside static mode to grow "
                "the workspaces", (h[0] & kOverflowBins) ? "tile lists" : "",
                (h[0] & kOverflowBins) && (h[0] & kOverflowFragments) ? " and " : "",
                (h[0] & kOverflowFragments) ? "fragment list" : "");
}

soup_status soup_ctx_set_counting(soup_ctx* c, int32_t on) {
    if (!c) return SOUP_ERR_INVALID;
    c->counting = on != 0;
    return SOUP_OK;
}

soup_status soup_ctx_workspace_bytes(const soup_ctx* c, int64_t* bytes) {
    if (!c || !bytes) return SOUP_ERR_INVALID;
    const DevBuf* bufs[] = {&c->views,      &c->recs,      &c->tile_count, &c->tile_fill,   &c->tile_start,
                            &c->bsum,       &c->entries,     &c->edge_w,    &c->partial,    &c->counters,    &c->tri_count,
                            &c->tri_fill,   &c->tri_off,     &c->tri_bsum,     &c->sorted,      &c->flags,
                            &c->flog.frag,  &c->flog.bary,   &c->flog.counts, &c->rlog.frag, &c->rlog.bary,  &c->rlog.counts,
                            &c->masks,      &c->ssim,        &c->chunk_base, &c->fwd_weights, &c->gvert,     &c->gtex};
    int64_t n = 0;
    for (const DevBuf* b : bufs) n += static_cast<int64_t>(b->bytes);
    *bytes = n;
    return SOUP_OK;
}

soup_status soup_last_stats(const soup_ctx* c, soup_stats* out) {
    if (!c || !out) return SOUP_ERR_INVALID;
    *out = c->stats;
    return SOUP_OK;
}

}  // extern "C"

namespace {

// Persistent grid of the decode kernel, workgroups of four waves: two per CU, as many as are
// resident with the 16->32->32->4 decoder (64 views: 2.71 ms; four 2.75, and twice the rows
// of partial sums; three 3.35, the third waits for the first two), fewer where the
// fragments (an upper bound; -1: unknown) give each wave less than a batch of 64. Of the
// 32->64->64->4 decoder, whose LDS leaves room for one, the second half starts behind the
// first (200,000 triangles, 16 views 1080p: 8.29 ms; one per CU 8.20).
int decode_blocks(soup_ctx* c, int64_t fragments) {
    const int64_t most = 2 * static_cast<int64_t>(std::max(1, c->num_cus));
    return static_cast<int>(fragments < 0 ? most : std::max<int64_t>(1, std::min(most, (fragments + 255) / 256)));
}

// The view of a log that its readers take. A region's batches are shared by as many waves as
// give each about eight, and down to one each while there are fewer than 8,192 waves (a batch is a
// chain of dependent loads and an atomic: 128 x 128 pixels, count 10.2 -> 5.4 us, place
// 11.1 -> 5.1; a view of 10,000 triangles 7.7 -> 6.0 and 11.0 -> 8.7).
FragLogView log_view(const soup_ctx::FragLog& g) {
    FragLogView v{};
    v.frag = static_cast<uint4*>(g.frag.p);
    v.bary = static_cast<uint2*>(g.bary.p);
    v.counts = static_cast<uint32_t*>(g.counts.p);
    v.region = static_cast<uint32_t>(g.region);
    v.n_regions = g.regions;
    const uint64_t fill = 8192 / static_cast<uint64_t>(std::max(1, g.regions));
    v.split = static_cast<int>(std::max<uint64_t>(1, std::min<uint64_t>(16, std::max(g.hint / 512, std::min(g.hint / 64, fill)))));
    return v;
}

// Buffers of a log of `regions` regions (a static-mode call takes what an earlier call sized);
// the raster's arguments are set to write it.
soup_status log_reserve(soup_ctx* c, soup_ctx::FragLog& g, int regions, uint64_t region, RasterArgs& a) {
    soup_status st;
    if (c->fixed) {
        if (g.regions != regions || g.region == 0)
            return fail(c, SOUP_ERR_CAPACITY, "static mode: no fragment log sized for this call; run it once "
                        "outside static mode");
    } else {
        if (region >= (uint64_t(1) << 31)) return fail(c, SOUP_ERR_CAPACITY, "fragment log region too large");
        if ((st = ensure(c, g.frag, static_cast<size_t>(region) * regions * sizeof(uint4))) ||
            (st = ensure(c, g.bary, static_cast<size_t>(region) * regions * sizeof(uint2))) ||
            (st = ensure(c, g.counts, static_cast<size_t>(kMaxRegions) * 4)))
            return st;
        g.region = region;
        g.regions = regions;
    }
    a.log_frag = static_cast<uint4*>(g.frag.p);
    a.log_bary = static_cast<uint2*>(g.bary.p);
    a.log_region = static_cast<uint32_t>(g.region);
    a.log_counts = static_cast<uint32_t*>(g.counts.p);
    return SOUP_OK;
}

// After the raster that wrote the log: an eager call leaves the counts to be read behind an event; in
// static mode an overflow is flagged.
soup_status log_written(soup_ctx* c, soup_ctx::FragLog& g, hipStream_t s) {
    unsigned long long* res = reinterpret_cast<unsigned long long*>(c->host_res) + (&g == &c->flog ? 2 : 4);
    launch_log_summary(static_cast<uint32_t*>(g.counts.p), g.regions, static_cast<uint32_t>(g.region),
                       c->fixed ? nullptr : res, c->fixed ? static_cast<unsigned int*>(c->flags.p) : nullptr, s);
    HIP_TRY(c, hipGetLastError());
    g.fits = c->fixed;
    g.pending = !c->fixed;
    if (g.pending) HIP_TRY(c, hipEventRecord(c->ev_log, s));
    return SOUP_OK;
}

// The counts of the last eager raster that wrote the log (waits for it).
soup_status log_read(soup_ctx* c, soup_ctx::FragLog& g) {
    if (!g.pending) return SOUP_OK;
    HIP_TRY(c, hipEventSynchronize(c->ev_log));
    const volatile uint64_t* res = reinterpret_cast<uint64_t*>(c->host_res) + (&g == &c->flog ? 2 : 4);
    g.total = res[0];
    g.hint = res[1];
    g.fits = g.hint <= g.region;
    g.pending = false;
    return SOUP_OK;
}

// Whether the forward's log is there (for these bins) and whole.
soup_status log_usable(soup_ctx* c, bool* ok) {
    *ok = false;
    if (!c->log_valid) return SOUP_OK;
    const soup_status st = log_read(c, c->flog);
    *ok = !st && c->flog.fits;
    return st;
}

// The log of exactly the fragments the backward (or log p: all_front) needs, from a walk with the
// winners known. Regions are sized from the last call's largest count, doubled, since per-wave
// counts vary between calls (else from 1.5 fragments per pixel); an overflow is detected and the
// walk runs again, sized exactly.
soup_status replay(soup_ctx* c, const Plan& p, const Opts& o, const uint64_t* vis, const float* grad_color,
                   const float* grad_logp, const float2* edge_w, bool all_front, hipStream_t s) {
    soup_ctx::FragLog& g = c->rlog;
    RasterArgs a = raster_args(c, p, o, MlpKind::kReplay);
    a.counter = nullptr;
    a.replay_vis = vis;
    a.replay_color = grad_color;
    a.replay_logp = grad_logp;
    a.replay_edge = edge_w;
    a.replay_all = all_front ? 1 : 0;
    const int nr = a.n_blocks;
    uint64_t hint = g.hint;
    if (hint && g.regions && g.regions != nr) hint = hint * g.regions / nr + 64;
    uint64_t region = hint ? 2 * hint + 1024 : (static_cast<uint64_t>(p.n_pix) * 3 / 2) / nr + 1024;
    for (int attempt = 0; attempt < 2; ++attempt) {
        soup_status st;
        if ((st = log_reserve(c, g, nr, region, a))) return st;
        {
            Timed t(c, SOUP_T_REPLAY, s);
            launch_fill_i32(reinterpret_cast<int32_t*>(a.work), kWorkCounters * kWorkStride, 0, s);
            launch_raster_fwd(a, c->tile, MlpKind::kReplay, s);
        }
        // the forward's counts are read before the event is recorded again
        if ((st = log_read(c, c->flog)) || (st = log_written(c, g, s)) || (st = log_read(c, g))) return st;
        if (g.fits) return SOUP_OK;
        region = g.hint + g.hint / 8 + 64;
    }
    return fail(c, SOUP_ERR_CAPACITY, "fragment log overflowed twice");
}

// Backward of an empty soup: no fragments, and a zero gradient of the MLP. (The kernels of the
// fragment list read the parameters, which such a soup may not have, before their first fragment.)
soup_status empty_backward(soup_ctx* c, float* grad_mlp, int n_params, const Opts& o, hipStream_t s) {
    if (!o.accumulate) launch_fill_f32(grad_mlp, n_params, 0.0f, s);
    HIP_TRY(c, hipGetLastError());
    return finish_stats(c, s, false);
}

// Backward, part 1: the fragments the backward needs, from the forward's log or a walk, sorted by
// triangle into c->sorted, with c->tri_off the triangles' ranges. z: what else the backward needs
// cleared before its decode. spare: a log that a static-mode repeat of the call would take instead
// (the forward's where it overflowed: in static mode it is cut and flagged), or null.
soup_status sorted_fragments(soup_ctx* c, const Plan& p, const Opts& o, const uint64_t* vis, const float* grad_color,
                             const float* grad_logp, const float2* edge_w, int T, bool from_log,
                             const soup_ctx::FragLog* spare, ZeroList& z, hipStream_t s) {
    soup_status st;
    if (!from_log && (st = replay(c, p, o, vis, grad_color, grad_logp, edge_w, false, s))) return st;
    const soup_ctx::FragLog& g = from_log ? c->flog : c->rlog;
    const FragLogView L = log_view(g);
    // the sorted list has at most as many entries as the log holds
    size_t entries = static_cast<size_t>(g.regions) * g.region;
    size_t slots = static_cast<size_t>(g.regions) * log_slots(L.region);
    if (spare && !c->fixed) {
        entries = std::max(entries, static_cast<size_t>(spare->regions) * spare->region);
        slots = std::max(slots, static_cast<size_t>(spare->regions) * log_slots(static_cast<uint32_t>(spare->region)));
    }
    if ((st = ensure(c, c->sorted, entries * sizeof(FragRec))) ||
        (st = ensure(c, c->masks, slots * sizeof(ulonglong2))) ||
        (st = ensure(c, c->tri_count, static_cast<size_t>(T) * 4)) ||
        (st = ensure(c, c->tri_fill, static_cast<size_t>(T) * 8)) ||
        (st = ensure(c, c->tri_off, static_cast<size_t>(T + 1) * 8)) ||
        (st = ensure(c, c->tri_bsum, static_cast<size_t>((T + 1023) / 1024 + 1) * 8)))
        return st;
    {
        Timed t(c, SOUP_T_FILL, s);
        z.add(c->tri_count.p, T);
        z.add(c->tri_fill.p, 2 * static_cast<int64_t>(T));
        launch_zero(z, s);
    }
    {
        Timed t(c, SOUP_T_REPLAY, s);
        launch_count(L, FragSelect{vis, grad_logp, 0}, static_cast<ulonglong2*>(c->masks.p),
                     static_cast<int32_t*>(c->tri_count.p), s);
    }
    {
        Timed t(c, SOUP_T_GRAD, s);
        launch_scan(static_cast<int32_t*>(c->tri_count.p), T, 1, static_cast<int64_t*>(c->tri_bsum.p),
                    static_cast<int64_t*>(c->tri_off.p), nullptr, s);
        launch_place(L, grad_logp, static_cast<ulonglong2*>(c->masks.p), static_cast<int64_t*>(c->tri_off.p),
                     static_cast<unsigned long long*>(c->tri_fill.p), static_cast<FragRec*>(c->sorted.p), s);
    }
    HIP_TRY(c, hipGetLastError());
    return SOUP_OK;
}

// The forward raster, with the log of its decoded fragments when `keep`: the
// log is sized from the last call's largest region count (twice, so that a
// static-mode call fits); whether it overflowed is read by who uses it.
soup_status raster_forward(soup_ctx* c, const Plan& p, const Opts& o, RasterArgs& a, bool keep,
                                  hipStream_t s) {
    soup_status st;
    // twice the last call's largest count: per-wave counts vary from call to call (regions are handed
    // out dynamically), and a static-mode call (which cannot grow the log) must fit
    if (keep && ((st = log_read(c, c->flog)) || (st = log_reserve(c, c->flog, a.n_blocks, c->flog.hint ? 2 * c->flog.hint + 1024
                                  : (static_cast<uint64_t>(p.n_pix) * 2) / a.n_blocks + 1024, a))))
        return st;
    {
        Timed t(c, SOUP_T_FWD, s);
        launch_raster_fwd(a, c->tile, p.kind, s);
    }
    HIP_TRY(c, hipGetLastError());
    if (keep) {
        // (an overflowing log is simply not used: the backward replays)
        if ((st = log_written(c, c->flog, s))) return st;
        c->log_valid = true;
        c->log_seed = o.seed;
        c->log_step = o.step;
        c->log_mode = o.mode;
    }
    return SOUP_OK;
}

DecodeArgs decode_args(soup_ctx* c, const Plan& p, const RasterArgs& a) {
    DecodeArgs d{};
    d.views = a.views;
    d.V = a.V;
    d.recs = a.recs;
    d.feats = p.scenes[0].feats;
    d.mlp = p.scenes[0].mlp;
    d.G = p.G;
    d.T = p.scenes[0].T;
    d.verts = p.scenes[0].verts;
    d.counter = a.counter;
    return d;
}

}  // namespace

extern "C" {

soup_status soup_rasterize_fwd(soup_ctx* c, const soup_scene* scene, const soup_views* views, const soup_opts* opts,
                               uint64_t* vis, float* color, float* logp, void* stream) {
    if (!c) return SOUP_ERR_INVALID;
    c->err.clear();
    hipStream_t s = static_cast<hipStream_t>(stream);
    soup_status st;
    Plan p;
    if ((st = plan_single(c, p, scene, views))) return st;
    if ((st = check_opts(c, opts))) return st;
    if (!vis || !color) return fail(c, SOUP_ERR_INVALID, "vis and color outputs are required");
    if (logp && opts->mode == 0 && (st = check_log_pixels(c, "log p", p.n_pix))) return st;
    HIP_TRY(c, hipSetDevice(c->device));
    const Opts o = to_opts(opts);
    if ((st = bin(c, p, o, true, s))) return st;
    RasterArgs a = raster_args(c, p, o, p.kind);
    a.vis = vis;
    a.color = color;
    // reuse_bins: keep a log of the decoded fragments for the backward
    const bool keep = o.reuse_bins != 0;
    if ((st = raster_forward(c, p, o, a, keep, s))) return st;
    if (logp) {
        Timed t(c, SOUP_T_LOGP, s);
        launch_fill_f32(logp, p.n_pix, 0.0f, s);
        if (o.mode == 0) {
            bool from_log = false;
            if (keep && (st = log_usable(c, &from_log))) return st;
            if (!from_log && (st = replay(c, p, o, vis, nullptr, nullptr, nullptr, true, s))) return st;
            LogpArgs la{};
            la.log = log_view(from_log ? c->flog : c->rlog);
            la.sel = FragSelect{vis, nullptr, 1};
            la.feats = p.scenes[0].feats;
            la.mlp = p.scenes[0].mlp;
            la.weights = static_cast<float*>(c->fwd_weights.p);
            la.G = p.G;
            la.logp = logp;
            launch_logp(la, p.kind, s);
        }
        HIP_TRY(c, hipGetLastError());
    }
    return finish_stats(c, s);
}

soup_status soup_rasterize_bwd(soup_ctx* c, const soup_scene* scene, const soup_views* views, const soup_opts* opts,
                               const uint64_t* vis, const float* color, const float* grad_color,
                               const float* grad_logp, float* grad_verts, float* grad_feats, float* grad_mlp,
                               void* stream) {
    if (!c) return SOUP_ERR_INVALID;
    c->err.clear();
    hipStream_t s = static_cast<hipStream_t>(stream);
    soup_status st;
    Plan p;
    if ((st = plan_single(c, p, scene, views))) return st;
    if ((st = check_opts(c, opts))) return st;
    if (!vis || !color || !grad_color) return fail(c, SOUP_ERR_INVALID, "vis, color and grad_color are required");
    if (!grad_verts || !grad_feats || !grad_mlp) return fail(c, SOUP_ERR_INVALID, "gradient outputs are required");
    if ((st = check_decode_lds(c, p.kind, p.G)) || (st = check_log_pixels(c, "backward", p.n_pix)) ||
        (st = check_capture(c, s)))
        return st;
    HIP_TRY(c, hipSetDevice(c->device));
    const Opts o = to_opts(opts);
    bool reused = false;
    if (o.reuse_bins && c->bins_valid && c->bins_tile == c->tile && c->bins_near_w == o.near_w &&
        same_descriptors(c, p)) {
        // the last forward's setup records and tile lists are those of these inputs
        if (c->counting) launch_fill_i32(static_cast<int32_t*>(c->counters.p), kCountersBytes / 4, 0, s);
        reused = true;
    } else if ((st = bin(c, p, o, false, s))) {
        return st;
    }
    const int T = scene->T;
    if (T == 0) return empty_backward(c, grad_mlp, p.n_params, o, s);
    const int64_t n_grid = static_cast<int64_t>(scene->G) * scene->G * scene->C;
    if ((st = ensure(c, c->edge_w, static_cast<size_t>(p.n_pix) * sizeof(float2))) ||
        (st = ensure(c, c->partial, static_cast<size_t>(decode_blocks(c, -1)) * 4 * p.n_params * 4)))
        return st;
    RasterArgs a = raster_args(c, p, o, p.kind);
    const float* gl = o.mode == 0 ? grad_logp : nullptr;
    const float2* ew = nullptr;
    if (o.edge_pairs != 2) {
        Timed t(c, SOUP_T_EDGE, s);
        launch_edge_weights(a.views, a.V, p.n_pix, o, vis, color, grad_color, static_cast<float2*>(c->edge_w.p), s);
        ew = static_cast<float2*>(c->edge_w.p);
    }
    // the last forward's fragment log, if it was made with these draws
    bool from_log = false;
    const bool log_here = reused && c->log_valid && c->log_seed == o.seed && c->log_step == o.step && c->log_mode == o.mode;
    if (log_here && (st = log_usable(c, &from_log))) return st;
    const soup_ctx::FragLog* const spare = log_here && !from_log ? &c->flog : nullptr;
    ZeroList z;
    if (!o.accumulate) {
        z.add(grad_feats, static_cast<int64_t>(T) * n_grid);
        z.add(grad_verts, static_cast<int64_t>(T) * 9);
    }
    if ((st = sorted_fragments(c, p, o, vis, grad_color, gl, ew, T, from_log, spare, z, s))) return st;
    const int nb = decode_blocks(c, c->fixed ? -1 : static_cast<int64_t>((from_log ? c->flog : c->rlog).total));
    {
        DecodeArgs d = decode_args(c, p, a);
        d.n_blocks = nb;
        d.short_list = !c->fixed && static_cast<int64_t>((from_log ? c->flog : c->rlog).total) < static_cast<int64_t>(nb) * 4 * 8 * 64;
        d.sorted = static_cast<FragRec*>(c->sorted.p);
        d.tri_off = static_cast<int64_t*>(c->tri_off.p);
        d.grad_color = grad_color;
        d.edge_w = ew;
        d.grad_feats = grad_feats;
        d.grad_verts = grad_verts;
        d.accumulate = o.accumulate;
        d.mlp_partial = static_cast<float*>(c->partial.p);
        Timed t(c, SOUP_T_BWD, s);
        launch_decode_bwd(d, p.kind, s);
    }
    HIP_TRY(c, hipGetLastError());
    {
        Timed t(c, SOUP_T_REDUCE, s);
        launch_mlp_reduce(static_cast<float*>(c->partial.p), nb * 4, p.n_params, grad_mlp, o.accumulate != 0, s);
    }
    HIP_TRY(c, hipGetLastError());
    return finish_stats(c, s, false);
}

soup_status soup_render(soup_ctx* c, const soup_scene* scenes, int32_t R, const soup_views* views,
                        const soup_opts* opts, float* const* color, void* stream) {
    if (!c) return SOUP_ERR_INVALID;
    c->err.clear();
    hipStream_t s = static_cast<hipStream_t>(stream);
    soup_status st;
    if (R < 1 || !scenes || !color) return fail(c, SOUP_ERR_INVALID, "render needs R >= 1 scenes and outputs");
    if ((st = check_views(c, views))) return st;
    if (views->V != R) return fail(c, SOUP_ERR_INVALID, "views.V = %d != R = %d", views->V, R);
    if ((st = check_opts(c, opts))) return st;
    Plan p;
    std::vector<int> sov(R);
    std::vector<int64_t> rb(R);
    int64_t recs = 0;
    for (int r = 0; r < R; ++r) {
        MlpKind k;
        if ((st = check_scene(c, &scenes[r], &k))) return st;
        if (r == 0) {
            p.kind = k;
            p.G = scenes[0].G;
        } else if (k != p.kind || scenes[r].G != p.G || scenes[r].C != scenes[0].C) {
            return fail(c, SOUP_ERR_INVALID, "request %d: all scenes of a batch must share G, C and the MLP shape", r);
        }
        if (!color[r]) return fail(c, SOUP_ERR_INVALID, "request %d: color output is NULL", r);
        SceneDesc sd{};
        sd.verts = scenes[r].verts;
        sd.feats = scenes[r].feats;
        sd.mlp = scenes[r].mlp;
        sd.T = scenes[r].T;
        p.scenes.push_back(sd);
        sov[r] = r;
        rb[r] = recs;
        recs += scenes[r].T;
    }
    p.n_recs = recs;
    plan_views(p, views, c->tile, sov, rb);
    for (int r = 0; r < R; ++r) p.views[r].color_out = color[r];
    HIP_TRY(c, hipSetDevice(c->device));
    const Opts o = to_opts(opts);
    if ((st = bin(c, p, o, true, s))) return st;
    RasterArgs a = raster_args(c, p, o, p.kind);
    a.vis = nullptr;
    a.color = nullptr;
    {
        Timed t(c, SOUP_T_FWD, s);
        launch_raster_fwd(a, c->tile, p.kind, s);
    }
    HIP_TRY(c, hipGetLastError());
    return finish_stats(c, s);
}

soup_status soup_pforward(soup_ctx* c, const soup_pscene* scene, const soup_views* views, const float* inv_view_proj,
                          const soup_opts* opts, uint64_t* vis, float* color, float* logp, void* stream) {
    if (!c) return SOUP_ERR_INVALID;
    c->err.clear();
    hipStream_t s = static_cast<hipStream_t>(stream);
    soup_status st;
    Plan p;
    if ((st = plan_paper(c, p, scene, views, inv_view_proj))) return st;
    if ((st = check_opts(c, opts))) return st;
    if (!vis || !color) return fail(c, SOUP_ERR_INVALID, "vis and color outputs are required");
    if (logp && opts->mode == 0 && (st = check_log_pixels(c, "log p", p.n_pix))) return st;
    HIP_TRY(c, hipSetDevice(c->device));
    const Opts o = to_opts(opts);
    if ((st = bin(c, p, o, true, s))) return st;
    RasterArgs a = raster_args(c, p, o, p.kind);
    a.vis = vis;
    a.color = color;
    const bool keep = o.reuse_bins != 0 || (logp && o.mode == 0);
    if ((st = raster_forward(c, p, o, a, keep, s))) return st;
    {
        Timed t(c, SOUP_T_SHADE, s);
        PShadeArgs sa{};
        sa.views = a.views;
        sa.V = a.V;
        sa.P = p.n_pix;
        sa.recs = a.recs;
        sa.tex = scene->tex;
        sa.mlp = scene->mlp;
        sa.R = scene->R;
        sa.vis = vis;
        sa.color = color;
        sa.o = o;
        launch_pshade(sa, s);
    }
    HIP_TRY(c, hipGetLastError());
    if (logp) {
        Timed t(c, SOUP_T_LOGP, s);
        launch_fill_f32(logp, p.n_pix, 0.0f, s);
        if (o.mode == 0) {
            bool from_log = false;
            if ((st = log_usable(c, &from_log))) return st;
            if (!from_log && (st = replay(c, p, o, vis, nullptr, nullptr, nullptr, true, s))) return st;
            PFragArgs fa{};
            fa.log = log_view(from_log ? c->flog : c->rlog);
            fa.sel = FragSelect{vis, nullptr, 1};
            fa.tex = scene->tex;
            fa.R = scene->R;
            fa.logp = logp;
            launch_pfrag(fa, true, s);
        }
        HIP_TRY(c, hipGetLastError());
    }
    return finish_stats(c, s);
}

static soup_status check_levels(soup_ctx* c, int32_t T, int32_t Rmin, int32_t Rtop, int32_t Rmax) {
    if (T < 0) return fail(c, SOUP_ERR_INVALID, "T = %d < 0", T);
    if (Rmin < 0 || Rtop < Rmin || Rmax < Rtop || Rmax > kPMaxR || Rtop - Rmin + 1 > kPMaxLevels)
        return fail(c, SOUP_ERR_INVALID, "levels Rmin = %d, Rtop = %d, Rmax = %d: need 0 <= Rmin <= Rtop <= Rmax <= %d",
                    Rmin, Rtop, Rmax, kPMaxR);
    return SOUP_OK;
}

// The learnable levels a backward writes instead of the assembled texture's gradient.
struct LevelsOut {
    int Rmin, Rtop;
    float* const* graw;
};

static soup_status pbackward_impl(soup_ctx* c, const soup_pscene* scene, const soup_views* views,
                                  const float* inv_view_proj, const soup_opts* opts, const uint64_t* vis,
                                  const float* color, const float* grad_color, const float* grad_logp,
                                  float* grad_verts, float* grad_tex, const LevelsOut* lv, float* grad_mlp,
                                  void* stream) {
    if (!c) return SOUP_ERR_INVALID;
    c->err.clear();
    hipStream_t s = static_cast<hipStream_t>(stream);
    soup_status st;
    Plan p;
    if ((st = plan_paper(c, p, scene, views, inv_view_proj))) return st;
    if ((st = check_opts(c, opts))) return st;
    if (!vis || !color || !grad_color) return fail(c, SOUP_ERR_INVALID, "vis, color and grad_color are required");
    // an empty soup has empty vertex and texture gradients (their pointers may be NULL)
    if (!grad_mlp || (scene->T > 0 && (!grad_verts || (!lv && !grad_tex))))
        return fail(c, SOUP_ERR_INVALID, "gradient outputs are required");
    if (lv) {
        if ((st = check_levels(c, scene->T, lv->Rmin, lv->Rtop, scene->R))) return st;
        if (scene->T > 0) {
            if (!lv->graw) return fail(c, SOUP_ERR_INVALID, "grad_raw is NULL");
            for (int l = 0; l <= lv->Rtop - lv->Rmin; ++l)
                if (!lv->graw[l]) return fail(c, SOUP_ERR_INVALID, "grad_raw[%d] (level %d) is NULL", l, lv->Rmin + l);
        }
    }
    // (the per-pixel path takes its score term alone from a log)
    if ((ptri_sorted(scene->R) || (grad_logp && opts->mode == 0)) &&
        ((st = check_log_pixels(c, "backward", p.n_pix)) || (st = check_capture(c, s))))
        return st;
    HIP_TRY(c, hipSetDevice(c->device));
    const Opts o = to_opts(opts);
    bool reused = false;
    if (o.reuse_bins && c->bins_valid && c->bins_tile == c->tile && c->bins_near_w == o.near_w &&
        same_descriptors(c, p)) {
        if (c->counting) launch_fill_i32(static_cast<int32_t*>(c->counters.p), kCountersBytes / 4, 0, s);
        reused = true;
    } else if ((st = bin(c, p, o, false, s))) {
        return st;
    }
    const int T = scene->T;
    if (T == 0) return empty_backward(c, grad_mlp, kPParams, o, s);
    const int64_t n_tex = static_cast<int64_t>(T) * mc_count(scene->R) * kPCh;
    // the triangle-sorted path keeps one triangle's texture gradient per wave in LDS
    // (18 KB at R = 5, with the levels' restriction 11); a texture too large for that
    // takes the per-pixel path with global atomics
    const bool sorted_path = ptri_sorted(scene->R);
    // levels: folded into the sorted path's flush; otherwise the texture gradient goes
    // to a workspace and through the assembly's backward
    const bool fused = lv && sorted_path;
    if (lv && !fused) {
        if ((st = ensure(c, c->gtex, static_cast<size_t>(n_tex) * sizeof(float)))) return st;
        grad_tex = static_cast<float*>(c->gtex.p);
    }
    const int nb = sorted_path ? ptri_blocks(c->num_cus, fused, scene->R, lv ? lv->Rmin : 0, lv ? lv->Rtop : 0)
                               : pwinner_blocks(c->num_cus);
    const int rows = sorted_path ? nb : nb * 4;
    // the partial sums' rows do not depend on the levels (eight waves per CU at most)
    const int most = sorted_path ? std::max(nb, 8 * c->num_cus) : rows;
    if ((st = ensure(c, c->edge_w, static_cast<size_t>(p.n_pix) * sizeof(float2))) ||
        (st = ensure(c, c->partial, static_cast<size_t>(most) * kPParams * 4)) ||
        (st = ensure(c, c->gvert, static_cast<size_t>(T) * 9 * sizeof(double))))
        return st;
    RasterArgs a = raster_args(c, p, o, p.kind);
    const float2* ew = nullptr;
    if (o.edge_pairs != 2) {
        Timed t(c, SOUP_T_EDGE, s);
        launch_edge_weights(a.views, a.V, p.n_pix, o, vis, color, grad_color, static_cast<float2*>(c->edge_w.p), s);
        ew = static_cast<float2*>(c->edge_w.p);
    }
    bool from_log = false;
    const bool log_here = reused && c->log_valid && c->log_seed == o.seed && c->log_step == o.step && c->log_mode == o.mode;
    if (log_here && (st = log_usable(c, &from_log))) return st;
    const soup_ctx::FragLog* const spare = log_here && !from_log ? &c->flog : nullptr;
    ZeroList z;
    z.add(c->gvert.p, static_cast<int64_t>(T) * 18);
    if (fused) {
        if (!o.accumulate)
            for (int l = 0; l <= lv->Rtop - lv->Rmin; ++l)
                z.add(lv->graw[l], static_cast<int64_t>(T) * mc_count(lv->Rmin + l) * kPCh);
    } else if (!o.accumulate || lv) {   // the workspace starts from zero
        z.add(grad_tex, n_tex);
    }
    const float* gl = o.mode == 0 ? grad_logp : nullptr;
    if (sorted_path) {
        // every winner and, where the pixel carries a score weight, every fragment in
        // front of it (Eq. (9)), sorted by triangle
        if ((st = sorted_fragments(c, p, o, vis, grad_color, gl, ew, T, from_log, spare, z, s))) return st;
        Timed t(c, SOUP_T_BWD, s);
        PTriArgs ta{};
        ta.views = a.views;
        ta.recs = a.recs;
        ta.verts = scene->verts;
        ta.tex = scene->tex;
        ta.mlp = scene->mlp;
        ta.R = scene->R;
        ta.T = T;
        ta.sorted = static_cast<FragRec*>(c->sorted.p);
        ta.tri_off = static_cast<int64_t*>(c->tri_off.p);
        ta.grad_color = grad_color;
        ta.edge_w = ew;
        ta.score = gl ? 1 : 0;
        ta.accumulate = lv && !fused ? 0 : o.accumulate;
        ta.grad_tex = fused ? nullptr : grad_tex;
        if (fused) {
            ta.levels = 1;
            ta.Rmin = lv->Rmin;
            ta.Rtop = lv->Rtop;
            for (int l = 0; l <= lv->Rtop - lv->Rmin; ++l) ta.graw[l] = lv->graw[l];
        }
        ta.gvert = static_cast<double*>(c->gvert.p);
        ta.mlp_partial = static_cast<float*>(c->partial.p);
        ta.n_blocks = nb;
        launch_ptri_bwd(ta, s);
    } else {
        {
            Timed t(c, SOUP_T_FILL, s);
            launch_zero(z, s);
        }
        if (gl) {
            // the score term (Eq. (9)): every fragment in front of a winner, and the winner
            if (!from_log && (st = replay(c, p, o, vis, grad_color, gl, nullptr, false, s))) return st;
            Timed t(c, SOUP_T_GRAD, s);
            PFragArgs fa{};
            fa.log = log_view(from_log ? c->flog : c->rlog);
            fa.sel = FragSelect{vis, gl, 0};
            fa.tex = scene->tex;
            fa.R = scene->R;
            fa.grad_tex = grad_tex;
            launch_pfrag(fa, false, s);
        }
        Timed t(c, SOUP_T_BWD, s);
        PWinArgs wa{};
        wa.views = a.views;
        wa.V = a.V;
        wa.P = p.n_pix;
        wa.recs = a.recs;
        wa.verts = scene->verts;
        wa.tex = scene->tex;
        wa.mlp = scene->mlp;
        wa.R = scene->R;
        wa.vis = vis;
        wa.grad_color = grad_color;
        wa.edge_w = ew;
        wa.grad_tex = grad_tex;
        wa.gvert = static_cast<double*>(c->gvert.p);
        wa.mlp_partial = static_cast<float*>(c->partial.p);
        wa.n_blocks = nb;
        launch_pwinner_bwd(wa, s);
    }
    HIP_TRY(c, hipGetLastError());
    if (lv && !fused) {   // the workspace's texture gradient through the assembly's backward
        Timed t(c, SOUP_T_ASSEMBLE_BWD, s);
        AssembleArgs aa{};
        for (int l = 0; l <= lv->Rtop - lv->Rmin; ++l) aa.graw[l] = lv->graw[l];
        aa.Rmin = lv->Rmin;
        aa.Rtop = lv->Rtop;
        aa.Rmax = scene->R;
        aa.T = T;
        aa.tex = scene->tex;
        aa.grad_tex = grad_tex;
        aa.accumulate = o.accumulate;
        if (mc_assemble_bwd_lds(aa.Rmin, aa.Rmax) > mc_assemble_bwd_lds_cap(c->lds_limit) && !o.accumulate)
            for (int l = 0; l <= aa.Rtop - aa.Rmin; ++l)
                launch_fill_f32(aa.graw[l], static_cast<int64_t>(T) * mc_count(aa.Rmin + l) * kPCh, 0.0f, s);
        launch_mc_assemble_bwd(aa, c->lds_limit, s);
    }
    {
        Timed t(c, SOUP_T_REDUCE, s);
        launch_pvert_finish(static_cast<double*>(c->gvert.p), grad_verts, static_cast<int64_t>(T) * 9,
                            o.accumulate != 0, s);
        launch_mlp_reduce(static_cast<float*>(c->partial.p), rows, kPParams, grad_mlp, o.accumulate != 0, s);
    }
    HIP_TRY(c, hipGetLastError());
    return finish_stats(c, s, false);
}

soup_status soup_pbackward(soup_ctx* c, const soup_pscene* scene, const soup_views* views, const float* inv_view_proj,
                           const soup_opts* opts, const uint64_t* vis, const float* color, const float* grad_color,
                           const float* grad_logp, float* grad_verts, float* grad_tex, float* grad_mlp,
                           void* stream) {
    return pbackward_impl(c, scene, views, inv_view_proj, opts, vis, color, grad_color, grad_logp, grad_verts, grad_tex,
                          nullptr, grad_mlp, stream);
}

soup_status soup_pbackward_levels(soup_ctx* c, const soup_pscene* scene, const soup_views* views,
                                  const float* inv_view_proj, const soup_opts* opts, const uint64_t* vis,
                                  const float* color, const float* grad_color, const float* grad_logp,
                                  int32_t Rmin, int32_t Rtop, float* grad_verts, float* const* grad_raw,
                                  float* grad_mlp, void* stream) {
    const LevelsOut lv{Rmin, Rtop, grad_raw};
    return pbackward_impl(c, scene, views, inv_view_proj, opts, vis, color, grad_color, grad_logp, grad_verts, nullptr,
                          &lv, grad_mlp, stream);
}

soup_status soup_mc_assemble(soup_ctx* c, int32_t T, int32_t Rmin, int32_t Rtop, int32_t Rmax, const float* const* raw,
                             float* tex, void* stream) {
    if (!c) return SOUP_ERR_INVALID;
    c->err.clear();
    soup_status st;
    if ((st = check_levels(c, T, Rmin, Rtop, Rmax))) return st;
    if (T > 0 && (!raw || !tex)) return fail(c, SOUP_ERR_INVALID, "mc_assemble: NULL buffers");
    if (T == 0) return SOUP_OK;
    AssembleArgs aa{};
    for (int l = 0; l <= Rtop - Rmin; ++l) {
        if (!raw[l]) return fail(c, SOUP_ERR_INVALID, "mc_assemble: level %d is NULL", Rmin + l);
        aa.raw[l] = raw[l];
    }
    aa.Rmin = Rmin;
    aa.Rtop = Rtop;
    aa.Rmax = Rmax;
    aa.T = T;
    aa.tex_out = tex;
    HIP_TRY(c, hipSetDevice(c->device));
    hipStream_t s = static_cast<hipStream_t>(stream);
    {
        Timed t(c, SOUP_T_ASSEMBLE, s);
        launch_mc_assemble(aa, s);
    }
    HIP_TRY(c, hipGetLastError());
    return SOUP_OK;
}

soup_status soup_mc_assemble_bwd(soup_ctx* c, int32_t T, int32_t Rmin, int32_t Rtop, int32_t Rmax, const float* tex,
                                 const float* grad_tex, float* const* grad_raw, int32_t accumulate, void* stream) {
    if (!c) return SOUP_ERR_INVALID;
    c->err.clear();
    soup_status st;
    if ((st = check_levels(c, T, Rmin, Rtop, Rmax))) return st;
    if (accumulate != 0 && accumulate != 1) return fail(c, SOUP_ERR_INVALID, "accumulate = %d (0 or 1)", accumulate);
    if (T > 0 && (!tex || !grad_tex || !grad_raw)) return fail(c, SOUP_ERR_INVALID, "mc_assemble_bwd: NULL buffers");
    if (T == 0) return SOUP_OK;
    AssembleArgs aa{};
    for (int l = 0; l <= Rtop - Rmin; ++l) {
        if (!grad_raw[l]) return fail(c, SOUP_ERR_INVALID, "mc_assemble_bwd: level %d is NULL", Rmin + l);
        aa.graw[l] = grad_raw[l];
    }
    aa.Rmin = Rmin;
    aa.Rtop = Rtop;
    aa.Rmax = Rmax;
    aa.T = T;
    aa.tex = tex;
    aa.grad_tex = grad_tex;
    aa.accumulate = accumulate;
    HIP_TRY(c, hipSetDevice(c->device));
    hipStream_t s = static_cast<hipStream_t>(stream);
    {
        Timed t(c, SOUP_T_ASSEMBLE_BWD, s);
        if (mc_assemble_bwd_lds(Rmin, Rmax) > mc_assemble_bwd_lds_cap(c->lds_limit) && !accumulate)
            for (int l = 0; l <= Rtop - Rmin; ++l)
                launch_fill_f32(grad_raw[l], static_cast<int64_t>(T) * mc_count(Rmin + l) * kPCh, 0.0f, s);
        launch_mc_assemble_bwd(aa, c->lds_limit, s);
    }
    HIP_TRY(c, hipGetLastError());
    return SOUP_OK;
}

soup_status soup_loss_l2(soup_ctx* c, const float* color, const float* target, int64_t P, float* grad_color,
                         float* grad_logp, float* loss, void* stream) {
    if (!c) return SOUP_ERR_INVALID;
    c->err.clear();
    if (P < 0 || (P > 0 && (!color || !target || !grad_color || !grad_logp)))
        return fail(c, SOUP_ERR_INVALID, "loss_l2: bad arguments");
    HIP_TRY(c, hipSetDevice(c->device));
    {
        Timed t(c, SOUP_T_LOSS, static_cast<hipStream_t>(stream));
        launch_loss_l2(color, target, P, grad_color, grad_logp, loss, static_cast<hipStream_t>(stream));
    }
    HIP_TRY(c, hipGetLastError());
    return SOUP_OK;
}

soup_status soup_coverage_count(soup_ctx* c, const uint64_t* vis, int64_t n, int32_t T, uint32_t* counts,
                                void* stream) {
    if (!c) return SOUP_ERR_INVALID;
    c->err.clear();
    if (n < 0 || T < 0 || (n > 0 && !vis) || (T > 0 && !counts))
        return fail(c, SOUP_ERR_INVALID, "coverage_count: bad arguments (n = %lld, T = %d)", (long long)n, T);
    HIP_TRY(c, hipSetDevice(c->device));
    {
        Timed t(c, SOUP_T_COVER, static_cast<hipStream_t>(stream));
        launch_coverage(vis, n, T, counts, c->num_cus, static_cast<hipStream_t>(stream));
    }
    HIP_TRY(c, hipGetLastError());
    return SOUP_OK;
}

soup_status soup_edge_lengths(soup_ctx* c, const float* verts, int32_t T, const soup_views* v, float near_w,
                              float* rel_len, void* stream) {
    if (!c) return SOUP_ERR_INVALID;
    c->err.clear();
    if (T < 0 || (T > 0 && (!verts || !rel_len))) return fail(c, SOUP_ERR_INVALID, "edge_lengths: bad arguments");
    if (!v || v->V < 1 || !v->width || !v->height || !v->view_proj)
        return fail(c, SOUP_ERR_INVALID, "edge_lengths: views missing");
    for (int i = 0; i < v->V; ++i)
        if (v->width[i] < 1 || v->width[i] > 16384 || v->height[i] < 1 || v->height[i] > 16384)
            return fail(c, SOUP_ERR_INVALID, "view %d size %dx%d outside [1, 16384]", i, v->width[i], v->height[i]);
    if (!(near_w > 0.0f)) return fail(c, SOUP_ERR_INVALID, "edge_lengths: near_w must be > 0");
    HIP_TRY(c, hipSetDevice(c->device));
    const hipStream_t s = static_cast<hipStream_t>(stream);
    {
        Timed t(c, SOUP_T_EDGELEN, s);
        for (int v0 = 0; v0 < v->V; v0 += soup::kEdgeViews) {
            soup::EdgeViews ev{};
            ev.n = std::min(soup::kEdgeViews, v->V - v0);
            for (int i = 0; i < ev.n; ++i) {
                std::memcpy(ev.m[i], v->view_proj + static_cast<size_t>(v0 + i) * 16, 16 * sizeof(float));
                ev.w[i] = static_cast<float>(v->width[v0 + i]);
                ev.h[i] = static_cast<float>(v->height[v0 + i]);
            }
            launch_edge_lengths(verts, T, ev, near_w, v0 == 0, rel_len, s);
        }
    }
    HIP_TRY(c, hipGetLastError());
    return SOUP_OK;
}

soup_status soup_adaptive_plan(soup_ctx* c, const uint32_t* counts, const float* rel_len, int32_t T, float split_frac,
                               int32_t target, int32_t flags, int32_t* actions, int32_t* offsets, int32_t* n_new) {
    if (c) c->err.clear();
    if (!n_new || T < 0 || T > (1 << 30) || target < 0 || (flags & ~3) != 0 ||
        (T > 0 && (!counts || !rel_len || !actions || !offsets)))
        return fail(c, SOUP_ERR_INVALID, "adaptive_plan: bad arguments (T = %d, target = %d, flags = %d)", T, target,
                    flags);
    if (!(split_frac == split_frac)) return fail(c, SOUP_ERR_INVALID, "adaptive_plan: split_frac is NaN");
    try {
        *n_new = soup::plan_host(counts, rel_len, T, split_frac, target, (flags & SOUP_PLAN_PRUNE_ZERO) != 0,
                                 (flags & SOUP_PLAN_FILL) != 0, actions, offsets);
    } catch (const std::bad_alloc&) {
        return fail(c, SOUP_ERR_OOM, "adaptive_plan: no host memory for %d triangles", T);
    }
    return SOUP_OK;
}

soup_status soup_adaptive_apply(soup_ctx* c, const soup_scene* sc, const int32_t* actions, const int32_t* offsets,
                                int32_t n_new, float* verts_out, float* feats_out, void* stream) {
    if (!c) return SOUP_ERR_INVALID;
    c->err.clear();
    if (!sc || sc->T < 0 || sc->G < 2 || sc->G > 256 || sc->C < 1 || n_new < 0)
        return fail(c, SOUP_ERR_INVALID, "adaptive_apply: bad scene or n_new");
    if (sc->T > 0 && (!sc->verts || !sc->feats || !actions || !offsets))
        return fail(c, SOUP_ERR_INVALID, "adaptive_apply: device pointers are NULL");
    if (n_new > 0 && (!verts_out || !feats_out))
        return fail(c, SOUP_ERR_INVALID, "adaptive_apply: output pointers are NULL");
    if ((reinterpret_cast<uintptr_t>(sc->feats) | reinterpret_cast<uintptr_t>(feats_out)) & 15)
        return fail(c, SOUP_ERR_INVALID, "adaptive_apply: feats and feats_out must be 16-byte aligned");
    HIP_TRY(c, hipSetDevice(c->device));
    {
        Timed t(c, SOUP_T_APPLY, static_cast<hipStream_t>(stream));
        launch_apply(sc->verts, sc->feats, actions, offsets, sc->T, sc->G, sc->C, n_new, verts_out, feats_out,
                     static_cast<hipStream_t>(stream));
    }
    HIP_TRY(c, hipGetLastError());
    return SOUP_OK;
}

namespace {

// Arguments of the L1 + D-SSIM loss: the total and the largest view's pixels.
soup_status check_loss_l1_ssim(soup_ctx* c, const float* color, const float* target, const soup_views* v,
                               float lambda, const float* grad_color, const float* grad_logp, int64_t* P_out,
                               int64_t* maxp_out) {
    if (!v || v->V < 1 || !v->width || !v->height) return fail(c, SOUP_ERR_INVALID, "loss_l1_ssim: views missing");
    if (!(lambda >= 0.0f && lambda <= 1.0f)) return fail(c, SOUP_ERR_INVALID, "loss_l1_ssim: lambda outside [0, 1]");
    int64_t P = 0, maxp = 0;
    for (int i = 0; i < v->V; ++i) {
        if (v->width[i] < 1 || v->width[i] > 16384 || v->height[i] < 1 || v->height[i] > 16384)
            return fail(c, SOUP_ERR_INVALID, "view %d size %dx%d outside [1, 16384]", i, v->width[i], v->height[i]);
        const int64_t np = static_cast<int64_t>(v->width[i]) * v->height[i];
        P += np;
        maxp = std::max(maxp, np);
    }
    if (!color || !target || !grad_color || !grad_logp)
        return fail(c, SOUP_ERR_INVALID, "loss_l1_ssim: device pointers are NULL");
    *P_out = P;
    *maxp_out = maxp;
    return SOUP_OK;
}

// The loss's launches, with the statistics record in `stats` (12 floats per pixel for
// stat_pixels pixels, at least the largest view's). Allocates nothing when `timed`
// is false (the timing events come from a pool that may grow).
void loss_l1_ssim_launch(soup_ctx* c, const float* color, const float* target, const soup_views* v, float lambda,
                         float* grad_color, float* grad_logp, float* loss, int64_t P, float* stats,
                         int64_t stat_pixels, double* parts, bool timed, hipStream_t s) {
    // the window: normalised 1-D Gaussian, sigma 1.5, summed in double
    soup::SsimWindow win{};
    double g[2 * soup::kSsimR + 1], sum = 0.0;
    for (int i = 0; i <= 2 * soup::kSsimR; ++i) {
        const double x = i - soup::kSsimR;
        g[i] = std::exp(-x * x / (2.0 * 1.5 * 1.5));
        sum += g[i];
    }
    for (int i = 0; i <= 2 * soup::kSsimR; ++i) win.g[i] = static_cast<float>(g[i] / sum);
    const float inv_n = static_cast<float>(1.0 / (3.0 * static_cast<double>(P)));
    auto run = [&]() {
        // views in order, as many per batch as the record and the kernel argument hold
        soup::SsimBatch b{};
        b.color = color;
        b.target = target;
        b.grad_color = grad_color;
        b.grad_logp = grad_logp;
        b.stats = stats;
        int64_t off = 0, in_batch = 0;
        for (int i = 0; i < v->V; ++i) {
            const int64_t np = static_cast<int64_t>(v->width[i]) * v->height[i];
            if (b.n > 0 && (b.n == soup::kSsimViews || in_batch + np > stat_pixels)) {
                launch_loss_l1_ssim(b, lambda, inv_n, win, loss, parts, s);
                b.n = 0;
                b.add = 1;
                in_batch = 0;
            }
            b.pix[b.n] = off;
            b.w[b.n] = v->width[i];
            b.h[b.n] = v->height[i];
            if (b.n == 0) b.tile[0] = 0;
            b.tile[b.n + 1] = b.tile[b.n] + soup::ssim_tiles(v->width[i], v->height[i]);
            ++b.n;
            off += np;
            in_batch += np;
        }
        b.last = 1;
        launch_loss_l1_ssim(b, lambda, inv_n, win, loss, parts, s);
    };
    if (timed) {
        Timed t(c, SOUP_T_TLOSS, s);
        run();
    } else {
        run();
    }
}

}  // namespace

soup_status soup_loss_l1_ssim(soup_ctx* c, const float* color, const float* target, const soup_views* v,
                              float lambda, float* grad_color, float* grad_logp, float* loss, void* stream) {
    if (!c) return SOUP_ERR_INVALID;
    c->err.clear();
    int64_t P = 0, maxp = 0;
    soup_status st = check_loss_l1_ssim(c, color, target, v, lambda, grad_color, grad_logp, &P, &maxp);
    if (st != SOUP_OK) return st;
    HIP_TRY(c, hipSetDevice(c->device));
    // records for the largest view, or for as many views as 4 Mpixel hold (192 MB) where that is more; where
    // that is not to be had (static mode, memory) the views share fewer launches
    constexpr size_t kRecord = 12 * sizeof(float), kParts = (kSumParts + 2) * sizeof(double);   // (16-byte multiples)
    int64_t stat_pixels = std::max(maxp, std::min<int64_t>(P, int64_t(1) << 22));
    if (c->fixed && c->ssim.bytes > kParts)
        stat_pixels = std::max(maxp, std::min(stat_pixels, static_cast<int64_t>((c->ssim.bytes - kParts) / kRecord)));
    st = ensure(c, c->ssim, kParts + static_cast<size_t>(stat_pixels) * kRecord);
    if (st == SOUP_ERR_OOM && stat_pixels > maxp) {
        stat_pixels = maxp;
        c->err.clear();
        st = ensure(c, c->ssim, kParts + static_cast<size_t>(stat_pixels) * kRecord);
    }
    if (st) return st;
    loss_l1_ssim_launch(c, color, target, v, lambda, grad_color, grad_logp, loss, P,
                        reinterpret_cast<float*>(static_cast<char*>(c->ssim.p) + kParts), stat_pixels,
                        static_cast<double*>(c->ssim.p), true, static_cast<hipStream_t>(stream));
    HIP_TRY(c, hipGetLastError());
    return SOUP_OK;
}

soup_status soup_loss_l1_ssim_noalloc(soup_ctx* c, const float* color, const float* target, const soup_views* v,
                                      float lambda, float* grad_color, float* grad_logp, float* loss, void* stream) {
    if (!c) return SOUP_ERR_INVALID;
    c->err.clear();
    int64_t P = 0, maxp = 0;
    soup_status st = check_loss_l1_ssim(c, color, target, v, lambda, grad_color, grad_logp, &P, &maxp);
    if (st != SOUP_OK) return st;
    const int64_t max_pixels = static_cast<int64_t>(kNoAllocScratchBytes / (12 * sizeof(float)));
    if (maxp > max_pixels)
        return fail(c, SOUP_ERR_CAPACITY, "loss_l1_ssim_noalloc: a view of %lld pixels exceeds the static scratch "
                    "(%zu MiB: views of at most %lld pixels); use soup_loss_l1_ssim", static_cast<long long>(maxp),
                    kNoAllocScratchBytes >> 20, static_cast<long long>(max_pixels));
    if (!c->scratch) return fail(c, SOUP_ERR_HIP, "loss_l1_ssim_noalloc: the static scratch has no device address");
    HIP_TRY(c, hipSetDevice(c->device));
    double* parts = reinterpret_cast<double*>(c->scratch + kNoAllocScratchBytes / sizeof(float));
    loss_l1_ssim_launch(c, color, target, v, lambda, grad_color, grad_logp, loss, P, c->scratch, max_pixels,
                        parts, false,
                        static_cast<hipStream_t>(stream));
    HIP_TRY(c, hipGetLastError());
    return SOUP_OK;
}

soup_status soup_adam_step(soup_ctx* c, float* p, const float* g, float* m, float* v, int64_t n, int32_t vec, float lr,
                           double beta1, double beta2, float eps, int32_t t, void* stream) {
    if (!c) return SOUP_ERR_INVALID;
    c->err.clear();
    if (n < 0 || vec < 1 || vec > 4 || n % vec != 0 || t < 1 || (n > 0 && (!p || !g || !m || !v)))
        return fail(c, SOUP_ERR_INVALID, "adam_step: bad arguments (n = %lld, vec = %d, t = %d)", (long long)n, vec, t);
    if (!(beta1 >= 0.0 && beta1 < 1.0 && beta2 >= 0.0 && beta2 < 1.0 && eps >= 0.0f))
        return fail(c, SOUP_ERR_INVALID, "adam_step: betas must lie in [0, 1) and eps >= 0");
    HIP_TRY(c, hipSetDevice(c->device));
    const float bc1 = static_cast<float>(1.0 - std::pow(beta1, t));
    const float bc2 = static_cast<float>(1.0 - std::pow(beta2, t));
    {
        Timed tm(c, SOUP_T_ADAM, static_cast<hipStream_t>(stream));
        launch_adam(p, g, m, v, n / vec, vec, lr, static_cast<float>(beta1), static_cast<float>(1.0 - beta1),
                    static_cast<float>(beta2), static_cast<float>(1.0 - beta2), eps, bc1, bc2,
                    static_cast<hipStream_t>(stream));
    }
    HIP_TRY(c, hipGetLastError());
    return SOUP_OK;
}

soup_status soup_selftest_sigmoid(soup_ctx* c, const float* x, float* y, int64_t n, void* stream) {
    if (!c) return SOUP_ERR_INVALID;
    if (n < 0 || (n > 0 && (!x || !y))) return fail(c, SOUP_ERR_INVALID, "selftest_sigmoid: bad arguments");
    HIP_TRY(c, hipSetDevice(c->device));
    launch_selftest_sigmoid(x, y, n, static_cast<hipStream_t>(stream));
    HIP_TRY(c, hipGetLastError());
    return SOUP_OK;
}

soup_status soup_selftest_uniform(soup_ctx* c, uint64_t seed, const uint32_t* pixel, const uint32_t* tri,
                                  uint32_t view_id, uint32_t step, float* u, int64_t n, void* stream) {
    if (!c) return SOUP_ERR_INVALID;
    if (n < 0 || (n > 0 && (!pixel || !tri || !u))) return fail(c, SOUP_ERR_INVALID, "selftest_uniform: bad arguments");
    HIP_TRY(c, hipSetDevice(c->device));
    launch_selftest_uniform(seed, pixel, tri, view_id, step, u, n, static_cast<hipStream_t>(stream));
    HIP_TRY(c, hipGetLastError());
    return SOUP_OK;
}

}  // extern "C"

// ---------------------------------------------------------------------------
// measured ceilings
// ---------------------------------------------------------------------------

soup_status soup_probe_copy(soup_ctx* c, const void* src, void* dst, int64_t bytes, void* stream) {
    if (!c) return SOUP_ERR_INVALID;
    c->err.clear();
    if (bytes < 0 || bytes % 16 != 0 || (bytes > 0 && (!src || !dst)) ||
        ((reinterpret_cast<uintptr_t>(src) | reinterpret_cast<uintptr_t>(dst)) & 15) != 0)
        return fail(c, SOUP_ERR_INVALID, "probe_copy: need 16-byte aligned buffers and a multiple of 16 bytes");
    HIP_TRY(c, hipSetDevice(c->device));
    soup::launch_probe_copy(static_cast<const float4*>(src), static_cast<float4*>(dst), bytes / 16, c->num_cus,
                            static_cast<hipStream_t>(stream));
    HIP_TRY(c, hipGetLastError());
    return SOUP_OK;
}

soup_status soup_probe_read(soup_ctx* c, const void* src, int64_t bytes, float* partial, int64_t n_partial,
                            void* stream) {
    if (!c) return SOUP_ERR_INVALID;
    c->err.clear();
    if (bytes < 0 || bytes % 16 != 0 || (bytes > 0 && (!src || !partial)) || n_partial < 1 ||
        (reinterpret_cast<uintptr_t>(src) & 15) != 0)
        return fail(c, SOUP_ERR_INVALID, "probe_read: need a 16-byte aligned buffer, a multiple of 16 bytes and "
                    "n_partial >= 1");
    HIP_TRY(c, hipSetDevice(c->device));
    soup::launch_probe_read(static_cast<const float4*>(src), bytes / 16, partial, n_partial,
                            static_cast<hipStream_t>(stream));
    HIP_TRY(c, hipGetLastError());
    return SOUP_OK;
}

soup_status soup_probe_atomic(soup_ctx* c, float* slots, int64_t n_slots, int64_t n_ops, void* stream) {
    if (!c) return SOUP_ERR_INVALID;
    c->err.clear();
    if (n_slots < 1 || n_ops < 0 || !slots) return fail(c, SOUP_ERR_INVALID, "probe_atomic: bad arguments");
    HIP_TRY(c, hipSetDevice(c->device));
    soup::launch_probe_atomic(slots, n_slots, n_ops, c->num_cus, static_cast<hipStream_t>(stream));
    HIP_TRY(c, hipGetLastError());
    return SOUP_OK;
}

soup_status soup_probe_fma(soup_ctx* c, float* out, int64_t n_threads, int32_t iters, void* stream) {
    if (!c) return SOUP_ERR_INVALID;
    c->err.clear();
    if (!out || n_threads < 256 || n_threads % 256 != 0 || n_threads / 256 > INT32_MAX || iters < 0 ||
        iters > (1 << 20))
        return fail(c, SOUP_ERR_INVALID, "probe_fma: n_threads a positive multiple of 256, 0 <= iters <= 2^20");
    HIP_TRY(c, hipSetDevice(c->device));
    soup::launch_probe_fma(out, n_threads, iters, static_cast<hipStream_t>(stream));
    HIP_TRY(c, hipGetLastError());
    return SOUP_OK;
}

soup_status soup_probe_mfma(soup_ctx* c, float* out, int64_t n_threads, int32_t iters, void* stream) {
    if (!c) return SOUP_ERR_INVALID;
    c->err.clear();
    if (!out || n_threads < 256 || n_threads % 256 != 0 || n_threads / 256 > INT32_MAX || iters < 0 ||
        iters > (1 << 18))
        return fail(c, SOUP_ERR_INVALID, "probe_mfma: n_threads a positive multiple of 256, 0 <= iters <= 2^18");
    HIP_TRY(c, hipSetDevice(c->device));
    soup::launch_probe_mfma(out, n_threads, iters, static_cast<hipStream_t>(stream));
    HIP_TRY(c, hipGetLastError());
    return SOUP_OK;
}
