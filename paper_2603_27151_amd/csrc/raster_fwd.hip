// Forward raster dispatch over the compiled MLP shapes and tile sizes (the
// kernel is in raster_fwd_impl.hpp, instantiated once per shape and tile in
// fwd_*.hip so that the units compile in parallel).
#include "raster_fwd_impl.hpp"

namespace soup {

void launch_raster_fwd_k8_16_1_t8(const RasterArgs& a, hipStream_t s);
void launch_raster_fwd_k8_16_1_t16(const RasterArgs& a, hipStream_t s);
void launch_raster_fwd_k8_16_1_t32(const RasterArgs& a, hipStream_t s);
void launch_raster_fwd_k16_32_2_t8(const RasterArgs& a, hipStream_t s);
void launch_raster_fwd_k16_32_2_t16(const RasterArgs& a, hipStream_t s);
void launch_raster_fwd_k16_32_2_t32(const RasterArgs& a, hipStream_t s);
void launch_raster_fwd_k32_64_2_t8(const RasterArgs& a, hipStream_t s);
void launch_raster_fwd_k32_64_2_t16(const RasterArgs& a, hipStream_t s);
void launch_raster_fwd_k32_64_2_t32(const RasterArgs& a, hipStream_t s);

void launch_raster_fwd_paper_t8(const RasterArgs& a, hipStream_t s);
void launch_raster_fwd_paper_t16(const RasterArgs& a, hipStream_t s);
void launch_raster_fwd_paper_t32(const RasterArgs& a, hipStream_t s);
int raster_fwd_per_cu_paper_t8(int region);
int raster_fwd_per_cu_paper_t16(int region);
int raster_fwd_per_cu_paper_t32(int region);

void launch_raster_replay_t8(const RasterArgs& a, hipStream_t s);
void launch_raster_replay_t16(const RasterArgs& a, hipStream_t s);
void launch_raster_replay_t32(const RasterArgs& a, hipStream_t s);
int raster_replay_per_cu_t8(int region);
int raster_replay_per_cu_t16(int region);
int raster_replay_per_cu_t32(int region);

int raster_fwd_per_cu_k8_16_1_t8(int region);
int raster_fwd_per_cu_k8_16_1_t16(int region);
int raster_fwd_per_cu_k8_16_1_t32(int region);
int raster_fwd_per_cu_k16_32_2_t8(int region);
int raster_fwd_per_cu_k16_32_2_t16(int region);
int raster_fwd_per_cu_k16_32_2_t32(int region);
int raster_fwd_per_cu_k32_64_2_t8(int region);
int raster_fwd_per_cu_k32_64_2_t16(int region);
int raster_fwd_per_cu_k32_64_2_t32(int region);

void launch_raster_fwd(const RasterArgs& a, int tile, MlpKind k, hipStream_t s) {
    switch (k) {
        case MlpKind::k8_16_1:
            if (tile == 8) launch_raster_fwd_k8_16_1_t8(a, s);
            else if (tile == 32) launch_raster_fwd_k8_16_1_t32(a, s);
            else launch_raster_fwd_k8_16_1_t16(a, s);
            break;
        case MlpKind::k16_32_2:
            if (tile == 8) launch_raster_fwd_k16_32_2_t8(a, s);
            else if (tile == 32) launch_raster_fwd_k16_32_2_t32(a, s);
            else launch_raster_fwd_k16_32_2_t16(a, s);
            break;
        case MlpKind::k32_64_2:
            if (tile == 8) launch_raster_fwd_k32_64_2_t8(a, s);
            else if (tile == 32) launch_raster_fwd_k32_64_2_t32(a, s);
            else launch_raster_fwd_k32_64_2_t16(a, s);
            break;
        case MlpKind::kPaper:
            if (tile == 8) launch_raster_fwd_paper_t8(a, s);
            else if (tile == 32) launch_raster_fwd_paper_t32(a, s);
            else launch_raster_fwd_paper_t16(a, s);
            break;
        case MlpKind::kReplay:
            if (tile == 8) launch_raster_replay_t8(a, s);
            else if (tile == 32) launch_raster_replay_t32(a, s);
            else launch_raster_replay_t16(a, s);
            break;
        default: break;
    }
}

size_t fwd_weights_bytes(MlpKind k) {
    switch (k) {
        case MlpKind::k16_32_2: return FwdWeights<MlpShape<16, 32, 2>>::kGroups * 16;
        case MlpKind::k32_64_2: return FwdWeights<MlpShape<32, 64, 2>>::kGroups * 16;
        default: return 0;
    }
}

template <class S>
static void launch_begin_s(const ZeroList& z, const SceneDesc* scenes, int n_scenes, float* weights, hipStream_t s) {
    int64_t n = 0;
    for (int r = 0; r < z.k; ++r) n += z.n[r];
    const int64_t zb = n + 1023 < int64_t(4096) * 1024 ? (n + 1023) / 1024 : 4096;
    hipLaunchKernelGGL(begin_kernel<S>, dim3(static_cast<unsigned>(zb + 8 * n_scenes)), dim3(256), 0, s, z,
                       static_cast<int>(zb), scenes, weights);
}

void launch_begin(const ZeroList& z, const SceneDesc* scenes, int n_scenes, MlpKind k, float* weights, hipStream_t s) {
    switch (k) {
        case MlpKind::k16_32_2: launch_begin_s<MlpShape<16, 32, 2>>(z, scenes, n_scenes, weights, s); break;
        case MlpKind::k32_64_2: launch_begin_s<MlpShape<32, 64, 2>>(z, scenes, n_scenes, weights, s); break;
        default: launch_zero(z, s); break;
    }
}

// Resident single-wave workgroups per CU of the forward for this shape, tile and region side.
int raster_fwd_blocks_per_cu(int tile, MlpKind k, int region) {
    switch (k) {
        case MlpKind::k8_16_1:
            return tile == 8 ? raster_fwd_per_cu_k8_16_1_t8(region) : tile == 32 ? raster_fwd_per_cu_k8_16_1_t32(region) : raster_fwd_per_cu_k8_16_1_t16(region);
        case MlpKind::k16_32_2:
            return tile == 8 ? raster_fwd_per_cu_k16_32_2_t8(region) : tile == 32 ? raster_fwd_per_cu_k16_32_2_t32(region) : raster_fwd_per_cu_k16_32_2_t16(region);
        case MlpKind::k32_64_2:
            return tile == 8 ? raster_fwd_per_cu_k32_64_2_t8(region) : tile == 32 ? raster_fwd_per_cu_k32_64_2_t32(region) : raster_fwd_per_cu_k32_64_2_t16(region);
        case MlpKind::kPaper:
            return tile == 8 ? raster_fwd_per_cu_paper_t8(region) : tile == 32 ? raster_fwd_per_cu_paper_t32(region) : raster_fwd_per_cu_paper_t16(region);
        case MlpKind::kReplay:
            return tile == 8 ? raster_replay_per_cu_t8(region) : tile == 32 ? raster_replay_per_cu_t32(region) : raster_replay_per_cu_t16(region);
        default: return 1;
    }
}

}  // namespace soup
