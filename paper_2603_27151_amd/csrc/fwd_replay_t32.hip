// The raster walk with the winners known (a backward without the forward's log), 32x32 tiles.
#include "raster_fwd_impl.hpp"

namespace soup {

void launch_raster_replay_t32(const RasterArgs& a, hipStream_t s) { launch_fwd_t<32, ReplayWalk>(a, s); }
int raster_replay_per_cu_t32(int region) { return fwd_blocks_per_cu<32, ReplayWalk>(region); }

}  // namespace soup
