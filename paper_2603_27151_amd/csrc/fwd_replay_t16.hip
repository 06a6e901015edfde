// The raster walk with the winners known (a backward without the forward's log), 16x16 tiles.
#include "raster_fwd_impl.hpp"

namespace soup {

void launch_raster_replay_t16(const RasterArgs& a, hipStream_t s) { launch_fwd_t<16, ReplayWalk>(a, s); }
int raster_replay_per_cu_t16(int region) { return fwd_blocks_per_cu<16, ReplayWalk>(region); }

}  // namespace soup
