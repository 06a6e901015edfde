// The raster walk with the winners known (a backward without the forward's log), 8x8 tiles.
#include "raster_fwd_impl.hpp"

namespace soup {

void launch_raster_replay_t8(const RasterArgs& a, hipStream_t s) { launch_fwd_t<8, ReplayWalk>(a, s); }
int raster_replay_per_cu_t8(int region) { return fwd_blocks_per_cu<8, ReplayWalk>(region); }

}  // namespace soup
