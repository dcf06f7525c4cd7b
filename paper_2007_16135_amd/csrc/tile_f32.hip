// tile_f32.hip -- the tile sweep with FP32 costs (see tile.hip).
#include "tile_impl.h"

namespace twed {

template hipError_t launch_tile_as<float>(const CostParams &, int, const WavefrontArgs &, const TileArgs &, hipStream_t);
template size_t tile_scratch_as<float>(const CostParams &, int, int);
template int tile_occupancy_as<float>(const CostParams &, int, int);

}  // namespace twed
