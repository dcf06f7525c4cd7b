// dp_f32.hip -- the sibling recurrences with FP32 costs (see dp.hip).
#include "dp_impl.h"

namespace twed {

template hipError_t launch_dp_as<float>(int, const CostParams &, int, const WavefrontArgs &, const TileArgs &,
                                        hipStream_t);
template size_t dp_scratch_as<float>(int, const CostParams &, int, int);
template int dp_occupancy_as<float>(int, const CostParams &, int, int);

}  // namespace twed
