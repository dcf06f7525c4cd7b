// dp.hip -- the strip sweep run on the sibling recurrences (DTW, edit
// distance, the indel distance that gives the LCS length), as tiles with FP64
// accumulators.  Section "Generalized Dynamic Programming Extensions" of the
// paper points out that such programs need only the cells above, to the left
// and up-left, so the band sweep carries over unchanged; only the cell update
// differs (lane_row_sibling in twed_device.h).
#include "dp_impl.h"

namespace twed {

hipError_t launch_dp(int rec, Prec prec, const CostParams &cp, int K, const WavefrontArgs &a, const TileArgs &t,
                     hipStream_t st)
{
    hipError_t e = hipErrorInvalidValue;
    if (prec == kF64) e = launch_dp_as<double>(rec, cp, K, a, t, st);
    else if (prec == kF32Acc64) e = launch_dp_as<float>(rec, cp, K, a, t, st);
    if (e != hipSuccess) return e;
    return launch_tile_edges(a.nA, a.nB, t, st);
}

size_t dp_scratch_bytes(int rec, Prec prec, const CostParams &cp, int K, int G)
{
    if (prec == kF64) return dp_scratch_as<double>(rec, cp, K, G);
    return prec == kF32Acc64 ? dp_scratch_as<float>(rec, cp, K, G) : (size_t)-1;
}

int dp_max_workers(int rec, Prec prec, const CostParams &cp, int K, int G)
{
    int per_cu = 0;
    if (prec == kF64) per_cu = dp_occupancy_as<double>(rec, cp, K, G);
    else if (prec == kF32Acc64) per_cu = dp_occupancy_as<float>(rec, cp, K, G);
    if (per_cu <= 0) return 0;
    int dev = 0, cus = 0;
    if (hipGetDevice(&dev) != hipSuccess) return 0;
    if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess) return 0;
    return per_cu * cus;
}

}  // namespace twed
