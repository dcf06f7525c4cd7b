// tile.hip -- the sweep of one rectangular block of the DP matrix.
//
// The paper's section "Improved Time Warp Edit Distance" keeps only the band
// of live diagonals; a row or a column of (DP, X = DP + e) cells is likewise
// the whole state the rest of the program needs.  The tile sweep is the
// strip pipeline of wavefront.hip started from a given top row and left
// column instead of the pad row and column, and it can hand back its bottom
// row and right column, checkpoint rows and columns at fixed intervals.
// Tiles in dependency order reproduce the
// pair sweep exactly: every cell is evaluated by the same lane code from the
// same operands.
//
// Tiles run with FP64 accumulators only (F64 and F32 costs with F64
// accumulators), where no cost offset is applied.
#include "tile_impl.h"

namespace twed {

namespace {

// Cell 0 of each output row (column 0 of the block) and of each output
// column (row 0 of the block) is not on the strips: it is copied from the
// left column and the top row, or is the +inf pad cell.
__global__ void tile_edges_kernel(TileArgs t, int64_t nA, int64_t nB)
{
    typedef Pair2<double> C;
    const C inf{__builtin_inf(), __builtin_inf()};
    const C *top = (const C *)t.top, *left = (const C *)t.left;
    const int64_t nr = t.ckrow ? (nA - 1) / t.ck_rows : 0;   // checkpoint rows below nA
    const int64_t nc = t.ckcol ? (nB - 1) / t.ck_cols : 0;   // checkpoint columns left of nB
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < nr + nc + 2;
         i += (int64_t)gridDim.x * blockDim.x) {
        if (i == 0) {
            if (t.bottom) ((C *)t.bottom)[0] = left ? left[nA] : inf;
        } else if (i == 1) {
            if (t.right) ((C *)t.right)[0] = top ? top[nB] : inf;
        } else if (i - 2 < nr) {
            const int64_t r = (i - 1) * t.ck_rows;
            ((C *)t.ckrow)[(i - 2) * (nB + 1)] = left ? left[r] : inf;
        } else {
            const int64_t k = i - 2 - nr;
            const int64_t c = (k + 1) * t.ck_cols;
            ((C *)t.ckcol)[k * (nA + 1)] = top ? top[c] : inf;
        }
    }
}

}  // namespace

hipError_t launch_tile(Prec prec, const CostParams &cp, int K, const WavefrontArgs &a, const TileArgs &t,
                       hipStream_t st)
{
    hipError_t e = hipErrorInvalidValue;
    if (prec == kF64) e = launch_tile_as<double>(cp, K, a, t, st);
    else if (prec == kF32Acc64) e = launch_tile_as<float>(cp, K, a, t, st);
    if (e != hipSuccess) return e;
    return launch_tile_edges(a.nA, a.nB, t, st);
}

hipError_t launch_tile_edges(int64_t nA, int64_t nB, const TileArgs &t, hipStream_t st)
{
    if (!(t.bottom || t.right || t.ckrow || t.ckcol)) return hipSuccess;
    hipLaunchKernelGGL(tile_edges_kernel, dim3(64), dim3(256), 0, st, t, nA, nB);
    return hipGetLastError();
}

size_t tile_scratch_bytes(Prec prec, const CostParams &cp, int K, int G)
{
    if (prec == kF64) return tile_scratch_as<double>(cp, K, G);
    return prec == kF32Acc64 ? tile_scratch_as<float>(cp, K, G) : (size_t)-1;
}

int tile_max_workers(Prec prec, const CostParams &cp, int K, int G)
{
    int per_cu = 0;
    if (prec == kF64) per_cu = tile_occupancy_as<double>(cp, K, G);
    else if (prec == kF32Acc64) per_cu = tile_occupancy_as<float>(cp, K, G);
    if (per_cu <= 0) return 0;
    int dev = 0, cus = 0;
    if (hipGetDevice(&dev) != hipSuccess) return 0;
    if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess) return 0;
    return per_cu * cus;
}

}  // namespace twed
