// tile_dirs.hip -- sweeps of blocks that also record the move into every cell
// (two bits per cell, for reading an alignment path back).  Kept apart from
// tile.hip: the recording code needs registers that the plain tile kernels
// then do not pay for.  Strips of one column per lane in groups of
// kResidentGroup.
#include "wavefront_impl.h"

#include <algorithm>
#include <type_traits>

namespace twed {

namespace {

template <typename CT, typename AT>
struct DirsBlock {
    const CT *rowsA, *rowsB;
    const Pair2<AT> *top, *left;
    Pair2<AT> *bnd, *dummy;
    uint32_t *flags, *ticket;
    AT *out;
    uint64_t *dirs;
    int nA, nB;
};

template <typename CT, typename AT>
struct DirsBlocks {
    DirsBlock<CT, AT> b[kMaxDirsBlocks];
};

// Workgroups (., y) sweep block y, each block with its own ticket, flags and
// boundary slots.  One block keeps 16 of 256 compute units busy (4,096 columns)
// and takes what its chain of diagonals takes, so the blocks a path may cross
// next run in the same launch beside it: as launches of their own on four
// streams, four ran at once at most (one hardware queue each), the walk among
// them.
template <typename CT, typename AT, int DIMT, int PM, int REC>
__global__ __launch_bounds__((kWave * kResidentGroup<CT, DIMT, PM>)) void dirs_kernel(DirsBlocks<CT, AT> blocks,
                                                                              CostArgs<CT> ca, int sub_shift)
{
    constexpr int G = kResidentGroup<CT, DIMT, PM>;
    __shared__ GroupShared<CT, AT, DIMT, G> sh;
    const DirsBlock<CT, AT> &d = blocks.b[blockIdx.y];
    const int nStrips = (d.nB + kWave - 1) / kWave;
    TileIO<AT> io{};
    io.top = d.top;
    io.left = d.left;
    io.dummy = d.dummy;
    io.dirs = d.dirs;
    claim_groups<G>(sh, d.ticket, nStrips, [&](int w, int g, int s) {
        sweep_strip<CT, AT, DIMT, PM, 1, G, false, true, REC, true>(
            sh, w, g, s, s * kWave, d.rowsA, d.rowsB, d.nA, d.nB, ca, d.bnd, d.flags, d.ticket + 1, nStrips, CT(0),
            d.out, nullptr, sub_shift, io);
    });
}

template <int REC, int DIMT>
constexpr bool kRecDim = REC == kRecTwed || REC == kRecDtw || DIMT == 1;

// fn.template operator()<CT, AT, DIMT, PM, REC>() for a compiled configuration
// (FP64 accumulators).
template <typename Fn>
hipError_t by_config(int rec, Prec prec, const CostParams &cp, Fn &&fn)
{
    if (prec != kF64 && prec != kF32Acc64) return hipErrorInvalidValue;
    auto with_rec = [&]<int REC>() -> hipError_t {
        return by_prec(prec, cp.dimt, cp.pm, [&]<typename CT, typename AT, int DIMT, int PM>() -> hipError_t {
            if constexpr (!std::is_same_v<AT, double> || !kRecDim<REC, DIMT>) return hipErrorInvalidValue;
            else return fn.template operator()<CT, AT, DIMT, PM, REC>();
        });
    };
    switch (rec) {
    case kRecTwed: return with_rec.template operator()<kRecTwed>();
    case kRecDtw: return with_rec.template operator()<kRecDtw>();
    case kRecEdit: return with_rec.template operator()<kRecEdit>();
    case kRecIndel: return with_rec.template operator()<kRecIndel>();
    default: return hipErrorInvalidValue;
    }
}

}  // namespace

hipError_t launch_dirs(int rec, Prec prec, const CostParams &cp, const DirsArgs *blocks, int n, hipStream_t st)
{
    if (n <= 0) return hipSuccess;
    if (n > kMaxDirsBlocks) return hipErrorInvalidValue;
    return by_config(rec, prec, cp, [&]<typename CT, typename AT, int DIMT, int PM, int REC>() -> hipError_t {
        constexpr int G = kResidentGroup<CT, DIMT, PM>;
        DirsBlocks<CT, AT> g{};
        int64_t groups = 0;
        for (int i = 0; i < n; ++i) {
            const DirsArgs &a = blocks[i];
            const int64_t strips = (a.nB + kWave - 1) / kWave;
            groups = std::max(groups, (strips + G - 1) / G);
            g.b[i] = DirsBlock<CT, AT>{(const CT *)a.rowsA,     (const CT *)a.rowsB, (const Pair2<AT> *)a.top,
                                       (const Pair2<AT> *)a.left, (Pair2<AT> *)a.bnd,  (Pair2<AT> *)a.dummy,
                                       a.flags,                 a.ticket,            (AT *)a.out,
                                       (uint64_t *)a.dirs,      (int)a.nA,           (int)a.nB};
        }
        // (workgroups claim groups until none is left: a grid smaller than the
        // groups of one very wide block is enough)
        const int grid = (int)std::min<int64_t>(groups, 1024);
        hipLaunchKernelGGL((dirs_kernel<CT, AT, DIMT, PM, REC>), dim3(grid, n), dim3(kWave * G), 0, st, g,
                           CostArgs<CT>::make(cp), kSubShift);
        return hipGetLastError();
    });
}

}  // namespace twed
