// tile_impl.h -- the tile sweep's launches for one cost type.  FP64 costs are
// compiled in tile.hip and FP32 costs in tile_f32.hip (one source took 20
// minutes).
#pragma once

#include "wavefront_impl.h"

#include <type_traits>

namespace twed {

template <typename CT, typename AT, int DIMT, int PM, int K, int G>
hipError_t launch_tile_kg(const WavefrontArgs &a, const TileIO<AT> &io, const CostParams &cp, hipStream_t st)
{
    hipLaunchKernelGGL((wavefront_kernel<CT, AT, DIMT, PM, K, G, false, true>), dim3(a.grid), dim3(kWave * G), 0, st,
                       (const CT *)a.rowsA, (const CT *)a.rowsB, (int)a.nA, (int)a.nB, CostArgs<CT>::make(cp),
                       (Pair2<AT> *)a.bnd, a.flags, a.ticket, a.ticket + 1, (int)a.nStrips, (const CT *)a.beta,
                       (AT *)a.out, nullptr, a.sub_shift, io);
    return hipGetLastError();
}

template <typename CT, typename AT, int DIMT, int PM, int K>
hipError_t launch_tile_k(const WavefrontArgs &a, const TileIO<AT> &io, const CostParams &cp, hipStream_t st)
{
    constexpr int G = kResidentGroup<CT, DIMT, PM>;
    if (a.group == G) return launch_tile_kg<CT, AT, DIMT, PM, K, G>(a, io, cp, st);
    if (a.group == 8) return launch_tile_kg<CT, AT, DIMT, PM, K, 8>(a, io, cp, st);
    return hipErrorInvalidValue;
}

template <typename AT>
TileIO<AT> typed(const TileArgs &t)
{
    TileIO<AT> io{};
    io.top = (const Pair2<AT> *)t.top;
    io.left = (const Pair2<AT> *)t.left;
    io.bottom = (Pair2<AT> *)t.bottom;
    io.right = (Pair2<AT> *)t.right;
    io.ckrow = (Pair2<AT> *)t.ckrow;
    io.ckcol = (Pair2<AT> *)t.ckcol;
    io.dummy = (Pair2<AT> *)t.dummy;
    io.ck_rows = t.ck_rows;
    io.ck_cols = t.ck_cols;
    return io;
}

// fn.template operator()<CT, AT, DIMT, PM, K>() for a compiled configuration of
// cost type COST (FP64 accumulators; G = kResidentGroup or 8).
template <typename COST, typename Fn>
hipError_t tile_by_config(const CostParams &cp, int K, Fn &&fn)
{
    return by_prec(std::is_same_v<COST, double> ? kF64 : kF32Acc64, cp.dimt, cp.pm,
                   [&]<typename CT, typename AT, int DIMT, int PM>() -> hipError_t {
        if constexpr (!std::is_same_v<AT, double> || !std::is_same_v<CT, COST>) {
            return hipErrorInvalidValue;
        } else {
            switch (K) {
            case 1: return fn.template operator()<CT, AT, DIMT, PM, 1>();
            case 2: return fn.template operator()<CT, AT, DIMT, PM, 2>();
            case 4:
                if constexpr (kStripCompiled<DIMT, 4>) return fn.template operator()<CT, AT, DIMT, PM, 4>();
                return hipErrorInvalidValue;
            case 8:
                if constexpr (kStripCompiled<DIMT, 8>) return fn.template operator()<CT, AT, DIMT, PM, 8>();
                return hipErrorInvalidValue;
            default: return hipErrorInvalidValue;
            }
        }
    });
}

template <typename COST>
hipError_t launch_tile_as(const CostParams &cp, int K, const WavefrontArgs &a, const TileArgs &t, hipStream_t st)
{
    return tile_by_config<COST>(cp, K, [&]<typename CT, typename AT, int DIMT, int PM, int KK>() -> hipError_t {
        return launch_tile_k<CT, AT, DIMT, PM, KK>(a, typed<AT>(t), cp, st);
    });
}

template <typename COST>
size_t tile_scratch_as(const CostParams &cp, int K, int G)
{
    size_t bytes = (size_t)-1;
    (void)tile_by_config<COST>(cp, K, [&]<typename CT, typename AT, int DIMT, int PM, int KK>() -> hipError_t {
        constexpr int R = kResidentGroup<CT, DIMT, PM>;
        if (G == R) bytes = scratch_kg<CT, AT, DIMT, PM, KK, R, true>();
        else if (G == 8) bytes = scratch_kg<CT, AT, DIMT, PM, KK, 8, true>();
        return hipSuccess;
    });
    return bytes;
}

template <typename COST>
int tile_occupancy_as(const CostParams &cp, int K, int G)
{
    int per_cu = 0;
    (void)tile_by_config<COST>(cp, K, [&]<typename CT, typename AT, int DIMT, int PM, int KK>() -> hipError_t {
        constexpr int R = kResidentGroup<CT, DIMT, PM>;
        if (G == R) per_cu = occupancy_kg<CT, AT, DIMT, PM, KK, R, true>();
        else if (G == 8) per_cu = occupancy_kg<CT, AT, DIMT, PM, KK, 8, true>();
        return hipSuccess;
    });
    return per_cu;
}

extern template hipError_t launch_tile_as<float>(const CostParams &, int, const WavefrontArgs &, const TileArgs &,
                                                 hipStream_t);
extern template size_t tile_scratch_as<float>(const CostParams &, int, int);
extern template int tile_occupancy_as<float>(const CostParams &, int, int);

}  // namespace twed
