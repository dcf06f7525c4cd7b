// dp_impl.h -- the sibling recurrences' launches for one cost type.  FP64 costs
// are compiled in dp.hip and FP32 costs in dp_f32.hip.
#pragma once

#include "wavefront_impl.h"

#include <type_traits>

namespace twed {

// Strip widths and group sizes compiled for the sibling recurrences.
template <int DIMT, int K>
constexpr bool kDpCompiled = kStripCompiled<DIMT, K>;

template <int REC, int DIMT>
constexpr bool kDpDim = REC == kRecDtw || DIMT == 1;

template <typename CT, typename AT, int DIMT, int PM, int K, int G, int REC>
hipError_t launch_dp_kg(const WavefrontArgs &a, const TileIO<AT> &io, const CostParams &cp, hipStream_t st)
{
    hipLaunchKernelGGL((wavefront_kernel<CT, AT, DIMT, PM, K, G, false, true, REC>), dim3(a.grid), dim3(kWave * G), 0,
                       st, (const CT *)a.rowsA, (const CT *)a.rowsB, (int)a.nA, (int)a.nB, CostArgs<CT>::make(cp),
                       (Pair2<AT> *)a.bnd, a.flags, a.ticket, a.ticket + 1, (int)a.nStrips, (const CT *)a.beta,
                       (AT *)a.out, nullptr, a.sub_shift, io);
    return hipGetLastError();
}

template <typename Fn>
hipError_t by_rec(int rec, Fn &&fn)
{
    switch (rec) {
    case kRecDtw: return fn.template operator()<kRecDtw>();
    case kRecEdit: return fn.template operator()<kRecEdit>();
    case kRecIndel: return fn.template operator()<kRecIndel>();
    default: return hipErrorInvalidValue;
    }
}

// Calls fn.template operator()<CT, AT, DIMT, PM, K, G, REC>() for a compiled
// configuration of cost type COST, else returns hipErrorInvalidValue.
template <typename COST, typename Fn>
hipError_t dp_by_config(int rec, const CostParams &cp, int K, int G, Fn &&fn)
{
    return by_rec(rec, [&]<int REC>() -> hipError_t {
        return by_prec(std::is_same_v<COST, double> ? kF64 : kF32Acc64, cp.dimt, cp.pm,
                       [&]<typename CT, typename AT, int DIMT, int PM>() -> hipError_t {
            if constexpr (!std::is_same_v<AT, double> || !std::is_same_v<CT, COST> || !kDpDim<REC, DIMT>) {
                return hipErrorInvalidValue;
            } else {
                auto withK = [&]<int KK>() -> hipError_t {
                    if constexpr (!kDpCompiled<DIMT, KK>) {
                        return hipErrorInvalidValue;
                    } else {
                        constexpr int R = kResidentGroup<CT, DIMT, PM>;
                        if (G == R) return fn.template operator()<CT, AT, DIMT, PM, KK, R, REC>();
                        if (G == 8) return fn.template operator()<CT, AT, DIMT, PM, KK, 8, REC>();
                        return hipErrorInvalidValue;
                    }
                };
                switch (K) {
                case 1: return withK.template operator()<1>();
                case 2: return withK.template operator()<2>();
                case 4: return withK.template operator()<4>();
                case 8: return withK.template operator()<8>();
                default: return hipErrorInvalidValue;
                }
            }
        });
    });
}

template <typename COST>
hipError_t launch_dp_as(int rec, const CostParams &cp, int K, const WavefrontArgs &a, const TileArgs &t, hipStream_t st)
{
    return dp_by_config<COST>(rec, cp, K, a.group,
                              [&]<typename CT, typename AT, int DIMT, int PM, int KK, int G, int REC>() -> hipError_t {
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
                                  return launch_dp_kg<CT, AT, DIMT, PM, KK, G, REC>(a, io, cp, st);
                              });
}

template <typename COST>
size_t dp_scratch_as(int rec, const CostParams &cp, int K, int G)
{
    size_t bytes = (size_t)-1;
    (void)dp_by_config<COST>(rec, cp, K, G, [&]<typename CT, typename AT, int DIMT, int PM, int KK, int GG, int REC>() {
        bytes = scratch_kg<CT, AT, DIMT, PM, KK, GG, true, REC>();
        return hipSuccess;
    });
    return bytes;
}

template <typename COST>
int dp_occupancy_as(int rec, const CostParams &cp, int K, int G)
{
    int per_cu = 0;
    (void)dp_by_config<COST>(rec, cp, K, G, [&]<typename CT, typename AT, int DIMT, int PM, int KK, int GG, int REC>() {
        per_cu = occupancy_kg<CT, AT, DIMT, PM, KK, GG, true, REC>();
        return hipSuccess;
    });
    return per_cu;
}

extern template hipError_t launch_dp_as<float>(int, const CostParams &, int, const WavefrontArgs &, const TileArgs &,
                                               hipStream_t);
extern template size_t dp_scratch_as<float>(int, const CostParams &, int, int);
extern template int dp_occupancy_as<float>(int, const CostParams &, int, int);

}  // namespace twed
