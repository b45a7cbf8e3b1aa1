// Definition of the per-(precision, kind) deep-tile launcher; included only by
// the kernels_d2d_<kind>_<precision>.hip files.
#pragma once

#include "pf_deep2d.h"
#include "pf_deep2d_kind.h"

namespace pf {

template <typename T, int KIND>
hipError_t launch_deep2d_kind(const Launch &L, const StepArgs<T> &a, const DeepPlan &plan, bool red, hipStream_t s)
{
    hipError_t err = hipErrorInvalidValue;
    auto go = [&](auto kern, auto tile, int per_wave) {
        using Tile = decltype(tile);
        if (plan.waves < 1 || plan.waves > Tile::NWM || plan.lds != per_wave * plan.waves) return;
        hipLaunchKernelGGL(kern, dim3((unsigned)plan.tiles), dim3(64 * plan.waves), (size_t)plan.lds, s, a, plan.args);
        err = hipGetLastError();
    };
    auto shape = [&](auto rc, auto redc, auto tile) {
        constexpr int R = decltype(rc)::value;
        constexpr bool RED = decltype(redc)::value;
        using Tile = decltype(tile);
        go(k_deep2d<T, KIND, R, Tile::W, Tile::LR, Tile::NWM, RED>, tile,
           DeepShape<T, KIND, R, Tile::W, Tile::LR>::LDS_PER_WAVE);
    };
    dispatch_r(L.r, DeepRadii{}, [&](auto rc) {
        constexpr int R = decltype(rc)::value;
        if (red)
            plan.wide ? shape(rc, std::true_type{}, DeepWide<T, KIND, R, true>{})
                      : shape(rc, std::true_type{}, DeepNarrow<T, KIND, R, true>{});
        else
            plan.wide ? shape(rc, std::false_type{}, DeepWide<T, KIND, R, false>{})
                      : shape(rc, std::false_type{}, DeepNarrow<T, KIND, R, false>{});
    });
    return err;
}

template <typename T, int KIND>
hipError_t launch_deep2d_batched_kind(const Launch &L, const BatchTable<T> &t, int32_t k, int32_t S, int32_t blocks,
                                      hipStream_t s)
{
    hipError_t err = hipErrorInvalidValue;
    dispatch_r(L.r, DeepRadii{}, [&](auto rc) {
        constexpr int R = decltype(rc)::value;
        using Tile = DeepServed<T, KIND, R>;
        constexpr size_t lds = Tile::NWM * DeepShape<T, KIND, R, Tile::W, Tile::LR>::LDS_PER_WAVE;
        if (S != deep_served_steps(KIND, R)) return;
        hipLaunchKernelGGL((k_deep2d_batched<T, KIND, R, Tile::W, Tile::LR, Tile::NWM>), dim3(blocks),
                           dim3(64 * Tile::NWM), lds, s, t, k, S);
        err = hipGetLastError();
    });
    return err;
}

}  // namespace pf
