// Definition of the per-(precision, kind) 3D deep-tile launcher; included only by
// the kernels_d3d_<kind>_<precision>.hip files.
#pragma once

#include "pf_deep3d.h"
#include "pf_deep3d_kind.h"

namespace pf {

template <typename T, int KIND>
hipError_t launch_deep3d_kind(const Launch &L, const StepArgs<T> &a, const DeepPlan &plan, bool red, hipStream_t s)
{
    hipError_t err = hipErrorInvalidValue;
    auto go = [&](auto rc, auto redc, auto tile) {
        constexpr int R = decltype(rc)::value;
        constexpr bool RED = decltype(redc)::value;
        using Tile = decltype(tile);
        using D = Deep3Shape<T, KIND, R, Tile::W, Tile::LZ>;
        if constexpr (2 * D::HS < Tile::LZ) {
            if (plan.waves < 1 || plan.waves > kDeep3Waves || plan.lds != D::LDS_PER_WAVE * plan.waves) return;
            hipLaunchKernelGGL((k_deep3d<T, KIND, R, Tile::W, Tile::LZ, Tile::EU, RED>), dim3((unsigned)plan.tiles),
                               dim3(64 * plan.waves), (size_t)plan.lds, s, a, plan.args3);
            err = hipGetLastError();
        }
    };
    dispatch_r(L.r, Deep3Radii{}, [&](auto rc) {
        constexpr int R = decltype(rc)::value;
        if (red) {
            if constexpr (deep3d_built<T, KIND, R, true>())
                plan.wide ? go(rc, std::true_type{}, Deep3Tall<T, KIND, R, true>{})
                          : go(rc, std::true_type{}, Deep3Flat<T, KIND, R, true>{});
        } else {
            plan.wide ? go(rc, std::false_type{}, Deep3Tall<T, KIND, R, false>{})
                      : go(rc, std::false_type{}, Deep3Flat<T, KIND, R, false>{});
        }
    });
    return err;
}

template <typename T, int KIND>
hipError_t launch_deep3d_batched_kind(const Launch &L, const BatchTable<T> &t, int32_t k, int32_t S, int32_t blocks,
                                      hipStream_t s)
{
    hipError_t err = hipErrorInvalidValue;
    dispatch_r(L.r, Deep3Radii{}, [&](auto rc) {
        constexpr int R = decltype(rc)::value;
        using V = Deep3Served<T, KIND, R>;
        using Tile = typename V::tile;
        constexpr size_t lds = V::waves * Deep3Shape<T, KIND, R, Tile::W, Tile::LZ>::LDS_PER_WAVE;
        if (S != V::steps) return;
        hipLaunchKernelGGL((k_deep3d_batched<T, KIND, R, Tile::W, Tile::LZ, Tile::EU>), dim3(blocks), dim3(64 * V::waves),
                           lds, s, t, k, S);
        err = hipGetLastError();
    });
    return err;
}

}  // namespace pf
