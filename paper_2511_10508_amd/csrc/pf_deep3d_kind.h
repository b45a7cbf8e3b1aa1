// Shapes and launchers of the 3D deep-tile kernels: one (precision, kind) pair
// each, instantiated in kernels_d3d_<kind>_<precision>.hip; kernels_deep3d.hip
// plans and dispatches.
#pragma once

#include "pf_dispatch.h"
#include "pf_internal.h"

namespace pf {

using Deep3Radii = RList<1, 2>;

// W values per lane, LZ planes, EU waves per SIMD that the registers must allow.
template <int W_, int LZ_, int EU_>
struct Deep3Tile {
    static constexpr int W = W_, LZ = LZ_, EU = EU_;
};
// Eight planes, two values per lane (four measured slower at either precision:
// Gray-Scott FP32 96^3 8.8 against 5.4 us a step).  FP32 without reductions
// keeps four waves per SIMD, which costs it at most a few spilled registers
// (192^3 Gray-Scott p4 38 against 42 us); with reductions or in FP64 that spills
// hundreds of bytes (96^3 Allen-Cahn FP64 p4 with reductions 66 against 15 us).
template <typename T, int KIND, int R, bool RED>
using Deep3Flat = Deep3Tile<2, 8, (sizeof(T) == 4 && !RED) ? 4 : 2>;
// Twelve planes: more steps per launch for r = 1, and the least that a
// Cahn-Hilliard step with r = 2 (halo 4) can do with; sixteen for FP32 there
// (96^3 12.5 against 16.5 us).
// FP64 two-field kernels with reductions stay flat (a tall Model C brick spills
// 880 B a lane, and no grid below the size limit planned one).
template <typename T, int KIND, int R, bool RED>
using Deep3Tall =
    std::conditional_t<sizeof(T) == 8 && RED && (KIND == kGS || KIND == kMC), Deep3Flat<T, KIND, R, RED>,
                       Deep3Tile<2, (KIND == kCH && R == 2 && sizeof(T) == 4 && !RED) ? 16 : 12, 2>>;
// FP64 two-field kernels with r = 2 and reductions spill a kilobyte a lane
// (96^3 66 us a step against 30 us marching): not built.
template <typename T, int KIND, int R, bool RED>
constexpr bool deep3d_built()
{
    return !(sizeof(T) == 8 && R == 2 && RED && KIND != kAC);
}

// The batched launches: flat bricks of four waves (32 x 16 x 8 sites, 28 x 12 x 4
// written), tall ones of six for Cahn-Hilliard with r = 2.  Two fields with r = 2
// keep two waves per SIMD: the arguments of a table entry stay in registers, and
// at four they spill (132-388 B a lane).
template <typename T, int KIND, int R>
struct Deep3Served {
    using tile = std::conditional_t<
        KIND == kCH && R == 2, Deep3Tall<T, KIND, R, false>,
        std::conditional_t<(KIND == kGS || KIND == kMC) && R == 2, Deep3Tile<2, 8, 2>, Deep3Flat<T, KIND, R, false>>>;
    static constexpr int waves = KIND == kCH && R == 2 ? 6 : 4;
    static constexpr int steps = KIND != kCH && R == 1 ? 2 : 1;
};

template <typename T, int KIND>
hipError_t launch_deep3d_batched_kind(const Launch &L, const BatchTable<T> &t, int32_t k, int32_t S, int32_t blocks,
                                      hipStream_t s);
template <typename T, int KIND>
hipError_t launch_deep3d_kind(const Launch &L, const StepArgs<T> &a, const DeepPlan &plan, bool red, hipStream_t s);

}  // namespace pf
